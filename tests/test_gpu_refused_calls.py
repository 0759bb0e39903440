"""What the host does when the HIP runtime refuses a call in the middle of a rollout: a refused launch is an error of the call (it
would otherwise return the bytes of an earlier one); where there is no pinned memory a continuous rollout does without; an error
that somebody else has left behind is no error of the call.  Each case is a process of its own, whose calls of the runtime go through
hip_refusals.c; nothing that is refused reaches the GPU."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path[:0] = [sys.argv[2], sys.argv[2] + "/tests"]
import numpy as np
from paper_2602_02192_amd import echo, synth
from gpu_util import make_ctx

shape, P, G, new = synth.TINY, 6, 2, 7
blob = synth.make_weights(shape, 0)
prompts, lens = synth.make_prompts(shape.vocab, P, 9, seed=1)
forced = np.random.default_rng(2).integers(0, shape.vocab, size=(P * G, new)).astype(np.int32)
stop = np.random.default_rng(3).integers(1, new + 1, P * G).astype(np.int32)

def run(ctx):
    return ctx.rollout(prompts, lens, G, new, 1.0, 4, stop_lens=stop, forced=forced, continuous=True)

ref_ctx = make_ctx(shape, 4, 9 + new, blob)
ref = run(ref_ctx)
"""


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("shim") / "hip_refusals.so")
    subprocess.check_call(["gcc", "-O2", "-Wall", "-shared", "-fPIC", "-o", lib, os.path.join(HERE, "hip_refusals.c"), "-ldl"])

    def run(body):
        r = subprocess.run([sys.executable, "-c", CHILD + body, lib, os.path.dirname(HERE)], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0 and r.stdout.strip().endswith("as expected"), r.stdout[-2000:] + r.stderr[-2000:]
    return run


@pytest.mark.parametrize("kernel", ["rows_to_host_kernel", "rows_from_host_kernel", "records_to_host_kernel", "records_begin_kernel"])
def test_a_refused_hand_over_is_an_error(child, kernel):
    """The first, the second and the last launch of the kernel in a call."""
    child(f"""
ctx = make_ctx(shape, 4, 9 + new, blob)
shim.hip_refuse(b"{kernel}", 1 << 30)
run(ctx)
n = shim.hip_seen()
assert n > 2
for after in (0, 1, n - 1):
    shim.hip_refuse(b"{kernel}", after)
    try:
        run(ctx)
    except echo.EchoError as e:
        assert e.code == echo.ECHO_EHIP and shim.hip_refused(), e
    else:
        raise SystemExit(f"succeeded with launch {{after}} of {{n}} refused")
    again = run(ctx)    # and the context is as good as before
    assert all(np.array_equal(again[k], ref[k]) for k in ("tokens", "logprobs", "lens", "versions"))
print("as expected")
""")


@pytest.mark.parametrize("kernel", ["dbg_gemm_kernel", "dbg_attention_kernel", "dbg_sample_kernel"])
@pytest.mark.parametrize("continuous", [False, True])
def test_a_refused_launch_of_a_step_is_an_error(child, kernel, continuous):
    """A launch in the middle of the call and the last one; sequences that all start together, and refilled ones."""
    child(f"""
slots = 4 if {continuous} else P * G
ctx = make_ctx(shape, slots, 9 + new, blob)
go = lambda: ctx.rollout(prompts, lens, G, new, 1.0, 4, stop_lens=stop, forced=forced, continuous={continuous})
shim.hip_refuse(b"{kernel}", 1 << 30)
want = go()
n = shim.hip_seen()
for after in (n // 2, n - 1):
    shim.hip_refuse(b"{kernel}", after)
    try:
        go()
    except echo.EchoError as e:
        assert e.code == echo.ECHO_EHIP and shim.hip_refused(), e
    else:
        raise SystemExit(f"succeeded with launch {{after}} of {{n}} refused")
    again = go()
    assert all(np.array_equal(again[k], want[k]) for k in ("tokens", "logprobs", "lens", "versions"))
print("as expected")
""")


def test_without_pinned_memory(child):
    """The same records, with forced tokens and free running; a later call finds pinned memory again and keeps it."""
    child("""
ctx = make_ctx(shape, 4, 9 + new, blob)
for k in range(2):
    shim.hip_refuse(b"hipHostMalloc", 0)
    got = run(ctx)
    assert shim.hip_refused()
    assert all(np.array_equal(got[k], ref[k]) for k in ("tokens", "logprobs", "lens", "versions"))
got = run(ctx)
assert all(np.array_equal(got[k], ref[k]) for k in ("tokens", "logprobs", "lens", "versions"))
shim.hip_refuse(b"hipHostMalloc", 0)
free = ctx.rollout(prompts, lens, G, new, 1.0, 4, eos_id=int(ref["tokens"][0, 0]), continuous=True)
assert not shim.hip_refused()      # (it has its memory by now)
want = ref_ctx.rollout(prompts, lens, G, new, 1.0, 4, eos_id=int(ref["tokens"][0, 0]), continuous=True)
assert all(np.array_equal(free[k], want[k]) for k in ("tokens", "logprobs", "lens", "versions"))
print("as expected")
""")


def test_an_error_of_the_callers_own_is_not_the_calls(child):
    """The runtime keeps the last error of a thread until it is read.  One that the caller's own HIP code has left there is none
    of the library's."""
    child("""
hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
plain = make_ctx(shape, P * G, 9 + new, blob)
refilled = make_ctx(shape, 4, 9 + new, blob)
tokens = np.random.default_rng(5).integers(0, shape.vocab, (4, 15)).astype(np.int32)
tlens, rewards = np.array([15, 1, 7, 12], np.int32), np.array([1, 0, 0, 1], np.float32)
version = iter(range(1, 100))
calls = dict(
    rollout=lambda: plain.rollout(prompts, lens, G, new, 1.0, 4, stop_lens=stop, forced=forced)["tokens"],
    one_token=lambda: plain.rollout(prompts, lens, G, 1, 1.0, 4)["tokens"],
    continuous=lambda: run(refilled)["tokens"],
    scores=lambda: plain.logprobs(tokens, tlens),
    grpo=lambda: plain.grpo_tensors(tokens, tlens, 2, 3, rewards)[2],
    grpo_static=lambda: plain.grpo_tensors(tokens, tlens, 2, 3, rewards, static_scratch=True)[2],
    draws=lambda: plain.draw_bits(1, 2, 3, 0, 9),
    install=lambda: plain.load_policy(next(version), blob),
)
failed = []
for name, call in calls.items():
    want = call()
    assert hip.hipSetDevice(4096) != 0 and hip.hipPeekAtLastError() != 0
    try:
        got = call()
        assert np.array_equal(got, want) or want is None, name
    except echo.EchoError as e:
        failed.append((name, str(e)))
    hip.hipGetLastError()
print(failed or "as expected")
""")


@pytest.mark.parametrize("call,kernel", [("one_token", "dbg_embed_kernel"), ("one_token", "dbg_gemm_kernel"), ("one_token", "gather_rows_kernel"),
                                         ("one_token", "dbg_sample_kernel"), ("one_token", "kv_replicate_kernel"),
                                         ("scores", "dbg_gemm_kernel"), ("scores", "dbg_target_logprob_kernel"), ("draws", "draw_bits_kernel")])
def test_a_refused_launch_outside_the_steps_is_an_error(child, call, kernel):
    """The first launch, one in the middle and the last one of a rollout that ends with its first token, of a scoring pass, of a read-out
    of the generator."""
    child(f"""
ctx = make_ctx(shape, P * G, 9 + new, blob)
tokens = np.random.default_rng(5).integers(0, shape.vocab, (4, 15)).astype(np.int32)
go = dict(one_token=lambda: ctx.rollout(prompts, lens, G, 1, 1.0, 4)["tokens"],
          scores=lambda: ctx.logprobs(tokens, np.array([15, 2, 7, 12], np.int32)),
          draws=lambda: ctx.draw_bits(1, 2, 3, 0, 9))["{call}"]
shim.hip_refuse(b"{kernel}", 1 << 30)
want = go()
n = shim.hip_seen()
assert n > 0
for after in sorted({{0, n // 2, n - 1}}):
    shim.hip_refuse(b"{kernel}", after)
    try:
        go()
    except echo.EchoError as e:
        assert e.code == echo.ECHO_EHIP and shim.hip_refused(), e
    else:
        raise SystemExit(f"succeeded with launch {{after}} of {{n}} refused")
    assert np.array_equal(go(), want)
print("as expected")
""")


@pytest.mark.parametrize("form,kernel", [("whole", "pack_weight_kernel"), ("q8", "pack_weight_kernel"), ("q8", "dequant_q8_kernel"),
                                         ("delta", "pack_span_kernel")])
def test_a_refused_launch_of_an_install_leaves_no_snapshot(child, form, kernel):
    """The first and the last launch; a load from the start afterwards is as good as ever."""
    child(f"""
shape = synth.ModelShape(1, 64, 2, 1, 64, 96, 200)
blob, q8 = synth.make_weights(shape, 1), synth.make_q8_weights(shape, 1)
tokens, tlens = np.random.default_rng(5).integers(0, shape.vocab, (2, 15)).astype(np.int32), np.array([15, 7], np.int32)
off = synth.blob_offsets(shape)["layers.0.w_gate"][0] * 2
data = np.random.default_rng(6).integers(0, 60, 200, dtype=np.uint8)
version = 0

def install(ctx):
    global version
    if "{form}" == "delta":
        ctx.load_policy(version + 1, blob)
        ctx.load_policy_delta(version + 1, version + 2, [off, off + 1000], [80, 120], data)
    elif "{form}" == "q8":
        ctx.load_policy_q8(version + 1, q8)
    else:
        ctx.load_policy(version + 1, blob)

ctx = make_ctx(shape, 2, 16)
shim.hip_refuse(b"{kernel}", 1 << 30)
install(ctx)
n = shim.hip_seen()
want = ctx.logprobs(tokens, tlens)
assert n > 0
for after in sorted({{0, n - 1}}):
    version += 10
    shim.hip_refuse(b"{kernel}", after)
    try:
        install(ctx)
    except echo.EchoError as e:
        assert e.code == echo.ECHO_EHIP and shim.hip_refused(), e
    else:
        raise SystemExit(f"succeeded with launch {{after}} of {{n}} refused")
    try:
        ctx.logprobs(tokens, tlens)
    except echo.EchoError as e:
        assert e.code == echo.ECHO_ESTATE, e
    else:
        raise SystemExit("a snapshot is there")
    version += 10
    install(ctx)
    assert np.array_equal(ctx.logprobs(tokens, tlens), want)
print("as expected")
""")
