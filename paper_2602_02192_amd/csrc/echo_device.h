// Device-side helpers shared by the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "echo_kernels.h"

namespace echo {

// MFMA operands are IEEE half precision (11-bit significand): activations, the KV cache and the attention
// probabilities are rounded to it, which keeps the logit error of a 36-layer, 151936-entry model an order of
// magnitude below what 8-bit-significand bf16 operands give.  The weights are bf16 values; they are held as
// half-precision values scaled by W_SCALE (a power of two, so exact for every bf16 weight of magnitude
// 2^-22 .. 255), and the fp32 accumulators are scaled back by W_UNSCALE in the epilogues.
typedef __attribute__((ext_vector_type(8))) _Float16 h16x8;
constexpr float W_SCALE = 256.0f, W_UNSCALE = 1.0f / 256.0f;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// round-to-nearest-even fp32 -> bf16 bits (finite inputs; NaN keeps a quiet NaN)
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// fp32 -> half bits, round to nearest even, saturating at the largest finite half
__device__ __forceinline__ uint16_t f32_to_h16_bits(float f) {
  _Float16 h = (_Float16)fminf(fmaxf(f, -65504.0f), 65504.0f);
  return __builtin_bit_cast(uint16_t, h);
}
// two of them, a in the low half
__device__ __forceinline__ uint32_t f32_to_h16_pair(float a, float b) {
  typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, h16x2{(_Float16)fminf(fmaxf(a, -65504.0f), 65504.0f), (_Float16)fminf(fmaxf(b, -65504.0f), 65504.0f)});
}
__device__ __forceinline__ float h16_bits_to_f32(uint16_t b) { return (float)__builtin_bit_cast(_Float16, b); }
__device__ __forceinline__ f32x16 mfma_h16(h16x8 a, h16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }

// silu(g) * u of the accumulators g W_SCALE and u W_SCALE, silu(x) = x / (1 + exp(-x)), in the bits of x / (1.0f + expf(-x)) * u wherever the half
// behind it is not zero (tests/test_gpu_swiglu_bits.py sweeps every g that a product can come to; bits of the compiler and device library that this is built
// with).  The steps are theirs without what the range makes idle.  exp(-x): the device library's expf (ROCm-Device-Libs, ocml, open source), a two-part log2 e
// multiplied out with fmas, 2^fraction by v_exp_f32, ldexp; without range checks (x is held between -87, where exp(-x) is finite and the
// quotient 1e-38 of x, and 126, where 1 + exp(-x) is 1).  The quotient: LLVM's AMDGPU expansion of the fp32 division, a Newton step on v_rcp_f32 and two
// corrections of the quotient by its residual (Markstein, IBM J. Res. Dev. 34, 1990); without the scaling of very large and very small
// operands (1 + exp(-x) lies in [1, 2^126]).  Nineteen instructions for twenty-six and the latency of their condition masks.  Accumulators are
// finite: a product's operands and the weights saturate.  Twelve instructions, a first-order term for the rounding of t and one Newton step for the
// reciprocal, take 2 % off the long passes' projection, but a rounding of half in a thousand then falls the other way, and with it a draw now and then.
__device__ __forceinline__ float swiglu(float g, float u) {
#pragma clang fp contract(off)
  constexpr float L2E = 1.44269504088896341f, L2E_LOW = 1.92596286e-8f;   // log2 e = L2E + L2E_LOW + 1.4e-15 (expf's; the nearest float is one ulp up)
  const float x = __builtin_amdgcn_fmed3f(g, -87.0f * W_SCALE, 126.0f * W_SCALE), t = x * (-L2E * W_UNSCALE), whole = rintf(t);
  const float low = fmaf(x, -L2E_LOW * W_UNSCALE, fmaf(x, -L2E * W_UNSCALE, -t));
  const float d = 1.0f + __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f((t - whole) + low), (int)whole);
  float r = __builtin_amdgcn_rcpf(d), q;
  r = fmaf(fmaf(-d, r, 1.0f), r, r);
  q = g * r;
  q = fmaf(fmaf(-d, q, g), r, q);
  q = fmaf(fmaf(-d, q, g), r, q);
  return q * (W_UNSCALE * W_UNSCALE) * u;
}

template <bool BF16>
__device__ __forceinline__ float load_w(const void *p, int64_t i) {
  if (BF16) return bf16_bits_to_f32(((const uint16_t *)p)[i]);
  return ((const float *)p)[i];
}

// Philox-4x32 with 10 rounds (Salmon et al., SC'11): multipliers 0xD2511F53 / 0xCD9E8D57, key
// increments 0x9E3779B9 / 0xBB67AE85.  Both halves of a product come from one v_mad_u64_u32 and the three words that meet are
// folded by one v_bitop3_b32: 20 multiplications and 20 folds a call, where the compiler makes 40 (a high and a low one each) and 38
// of the plain form.  128 rows of 151936: topp_draw_kernel, which the vector unit bounds, 52.8 -> 46.0 us; the lm_head's sampler, which
// hides most of it behind its loads, 254 -> 249 (256 rows) and 134.0 -> 132.6 (64).
struct u32x4 { uint32_t x, y, z, w; };
__device__ __forceinline__ u32x4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                               uint32_t k1) {
  constexpr uint32_t XOR3 = 0x96;   // truth table of a ^ b ^ c
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, XOR3);
    c2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, XOR3);
    c1 = (uint32_t)p1; c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
  return {c0, c1, c2, c3};
}

// Four draws for vocabulary entries 4*i4 .. 4*i4+3 of sequence n at generation step s.
__device__ __forceinline__ u32x4 draw4(uint64_t seed, uint32_t n, uint32_t s, uint32_t i4) {
  return philox4x32_10(i4, s, n, 0u, (uint32_t)seed, (uint32_t)(seed >> 32));
}

// Step and stream words of row m's draws.
__device__ __forceinline__ uint32_t draw_step(const DrawIds &d, int m) { return (uint32_t)(d.row_step ? d.row_step[m] : *d.d_step); }
__device__ __forceinline__ uint32_t draw_stream(const DrawIds &d, int m) { return (uint32_t)(d.row_stream ? d.row_stream[m] : m); }

// 23 random bits k -> u = (2k + 1) 2^-24: the bits as the significand of a number from 1 to 2, less what is too much (exact).
__device__ __forceinline__ float uniform_from_bits(uint32_t bits) {
  return __uint_as_float(__builtin_amdgcn_alignbit(127u, bits, 9)) - (1.0f - 0x1p-24f);
}

// The standard Gumbel variate -log(-log u) of the same u in fp32.
__device__ __forceinline__ float gumbel_from_bits(uint32_t bits) {
  float u = (float)(2u * (bits >> 9) + 1u) * 0x1p-24f;
  return -logf(-logf(u));
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Running Gumbel-max / log-sum-exp state for one row over a subset of the vocabulary.
struct SampleAcc {
  float zmax, zsum;   // max z and sum exp(z - zmax)
  float best, zbest;  // best perturbed score and the z at that entry
  int32_t idx;        // its vocabulary index (lowest index on exact ties)
};
__device__ __forceinline__ SampleAcc sample_acc_init() { return {-INFINITY, 0.f, -INFINITY, 0.f, 0x7fffffff}; }
__device__ __forceinline__ void sample_acc_add(SampleAcc &a, float z, float score, int32_t i) {
  if (z > a.zmax) { a.zsum = a.zsum * expf(a.zmax - z) + 1.f; a.zmax = z; }
  else a.zsum += expf(z - a.zmax);
  if (score > a.best || (score == a.best && i < a.idx)) { a.best = score; a.idx = i; a.zbest = z; }
}
__device__ __forceinline__ void sample_acc_merge(SampleAcc &a, const SampleAcc &b) {
  if (b.zmax > a.zmax) { a.zsum = a.zsum * expf(a.zmax - b.zmax) + b.zsum; a.zmax = b.zmax; }
  else if (b.zmax > -INFINITY) a.zsum += b.zsum * expf(b.zmax - a.zmax);
  if (b.best > a.best || (b.best == a.best && b.idx < a.idx)) { a.best = b.best; a.idx = b.idx; a.zbest = b.zbest; }
}
__device__ __forceinline__ SampleAcc sample_acc_shfl_xor(const SampleAcc &a, int o) {
  SampleAcc b;
  b.zmax = __shfl_xor(a.zmax, o, 64); b.zsum = __shfl_xor(a.zsum, o, 64);
  b.best = __shfl_xor(a.best, o, 64); b.zbest = __shfl_xor(a.zbest, o, 64);
  b.idx = __shfl_xor(a.idx, o, 64);
  return b;
}

// A workgroup's partial of a row, at o = workgroup * rows + row of a buffer of `plane` partials: (max z, sum, best score, its z) side by
// side, so that the row's reader fetches one line of them, and the index in a plane of its own.  A scoring pass has the first two only.
__device__ __forceinline__ void sample_part_store(float *part, int64_t o, int64_t plane, const SampleAcc &a) {
  *(f32x4 *)(part + 4 * o) = f32x4{a.zmax, a.zsum, a.best, a.zbest};
  part[4 * plane + o] = __int_as_float(a.idx);
}
__device__ __forceinline__ SampleAcc sample_part_load(const float *part, int64_t o, int64_t plane) {
  const f32x4 v = *(const f32x4 *)(part + 4 * o);
  return {v[0], v[1], v[2], v[3], __float_as_int(part[4 * plane + o])};
}
__device__ __forceinline__ void score_part_store(float *part, int64_t o, const SampleAcc &a) { *(float2 *)(part + 2 * o) = make_float2(a.zmax, a.zsum); }

// Entry idx = m * half + i of the rotary table: cos/sin of pos * base^(-2i/hd), evaluated in double and stored as fp32.
__device__ __forceinline__ void rope_entry(float2 *cs, const int32_t *pos, int idx, int M, int half, float base) {
  if (idx >= M * half) return;
  const int m = idx / half, i = idx % half, p = max(pos[m], 0);
  const double theta = pow((double)base, -2.0 * (double)i / (double)(2 * half)), ang = (double)p * theta;
  double s, c;
  sincos(ang, &s, &c);
  cs[idx] = make_float2((float)c, (float)s);
}

// Bookkeeping of a generation step for row n, by one thread of the workgroup that has drawn its token: records the token, chooses
// the one that is fed back (forced or sampled), applies the stop rules and prepares the row for the next decode pass.  All b.n rows
// of the batch pass here; the last to arrive closes the step (*d_step, *n_active).  Rows are counted, and the live ones among
// them, in one atomic, so nothing else has to be visible to that last one; and what a workgroup reads of *d_step has arrived
// before it counts itself, hence before the last one moves the step on.
__device__ __forceinline__ void book_row(const StepBook &b, int n, int tok, float lp) {
  const int s0 = *b.d_step;
  unsigned long long live = 0;
  if (b.rows.active[n]) {
    const int s = b.per_row ? b.gen_len[n] : s0;
    const int64_t o = (int64_t)b.rows.slot[n] * b.max_new + s;   // records are kept per cache slot (= row unless rows were compacted)
    b.out_tok[o] = tok;
    b.out_lp[o] = lp;
    b.out_ver[o] = b.version;
    const int fed = b.forced ? b.forced[o] : tok == 0x7fffffff ? 0 : tok;   // (logits of NaN yield no entry of the vocabulary, and none to read an embedding at)
    const int len = s + 1;
    b.gen_len[n] = len;
    const bool done = len >= b.limit[n] || (b.eos >= 0 && fed == b.eos);
    b.rows.token[n] = fed;
    b.rows.pos[n] = b.prompt_len[n] + s;
    b.rows.active[n] = done ? 0 : 1;
    live = done ? 0 : 1;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  const unsigned long long before = atomicAdd(b.arrived, live << 32 | 1);
  if ((int)(uint32_t)before + 1 == b.n) {
    *b.n_active = (int)(before >> 32) + (int)live;
    *b.d_step = s0 + 1;
    atomicExch(b.arrived, 0ull);
  }
}

}  // namespace echo
