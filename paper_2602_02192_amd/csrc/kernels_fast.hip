// MFMA path, everything that is not a dense contraction: residual + RMSNorm (with the split-K
// reduction folded in), QKV post-processing (reduction, per-head norm, rotary embedding, KV append).
#include <type_traits>

#include "attn_plan.h"
#include "echo_device.h"
#include "echo_kernels.h"

namespace echo {

// Calls f(std::integral_constant<int, n>) for a split count n in 0 .. REDUCE_MAX_SPLIT that is known only at run time: the
// reducing kernels take it as a template parameter, because loads behind run-time conditions made the compiler wait for the
// first of them before it issued the rest.
template <int N = REDUCE_MAX_SPLIT, typename F>
static void with_split_count(int n, F f) {
  if constexpr (N >= 0) {
    if (n == N) f(std::integral_constant<int, N>{});
    else with_split_count<N - 1>(n, f);
  }
}

// The row that workgroup blockIdx.x of n takes.  Workgroup i starts on XCD i % 8; the rows are dealt to the XCDs in contiguous
// eighths, because a 128-byte line of the K8 activation layout, or of a key or value tile, holds 16 bytes or less of each of
// several neighbouring rows: written from one XCD its pieces meet in that XCD's L2, written from eight they reach memory one by
// one (4096 rows: residual + norm 35.7 -> 29.4 us, qkv_post_wide_kernel 47.6 -> 44.4 at the 4B width).
__device__ __forceinline__ int xcd_row(int n) {   // (of workgroups 0 .. n - 1)
  const int id = blockIdx.x, x = id & 7;
  return x * (n >> 3) + min(x, n & 7) + (id >> 3);
}

// grid M rows, block <= 1024 (a multiple of 64 covering d/4 (CH = 1) or d/8 (CH = 2) lanes).
//   EMBED: h[m] = embed[token[m]];  else h[m] += sum_s partials[s][..][m]  (NS partials, summed in split order)
// then Xp[m] = half(h[m] * rsqrt(mean(h[m]^2) + eps) * gain).  d % 8 == 0, d <= 8192.
// A decode step's launch is bound by latency (kilobytes per workgroup, partials that other XCDs wrote): every load of a thread --
// residual, all partials, the gain -- is issued before the first use, so the kernel costs one memory round trip whatever the
// split count: 64 rows of 2560, 8 or 9 partials, 4.87 -> 4.80 us (an empty launch takes 3).  Long passes are bound by HBM: 4096 rows
// of 2560 37.8 -> 29.4 us (14 bytes per element, 5.0 TB/s), of 5120 with two planes 86 -> 77.5 (4.9), for most part by xcd_row.
constexpr int RN_THREADS = 1024;
template <int NS, int CH, bool EMBED>
__device__ __forceinline__ void resid_norm_row(int m, int lanes, float *__restrict__ h, const uint16_t *__restrict__ embed, const int32_t *__restrict__ token,
                                               const f32x4 *__restrict__ partials, int Np, uint16_t *__restrict__ Xp,
                                               const uint16_t *__restrict__ gain, int Mp, int d, float eps) {
  __shared__ float sh[RN_THREADS / 64];
  const int d4 = d >> 2;
  f32x4 v[CH], pp[CH][NS > 0 ? NS : 1];
  uint2 gn[CH], em[CH];
  const int tok = EMBED ? token[m] : 0;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int n4 = min((int)threadIdx.x + c * lanes, d4 - 1);   // lanes past the row repeat its last unit and store nothing
    if (EMBED) em[c] = *(const uint2 *)(embed + (int64_t)max(tok, 0) * d + n4 * 4);
    else v[c] = *(const f32x4 *)(h + (int64_t)m * d + n4 * 4);
#pragma unroll
    for (int s = 0; s < NS; ++s) pp[c][s] = partials[((int64_t)s * Mp + m) * (Np >> 2) + n4];
    gn[c] = *(const uint2 *)(gain + n4 * 4);
  }
  __builtin_amdgcn_sched_barrier(0);   // the loads above stay ahead of everything below
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int n4 = (int)threadIdx.x + c * lanes;
    f32x4 a = v[c];
    if (EMBED) {
      const uint2 e = em[c];
      a = {__uint_as_float(e.x << 16), __uint_as_float(e.x & 0xffff0000u), __uint_as_float(e.y << 16), __uint_as_float(e.y & 0xffff0000u)};
      if (tok < 0) a = {0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) a += pp[c][s];
    v[c] = a;
    if (n4 < d4 && (int)threadIdx.x < lanes) {
      if (EMBED || NS > 0) *(f32x4 *)(h + (int64_t)m * d + n4 * 4) = a;
      ss += a[0] * a[0] + a[1] * a[1] + a[2] * a[2] + a[3] * a[3];
    }
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = 0.f;
  for (int i = 0; i < (int)blockDim.x / 64; ++i) ss += sh[i];
  float inv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int n4 = (int)threadIdx.x + c * lanes, n = n4 * 4;
    const uint2 g = gn[c];
    float g0 = __uint_as_float(g.x << 16), g1 = __uint_as_float(g.x & 0xffff0000u);
    float g2 = __uint_as_float(g.y << 16), g3 = __uint_as_float(g.y & 0xffff0000u);
    uint2 o;
    o.x = (uint32_t)f32_to_h16_bits(v[c][0] * inv * g0) | ((uint32_t)f32_to_h16_bits(v[c][1] * inv * g1) << 16);
    o.y = (uint32_t)f32_to_h16_bits(v[c][2] * inv * g2) | ((uint32_t)f32_to_h16_bits(v[c][3] * inv * g3) << 16);
    if (n4 < d4 && (int)threadIdx.x < lanes) *(uint2 *)(Xp + ((int64_t)(n >> 3) * Mp + m) * 8 + (n & 7)) = o;
  }
}

template <int NS, int CH>
__global__ __launch_bounds__(RN_THREADS) void resid_norm_kernel(float *__restrict__ h, const f32x4 *__restrict__ partials, int Np, uint16_t *__restrict__ Xp,
                                                                const uint16_t *__restrict__ gain, int Mp, int d, float eps) {
  resid_norm_row<NS, CH, false>(xcd_row(gridDim.x), blockDim.x, h, nullptr, nullptr, partials, Np, Xp, gain, Mp, d, eps);
}

// Begins a pass in one launch: workgroups 0 .. M - 1 embed and norm a row each, the next one (with a plan; blocks are of
// ATT_ROWS_BATCH_MAX threads then) writes the tile lists of the decode attention, the rest the rotary table.  None needs another's
// result, and each is a dependent launch saved per step: 64 rows of the 4B shape 4.7 + 5.4 + 4.9 us apart, 6.6 us together; one
// row (no plan) 4.5 + 4.4 us, 4.7 us.  `lanes` threads share a row whatever the block, so that its sum keeps its order.
template <int CH>
__global__ __launch_bounds__(RN_THREADS) void step_begin_kernel(float *__restrict__ h, const uint16_t *__restrict__ embed, RowState rows, uint16_t *__restrict__ Xp,
                                                                const uint16_t *__restrict__ gain, int M, int Mp, int d, int lanes, float eps, RopeTable rope,
                                                                RowsPlan plan, int grp) {
  const int extra = (int)blockIdx.x - M, planners = plan.plan ? 1 : 0;
  if (extra < 0) resid_norm_row<0, CH, true>(xcd_row(M), lanes, h, embed, rows.token, nullptr, 0, Xp, gain, Mp, d, eps);
  else if (extra < planners) attn_rows_plan(plan.plan, rows, M, grp, plan.sets);
  else rope_entry((float2 *)rope.cs, rope.pos, (extra - planners) * blockDim.x + threadIdx.x, M, rope.hd / 2, rope.base);
}

static_assert(RN_THREADS == ATT_ROWS_BATCH_MAX, "a workgroup of the largest size can write the plan");
// One float4 per thread when a row of d fits a workgroup so, else two.
static int row_loads(int d) { return ((d >> 2) + 63) / 64 * 64 <= RN_THREADS ? 1 : 2; }
static int row_threads(int d) { return ((d >> (row_loads(d) + 1)) + 63) / 64 * 64; }

void fast_step_begin(float *h, const void *embed_bf16, RowState rows, void *Xp, const void *gain_bf16, int M, int Mp, int d, float eps, RopeTable rope,
                     RowsPlan plan, int grp, hipStream_t st) {
  if (M <= 0) return;
  const int threads = plan.plan ? RN_THREADS : row_threads(d), grid = M + (plan.plan ? 1 : 0) + (M * (rope.hd / 2) + threads - 1) / threads;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, h, (const uint16_t *)embed_bf16, rows, (uint16_t *)Xp, (const uint16_t *)gain_bf16, M, Mp, d,
                       row_threads(d), eps, rope, plan, grp);
  };
  if (row_loads(d) == 1) launch(step_begin_kernel<1>); else launch(step_begin_kernel<2>);
}

void fast_resid_norm(float *h, const float *partials, int nsplit, int Np, void *Xp, const void *gain_bf16, int M, int Mp, int d, float eps,
                     hipStream_t st) {
  if (M <= 0) return;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(M), dim3(row_threads(d)), 0, st, h, (const f32x4 *)partials, Np, (uint16_t *)Xp, (const uint16_t *)gain_bf16, Mp, d, eps);
  };
  with_split_count(nsplit, [&](auto n) {
    if (row_loads(d) == 1) launch(resid_norm_kernel<decltype(n)::value, 1>);
    else launch(resid_norm_kernel<decltype(n)::value, 2>);
  });
}

// grid (M, ceil((Hq + 2*Hkv) / QP_HEADS)), block QP_HEADS * hd/2 with hd/2 <= 64: each group of hd/2 lanes sums the
// split-K partials of one head of one row, applies the optional per-head RMSNorm and the rotary embedding, and writes
// q (half [M][Hq][hd]) or appends k / v to the half-precision cache.  Bound by latency like resid_norm_kernel: the row's
// state, the partials, the rotation and the gains are all requested before the first sum, and a row that is not generating
// only drops its stores.  64 rows, 5 partials of 6144: 5.41 -> 5.19 us.
// The fused products are written out here and in the wide kernel below, because which product of a sum the compiler rounds differs
// from one instantiation to the next, a last bit of fp32 that flips half-precision roundings in every later layer.
constexpr int QP_HEADS = 8;
template <int NS, bool NORM>
__global__ void qkv_post_kernel(const float *__restrict__ partials, int Np, int Mp, uint16_t *__restrict__ q_out, const uint16_t *__restrict__ q_gain,
                                const uint16_t *__restrict__ k_gain, float eps, const float2 *__restrict__ rope_cs, RowState rows,
                                KvGeom kv, int layer, int Hq, int Hkv) {
  int hd = kv.head_dim, half = hd / 2;
  int m = blockIdx.x, j = blockIdx.y * QP_HEADS + threadIdx.x / half, i = threadIdx.x % half;
  if (j >= Hq + 2 * Hkv) return;
  bool is_q = j < Hq, is_k = !is_q && j < Hq + Hkv;
  int act = rows.active[m], pos = rows.pos[m], slot = rows.slot[m];
  int n0 = j * hd + i, n1 = n0 + half;
  float a = 0.f, b = 0.f, pa[NS], pb[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    pa[s] = partials[((int64_t)s * Mp + m) * Np + n0];
    pb[s] = partials[((int64_t)s * Mp + m) * Np + n1];
  }
  const float2 cs = rope_cs[(int64_t)m * half + i];
  uint16_t w0 = 0, w1 = 0;
  if (NORM) {
    const uint16_t *g = is_q ? q_gain : k_gain;   // (loaded and not used for a value head)
    w0 = g[i]; w1 = g[i + half];
  }
  __builtin_amdgcn_sched_barrier(0);   // all loads issued before the sums, the row's state among them
  asm volatile("" : "+s"(act), "+s"(pos), "+s"(slot));
#pragma unroll
  for (int s = 0; s < NS; ++s) { a += pa[s]; b += pb[s]; }
  if (is_q || is_k) {
    if (NORM) {
      float ss = fmaf(b, b, a * a);   // the head's lanes are an aligned power-of-two group within the wave
      for (int off = half >> 1; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
      float inv = 1.0f / sqrtf(ss / (float)hd + eps);
      a = a * inv * bf16_bits_to_f32(w0);
      b = b * inv * bf16_bits_to_f32(w1);
    }
    float ra = fmaf(a, cs.x, -(b * cs.y)), rb = fmaf(b, cs.x, a * cs.y);
    a = ra; b = rb;
  }
  if (is_q) {
    uint16_t *dst = q_out + ((int64_t)m * Hq + j) * hd;
    dst[i] = f32_to_h16_bits(a);
    dst[i + half] = f32_to_h16_bits(b);
  } else if (act) {   // append to the tiled cache
    int kvh = is_k ? j - Hq : j - Hq - Hkv;
    uint16_t *head = (uint16_t *)kv.base + kv.tiled_head_off(slot, layer, kvh);
    if (is_k) { head[kv.tiled_k_off(pos, i)] = f32_to_h16_bits(a); head[kv.tiled_k_off(pos, i + half)] = f32_to_h16_bits(b); }
    else { head[kv.tiled_v_off(pos, i)] = f32_to_h16_bits(a); head[kv.tiled_v_off(pos, i + half)] = f32_to_h16_bits(b); }
  }
}

// The same for batches of hundreds of rows and more (prefill, scoring, wide decode steps), where the kernel above is a
// launch of millions of threads that move 14 bytes each: here a thread takes four consecutive dims of the head's first half
// and their four rotation partners, with 16-byte loads of the partials and of the rotation table and 8-byte stores of q and
// of the key tile (a value tile holds eight keys of one dim per unit, so values still leave as single halves).  Same sums in
// the same order: bit-identical to the kernel above, except that with a per-head norm each square pair rounds the other
// product (b's here, a's there), as results of the two forms always have.  grid (M, ceil((Hq + 2*Hkv) / QPW_HEADS)), block QPW_HEADS * hd/8.
constexpr int QPW_HEADS = 16;
template <int NS, bool NORM>
__global__ void qkv_post_wide_kernel(const float *__restrict__ partials, int Np, int Mp, uint16_t *__restrict__ q_out, const uint16_t *__restrict__ q_gain,
                                     const uint16_t *__restrict__ k_gain, float eps, const float2 *__restrict__ rope_cs, RowState rows,
                                     KvGeom kv, int layer, int Hq, int Hkv) {
  const int hd = kv.head_dim, half = hd / 2, per_head = half / 4;
  const int m = xcd_row(gridDim.x), j = blockIdx.y * QPW_HEADS + threadIdx.x / per_head, i = (threadIdx.x % per_head) * 4;
  if (j >= Hq + 2 * Hkv) return;
  const bool is_q = j < Hq, is_k = !is_q && j < Hq + Hkv;
  int act = rows.active[m], pos = rows.pos[m], slot = rows.slot[m];
  const int n0 = j * hd + i, n1 = n0 + half;
  f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f}, pa[NS], pb[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const float *row = partials + ((int64_t)s * Mp + m) * Np;
    pa[s] = *(const f32x4 *)(row + n0);
    pb[s] = *(const f32x4 *)(row + n1);
  }
  const f32x4 *cs = (const f32x4 *)(rope_cs + (int64_t)m * half + i);
  const f32x4 c01 = cs[0], c23 = cs[1];
  __builtin_amdgcn_sched_barrier(0);   // all loads issued before the sums
  asm volatile("" : "+s"(act), "+s"(pos), "+s"(slot));
#pragma unroll
  for (int s = 0; s < NS; ++s) { a += pa[s]; b += pb[s]; }
  if (is_q || is_k) {
    if (NORM) {
      // Summed in the order of the one-pair-per-lane kernel, whose tree adds lane i ^ off to lane i for off = half/2 .. 1:
      // its lanes 4q .. 4q+3 sit in this thread, so its offsets >= 4 are shuffles over the head's threads, element by
      // element, and its offsets 2 and 1 are the local sums at the end.
      float t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = fmaf(a[e], a[e], b[e] * b[e]);
      for (int off = per_head >> 1; off > 0; off >>= 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] += __shfl_xor(t[e], off);
      }
      const float ss = (t[0] + t[2]) + (t[1] + t[3]);
      float inv = 1.0f / sqrtf(ss / (float)hd + eps);
      const uint16_t *g = is_q ? q_gain : k_gain;
#pragma unroll
      for (int e = 0; e < 4; ++e) { a[e] = a[e] * inv * bf16_bits_to_f32(g[i + e]); b[e] = b[e] * inv * bf16_bits_to_f32(g[i + e + half]); }
    }
    const float cx[4] = {c01[0], c01[2], c23[0], c23[2]}, sy[4] = {c01[1], c01[3], c23[1], c23[3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float ra = fmaf(a[e], cx[e], -(b[e] * sy[e])), rb = fmaf(b[e], cx[e], a[e] * sy[e]);
      a[e] = ra; b[e] = rb;
    }
  }
  uint2 ha, hb;
  ha.x = (uint32_t)f32_to_h16_bits(a[0]) | ((uint32_t)f32_to_h16_bits(a[1]) << 16);
  ha.y = (uint32_t)f32_to_h16_bits(a[2]) | ((uint32_t)f32_to_h16_bits(a[3]) << 16);
  hb.x = (uint32_t)f32_to_h16_bits(b[0]) | ((uint32_t)f32_to_h16_bits(b[1]) << 16);
  hb.y = (uint32_t)f32_to_h16_bits(b[2]) | ((uint32_t)f32_to_h16_bits(b[3]) << 16);
  if (is_q) {
    uint16_t *dst = q_out + ((int64_t)m * Hq + j) * hd;
    *(uint2 *)(dst + i) = ha;
    *(uint2 *)(dst + i + half) = hb;
  } else if (act) {
    const int kvh = is_k ? j - Hq : j - Hq - Hkv;
    uint16_t *head = (uint16_t *)kv.base + kv.tiled_head_off(slot, layer, kvh);
    if (is_k) {   // four dims of one 8-dim unit of the key
      *(uint2 *)(head + kv.tiled_k_off(pos, i)) = ha;
      *(uint2 *)(head + kv.tiled_k_off(pos, i + half)) = hb;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        head[kv.tiled_v_off(pos, i + e)] = f32_to_h16_bits(a[e]);
        head[kv.tiled_v_off(pos, i + e + half)] = f32_to_h16_bits(b[e]);
      }
    }
  }
}

void fast_qkv_post(const float *partials, int nsplit, int Np, int Mp, void *q_h16, const void *q_gain, const void *k_gain,
                   int qk_norm, float eps, const float *rope_cs, RowState rows, KvGeom kv, int layer, int M, int Hq, int Hkv,
                   hipStream_t st) {
  const int heads = Hq + 2 * Hkv, hd = kv.head_dim;
  auto launch = [&](auto kernel, int per_wg, int threads) {
    hipLaunchKernelGGL(kernel, dim3(M, (heads + per_wg - 1) / per_wg), dim3(threads), 0, st, partials, Np, Mp, (uint16_t *)q_h16,
                       (const uint16_t *)q_gain, (const uint16_t *)k_gain, eps, (const float2 *)rope_cs, rows, kv, layer, Hq, Hkv);
  };
  with_split_count(nsplit, [&](auto n) {
    constexpr int NS = decltype(n)::value > 0 ? decltype(n)::value : 1;   // (a projection leaves at least one plane)
    if (M >= 256) {
      if (qk_norm) launch(qkv_post_wide_kernel<NS, true>, QPW_HEADS, QPW_HEADS * hd / 8);
      else launch(qkv_post_wide_kernel<NS, false>, QPW_HEADS, QPW_HEADS * hd / 8);
    } else {
      if (qk_norm) launch(qkv_post_kernel<NS, true>, QP_HEADS, QP_HEADS * hd / 2);
      else launch(qkv_post_kernel<NS, false>, QP_HEADS, QP_HEADS * hd / 2);
    }
  });
}

// ---- nucleus (top-p) sampling over materialised logits ---------------------------------------------------------
// With p = softmax(logits / T): keep the shortest prefix of the tokens in descending order of p (lower index first
// among equals) whose probabilities reach top_p, draw by Gumbel-max over the kept set with the usual per-index noise,
// return the log-prob renormalised over the kept set (Sec. 5.1 runs rollouts at top-p 0.95).  Three launches:
// 1. topp_cut_kernel, one workgroup per row, finds the cut without sorting.  A histogram of the probability mass over bins of
//    z = logit / T that divide the row's own spread evenly, from its maximum down, names the bin that the cut lies in; if that bin
//    must hold more keys than the list, a second histogram divides it.  The keys of the bin (a few hundred of 150 thousand) go to a
//    list, and a radix select over the order-preserving integer image of the logit finds the cut among them.  Mass is summed in
//    integers, q_i = floor(exp(z_i - max) * 2^40), so the sums do not depend on the order of the additions and the kept set is the
//    same on every run.  Equal keys have equal mass; of the keys equal to the cut the lowest indices are kept until the
//    target is met, so the kernel also returns the last kept index among them.  What bounds it is the vector unit of one
//    compute unit per row, so it counts what a logit costs: three passes (extremes; histogram; list) with one exponential, one
//    pass more for rows that are flat but for a few large scores.  128 rows of 151936 logits, against a byte-wise select over the
//    whole row (five passes, an exponential each): N(0, 1) 99 -> 61 us, the same at T = 1000 98 -> 59 us, one score that weighs
//    as much as all others, which are equal to 1e-4, 103 -> 103 us, two values 357 -> 219 us, all equal 467 -> 131 us; 8 rows of
//    2000 logits, with the draw and the merge, 18.2 -> 17.7 us.  (Bins of a fixed width, 1/128 of z, put a whole flat row in one: 185 us
//    at T = 1000.  More copies or bins cost more to clear and walk than they save; fewer than four copies queue up at equal
//    logits: a third of the row equal 113 -> 123 us with the draw.)
// 2. topp_draw_kernel, TOPP_CHUNKS workgroups per row: (max, sum-exp, best perturbed score) over the kept tokens of one
//    slice of the vocabulary, in the partial layout of the fused sampler;
// 3. sample_combine_kernel merges the slices.
constexpr int TOPP_THREADS = 1024, TOPP_CHUNKS = TOPP_CHUNKS_PER_ROW;
__device__ __forceinline__ uint32_t float_order_key(float f) {   // a < b  <=>  key(a) < key(b)
  uint32_t u = __float_as_uint(f);
  return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}
__device__ __forceinline__ float order_key_float(uint32_t key) {   // the float whose key this is
  return __uint_as_float((key & 0x80000000u) ? key ^ 0x80000000u : ~key);
}
constexpr int TOPP_CAND = 1024;   // keys that the select can take from the list (more, not all equal: it walks the row in each round)
// LDS: the histogram, lanes that meet in one bin spread over TOPP_COPIES copies of it; the radix rounds reuse it.
constexpr int TOPP_BINS = 2048, TOPP_COPIES = 4, TOPP_RADIX_COPIES = 16, TOPP_PER_THREAD = TOPP_BINS / TOPP_THREADS, TOPP_LDS = TOPP_BINS * TOPP_COPIES * 8;
constexpr int TOPP_LOADS = 4;   // 16-byte loads of a thread in flight
// keys that are summed up pair by pair (8 rows of 32000 logits, some 50 keys: 30.6 us so, 28.1 by the radix rounds; of 2000, a few keys: 17.7, 20.0)
constexpr int TOPP_FEW = 32;
constexpr float TOPP_SPAN = 32.0f;   // units of z below the maximum that matter: beyond 27.8 the mass is zero
static_assert(TOPP_RADIX_COPIES * 256 <= TOPP_BINS * TOPP_COPIES && TOPP_BINS % TOPP_THREADS == 0, "the rounds fit; whole bins per thread");
__global__ __launch_bounds__(TOPP_THREADS) void topp_cut_kernel(uint32_t *cut_key, int32_t *cut_last, const float *logits, int64_t ld,
                                                                 int V, float temperature, float top_p) {
  extern __shared__ unsigned long long topp_hist[];
  __shared__ unsigned long long sh_u64[TOPP_THREADS / 64];
  __shared__ float sh_f[2][TOPP_THREADS / 64];
  __shared__ uint32_t sh_k[2][TOPP_THREADS / 64];
  __shared__ int sh_i[TOPP_THREADS / 64];
  __shared__ uint32_t cand[TOPP_CAND];
  __shared__ unsigned long long sel_above, sel_mass;
  __shared__ uint32_t sel_digit;
  __shared__ int cand_n;
  const int m = blockIdx.x, tid = threadIdx.x, wv = tid >> 6;
  const float *lg = logits + (int64_t)m * ld;
  // Every pass visits the row, four logits at a time, with a stride of the block, TOPP_LOADS loads in flight per thread (a plain loop
  // waits out one memory latency per element); an index past the end yields `past`.
  const int n4 = (ld & 3) == 0 ? V >> 2 : 0;   // 16-byte loads need aligned rows
  auto visit = [&](float past, auto &&f) {
    const f32x4 *lg4 = (const f32x4 *)lg;
    for (int i = tid; i < n4; i += TOPP_LOADS * TOPP_THREADS) {
      f32x4 v[TOPP_LOADS];
#pragma unroll
      for (int u = 0; u < TOPP_LOADS; ++u) { int j = i + u * TOPP_THREADS; v[u] = j < n4 ? lg4[j] : f32x4{past, past, past, past}; }
#pragma unroll
      for (int u = 0; u < TOPP_LOADS; ++u) f(v[u]);
    }
    auto at = [&](int i) { return i < V ? lg[i] : past; };
    for (int i = n4 * 4 + tid; i < V; i += 4 * TOPP_THREADS) f(f32x4{lg[i], at(i + TOPP_THREADS), at(i + 2 * TOPP_THREADS), at(i + 3 * TOPP_THREADS)});
  };
  const float nan = __uint_as_float(0x7fc00000u);
  if (tid == 0) cand_n = 0;
  // 1/T instead of the division: nothing here is returned, the kept set only needs the same arithmetic in every pass
  const float inv_t = 1.0f / temperature;
  float mx = -INFINITY, mn = INFINITY;
  visit(nan, [&](f32x4 v) {   // (a NaN counts for neither)
#pragma unroll
    for (int e = 0; e < 4; ++e) { mx = fmaxf(mx, v[e]); mn = fminf(mn, v[e]); }
  });
  mx = wave_max(mx);
  mn = -wave_max(-mn);
  if ((tid & 63) == 0) { sh_f[0][wv] = mx; sh_f[1][wv] = mn; }
  __syncthreads();
  float bulk_hi = INFINITY, bulk_lo = -INFINITY;
  for (int w = 0; w < TOPP_THREADS / 64; ++w) {
    mx = fmaxf(mx, sh_f[0][w]); mn = fminf(mn, sh_f[1][w]);
    bulk_hi = fminf(bulk_hi, sh_f[0][w]); bulk_lo = fmaxf(bulk_lo, sh_f[1][w]);
  }
  // most logits within an eighth of the row's spread, by what the sixteen wavefronts saw
  const bool flat = bulk_hi > bulk_lo && (bulk_hi - bulk_lo) * 8.0f < mx - mn;
  const float zmax = mx * inv_t;
  // probability mass in units of 2^-40 of the largest one, as an integer: sums of it do not depend on the order of the
  // additions.  (Two 32-bit conversions; a float -> 64-bit integer conversion is a long instruction sequence.)
  auto mass = [&](float logit) {
    float e = __expf(fmaf(logit, inv_t, -zmax)) * 256.0f;   // <= 256
    uint32_t hi = (uint32_t)e;
    uint32_t lo = (uint32_t)((e - (float)hi) * 4294967296.0f);
    return ((unsigned long long)hi << 32) | lo;
  };
  // Place of a logit on the scale of the bins, falling in it: 0 at the maximum, near TOPP_BINS at the row's minimum or TOPP_SPAN units
  // below, where the mass is zero and the last bin takes all.  Clamped before any conversion, so that any value at all names a bin.
  const float scale = fminf(((float)TOPP_BINS - 0.5f) / fminf(zmax - mn * inv_t, TOPP_SPAN), 1e30f);
  auto place = [&](float logit) { return fminf(fmaxf(fmaf(logit, inv_t, -zmax) * -scale, 0.0f), (float)TOPP_BINS - 0.25f); };
  auto bin = [&](float logit) { return (int)place(logit); };
  int cut_bin = -1, cut_sub = -1;   // the bin that the cut lies in, and, where that bin is divided, its part
  auto sub = [&](float logit) { return (int)fminf((place(logit) - (float)cut_bin) * (float)TOPP_BINS, (float)(TOPP_BINS - 1)); };
  auto member = [&](float logit) { return bin(logit) == cut_bin && (cut_sub < 0 || sub(logit) == cut_sub); };
  unsigned long long target = 0, above = 0;   // mass to reach; mass of the keys above the range that the cut is known to lie in
  // Clears the histogram, has `fill` add to it, and walks it from the top: exactly one bin takes the running mass across the target.
  // A sum over the whole row (target 0) first says what the target is.  Returns false if there is no mass at all.
  auto histogram = [&](auto &&fill) {
    __syncthreads();
    for (int j = tid; j < TOPP_BINS * TOPP_COPIES; j += TOPP_THREADS) topp_hist[j] = 0;
    __syncthreads();
    fill();
    __syncthreads();
    unsigned long long h[TOPP_PER_THREAD], incl = 0, total = 0;
#pragma unroll
    for (int k = 0; k < TOPP_PER_THREAD; ++k) {   // the copies of bin k * TOPP_THREADS + tid, then (from LDS) consecutive bins per thread
      h[k] = 0;
#pragma unroll
      for (int j = 0; j < TOPP_COPIES; ++j) h[k] += topp_hist[(k * TOPP_THREADS + tid) * TOPP_COPIES + j];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TOPP_PER_THREAD; ++k) topp_hist[k * TOPP_THREADS + tid] = h[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TOPP_PER_THREAD; ++k) { h[k] = topp_hist[TOPP_PER_THREAD * tid + k]; incl += h[k]; }
    const unsigned long long mine = incl;
    for (int o = 1; o < 64; o <<= 1) { unsigned long long v = __shfl_up(incl, o, 64); if ((tid & 63) >= o) incl += v; }
    if ((tid & 63) == 63) sh_u64[wv] = incl;
    __syncthreads();
    for (int w = 0; w < TOPP_THREADS / 64; ++w) { if (w < wv) incl += sh_u64[w]; total += sh_u64[w]; }
    if (total == 0) return false;
    if (target == 0) {
      target = (unsigned long long)ceil((double)total * (double)top_p);
      if (target < 1) target = 1;
      if (target > total) target = total;
    }
    unsigned long long at = above + incl - mine;
    if (at < target && at + mine >= target) {
      int k = 0;
      while (k < TOPP_PER_THREAD - 1 && at + h[k] < target) at += h[k++];
      sel_digit = (uint32_t)(TOPP_PER_THREAD * tid + k);
      sel_above = at;
      sel_mass = h[k];
    }
    __syncthreads();
    above = sel_above;
    return true;
  };
  // Four masses to four places of the histogram; neighbours that share one -- flat or equal scores, which would otherwise queue up at one
  // address -- go there as one sum.
  auto add4 = [&](const int (&at)[4], const unsigned long long (&q)[4]) {
    if (at[0] == at[1] && at[0] == at[2] && at[0] == at[3]) {
      const unsigned long long sum = (q[0] + q[1]) + (q[2] + q[3]);
      if (sum) atomicAdd(&topp_hist[at[0]], sum);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (q[e]) atomicAdd(&topp_hist[at[e]], q[e]);
    }
  };
  const int copy = tid & (TOPP_COPIES - 1);
  uint32_t kmin = 0xffffffffu, kmax = 0;
  const bool one_value = mn == mx;   // (zeros may differ in sign)
  if (!histogram([&] {
        if (one_value) {
          int n = 0;
          visit(nan, [&](f32x4 v) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (v[e] == mx) { ++n; kmin = min(kmin, float_order_key(v[e])); kmax = max(kmax, float_order_key(v[e])); }
          });
          if (n) atomicAdd(&topp_hist[bin(mx) * TOPP_COPIES + copy], mass(mx) * (unsigned long long)n);
          if (tid == 0) cand_n = TOPP_CAND + 1;   // no list
        } else if (flat) {
          visit(-INFINITY, [&](f32x4 v) {
            int at[4];
            unsigned long long q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) { at[e] = bin(v[e]) * TOPP_COPIES + copy; q[e] = mass(v[e]); }
            add4(at, q);
          });
        } else {
          visit(-INFINITY, [&](f32x4 v) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const unsigned long long q = mass(v[e]);
              if (q) atomicAdd(&topp_hist[bin(v[e]) * TOPP_COPIES + copy], q);
            }
          });
        }
      })) {   // no finite maximum: every token is kept
    if (tid == 0) { cut_key[m] = 0; cut_last[m] = V; }
    return;
  }
  cut_bin = (int)sel_digit;
  // The bin's keys have at most the mass at its upper edge each.  If it holds more of them than the list for certain, it is
  // divided (flat scores below a few large ones; equal ones stay together however it is divided).
  if (!one_value && (float)sel_mass > (float)TOPP_CAND * 1.0995116e12f * __expf(-(float)cut_bin / scale)) {
    histogram([&] {
      visit(-INFINITY, [&](f32x4 v) {
        int at[4];
        unsigned long long q[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in = bin(v[e]) == cut_bin;
          at[e] = (in ? sub(v[e]) : 0) * TOPP_COPIES + copy;
          q[e] = in ? mass(v[e]) : 0;
        }
        add4(at, q);
      });
    });
    cut_sub = (int)sel_digit;
  }
  if (!one_value)
    visit(nan, [&](f32x4 v) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (member(v[e]) && v[e] == v[e]) {
          const int k = cand_n > TOPP_CAND ? TOPP_CAND : atomicAdd(&cand_n, 1);
          const uint32_t key = float_order_key(v[e]);
          if (k < TOPP_CAND) cand[k] = key;
          kmin = min(kmin, key);
          kmax = max(kmax, key);
        }
    });
  for (int o = 32; o > 0; o >>= 1) { kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, o, 64)); kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, o, 64)); }
  if ((tid & 63) == 0) { sh_k[0][wv] = kmin; sh_k[1][wv] = kmax; }
  __syncthreads();
  for (int w = 0; w < TOPP_THREADS / 64; ++w) { kmin = min(kmin, sh_k[0][w]); kmax = max(kmax, sh_k[1][w]); }
  if (cand_n <= TOPP_FEW && kmin != kmax) {   // few keys: each thread sums over all of them what its own one has above and beside it
    __syncthreads();
    const uint32_t key = tid < cand_n ? cand[tid] : 0;
    if (tid < cand_n) topp_hist[tid] = mass(order_key_float(key));
    __syncthreads();
    if (tid < cand_n) {
      unsigned long long over = above, equal = 0;
      for (int j = 0; j < cand_n; ++j) {
        if (cand[j] > key) over += topp_hist[j];
        if (cand[j] == key) equal += topp_hist[j];
      }
      if (over < target && over + equal >= target) { sel_digit = key; sel_above = over; sel_mass = equal; }   // (the same from equal keys)
    }
    __syncthreads();
    kmin = kmax = sel_digit;
    above = sel_above;
  }
  // Radix select of the cut key among the members: the largest key K with mass{key >= K} >= target.  The leading bytes that all of them
  // share are known already, all four where they are equal.
  const int shared_bytes = kmin == kmax ? 4 : __clz((int)(kmin ^ kmax)) >> 3;
  uint32_t prefix = shared_bytes ? kmin >> (32 - 8 * shared_bytes) : 0;
  for (int round = shared_bytes; round < 4; ++round) {
    const int shift = 24 - 8 * round;
    __syncthreads();
    for (int j = tid; j < TOPP_RADIX_COPIES * 256; j += TOPP_THREADS) topp_hist[j] = 0;
    __syncthreads();
    // (a key outside the prefix adds nothing, anywhere)
    const int rcopy = (tid & (TOPP_RADIX_COPIES - 1)) * 256;
    auto digit = [&](uint32_t key) { return rcopy + (int)((key >> shift) & 255u); };
    auto weight = [&](uint32_t key) { return round == 0 || (key >> (shift + 8)) == prefix ? mass(order_key_float(key)) : 0; };
    if (cand_n <= TOPP_CAND) {
      for (int j = tid; j < cand_n; j += TOPP_THREADS) {
        const unsigned long long q = weight(cand[j]);
        if (q) atomicAdd(&topp_hist[digit(cand[j])], q);
      }
    } else {
      visit(-INFINITY, [&](f32x4 v) {
        int at[4];
        unsigned long long q[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) { at[e] = digit(float_order_key(v[e])); q[e] = member(v[e]) ? weight(float_order_key(v[e])) : 0; }
        add4(at, q);
      });
    }
    __syncthreads();
    // thread t of the first four wavefronts owns digit 255 - t; exactly one digit takes the running mass across the target
    unsigned long long h = 0, incl = 0;
    if (tid < 256) {
      for (int j = 0; j < TOPP_RADIX_COPIES; ++j) h += topp_hist[j * 256 + 255 - tid];
      incl = h;
      for (int o = 1; o < 64; o <<= 1) { unsigned long long v = __shfl_up(incl, o, 64); if ((tid & 63) >= o) incl += v; }
      if ((tid & 63) == 63) sh_u64[wv] = incl;
    }
    __syncthreads();
    if (tid < 256) {
      for (int w = 0; w < wv; ++w) incl += sh_u64[w];
      const unsigned long long at = above + incl, before = at - h;
      if (at >= target && before < target) { sel_digit = (uint32_t)(255 - tid); sel_above = before; sel_mass = h; }
    }
    __syncthreads();
    prefix = (prefix << 8) | sel_digit;
    above = sel_above;
  }
  const uint32_t cut = prefix;
  // Keys equal to the cut share one mass, so the last round's bin of the cut -- whose keys are exactly those -- holds
  // their number times that mass; the first `take` of them in index order are kept.  (A mass of zero, far below the
  // maximum: every such key is kept, and their number does not matter.)
  const unsigned long long qc = mass(order_key_float(cut));
  const long long n_ties = qc ? (long long)(sel_mass / qc) : 0;
  const unsigned long long need = target - above;   // > 0: mass still missing once every key above the cut is kept
  const long long take = qc ? (long long)((need + qc - 1) / qc) : (long long)V;   // >= 1
  if (tid == 0) { cut_key[m] = cut; cut_last[m] = V; }   // V: every key equal to the cut is kept
  if (take >= n_ties) return;
  // Only some of the equal keys are kept (exact ties at the cut: rare): their indices are collected and the take-th
  // smallest one closes the kept set.  More ties than the list holds (flat logits): ranks by a scan over contiguous runs.
  __shared__ int tie_list[TOPP_THREADS];
  __shared__ int tie_n;
  if (tid == 0) tie_n = 0;
  __syncthreads();
  if (n_ties <= TOPP_THREADS) {
    for (int i = tid; i < V; i += TOPP_THREADS)
      if (float_order_key(lg[i]) == cut) tie_list[atomicAdd(&tie_n, 1)] = i;
    __syncthreads();
    if (tid < n_ties) {
      const int mine = tie_list[tid];
      int smaller = 0;
      for (int u = 0; u < n_ties; ++u) smaller += tie_list[u] < mine;
      if (smaller == take - 1) cut_last[m] = mine;
    }
    return;
  }
  // each wavefront counts its share of the row, then the one whose share holds the take-th looks for it
  const int share = (V + TOPP_THREADS - 1) / TOPP_THREADS * 64, i0 = wv * share, i1 = min(V, i0 + share), lane = tid & 63;
  auto tie = [&](int i) { return __ballot(i < i1 && float_order_key(lg[min(i, V - 1)]) == cut); };
  int mine = 0, rank = 0;
  for (int i = i0; i < i1; i += 64) mine += __popcll(tie(i + lane));
  if (lane == 0) sh_i[wv] = mine;
  __syncthreads();
  for (int w = 0; w < wv; ++w) rank += sh_i[w];   // ties before this share
  if (rank >= take || take > rank + mine) return;
  for (int i = i0; i < i1; i += 64) {
    const unsigned long long b = tie(i + lane);
    if (rank < take && take <= rank + __popcll(b) && (b >> lane & 1) && rank + __popcll(b & ((1ull << lane) - 1)) == take - 1) cut_last[m] = i + lane;
    rank += __popcll(b);
  }
}

// grid (TOPP_CHUNKS, M), block 256: slice c of row m.  The score that decides is the fp32 one (division by T, two logf), some
// sixty instructions per token in a kernel that the vector unit bounds; so, as in the lm_head's sampler, a thread compares its
// kept tokens by z/ln2 - log2(-log2 u) and evaluates the winner in full.  Both orders agree unless its best two are closer than
// the roundings of two hardware logarithms and of z: below 1e-5 plus 1e-6 of the score's magnitude; within ten times that
// the wavefront evaluates all its kept tokens in full.  Four tokens of which none is kept draw no numbers.  128 rows of 151936
// logits, three quarters of them kept: 62 -> 52 us, 46 with the generator in its present form (philox4x32_10).
__global__ void topp_draw_kernel(float *part, int Mp, const uint32_t *cut_key, const int32_t *cut_last, const float *logits, int64_t ld,
                                 int V, float temperature, uint64_t seed, DrawIds ids) {
  __shared__ SampleAcc sh[4];
  const int c = blockIdx.x, m = blockIdx.y;
  const uint32_t step = draw_step(ids, m), stream = draw_stream(ids, m), cut = cut_key[m];
  const int last = cut_last[m];
  const int v4 = (V + 3) / 4, per = (v4 + TOPP_CHUNKS - 1) / TOPP_CHUNKS, b4 = c * per, e4 = min(v4, b4 + per);
  const float *lg = logits + (int64_t)m * ld;
  const bool aligned = (ld & 3) == 0;
  // the four logits of a group, -inf for those that are not kept (a kept -inf has no mass and no score either)
  auto group = [&](int i4) {
    f32x4 x;
    if (aligned && 4 * i4 + 4 <= V) x = ((const f32x4 *)lg)[i4];
    else
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = 4 * i4 + e < V ? lg[4 * i4 + e] : -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t key = float_order_key(x[e]);
      if (!(key > cut || (key == cut && 4 * i4 + e <= last))) x[e] = -INFINITY;
    }
    return x;
  };
  const float c2 = 1.44269504088896341f / temperature;
  float xm = -INFINITY, sum = 0.f, best = -INFINITY, second = -INFINITY, xbest = 0.f;
  uint32_t wbest = 0;
  int ibest = 0x7fffffff;
  for (int i4 = b4 + threadIdx.x; i4 < e4; i4 += blockDim.x) {
    const f32x4 x = group(i4);
    const float x4 = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    if (!(x4 > -INFINITY)) continue;
    if (x4 > xm) { sum *= __builtin_amdgcn_exp2f((xm - x4) * c2); xm = x4; }
    const u32x4 r = draw4(seed, stream, step, (uint32_t)i4);
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sum += __builtin_amdgcn_exp2f((x[e] - xm) * c2);   // the difference first: as exact at scores of thousands
      const float u = uniform_from_bits(w[e]);
      const float f = fmaf(x[e], c2, -__builtin_amdgcn_logf(-__builtin_amdgcn_logf(u)));
      const bool better = f > best;
      second = __builtin_amdgcn_fmed3f(f, best, second);   // (the smaller of the two others where f is NaN)
      best = better ? f : best;
      xbest = better ? x[e] : xbest;
      wbest = better ? w[e] : wbest;
      ibest = better ? 4 * i4 + e : ibest;
    }
  }
  SampleAcc a = sample_acc_init();
  if (xm > -INFINITY) { a.zmax = xm / temperature; a.zsum = sum; }
  // (everything kept and no score above -inf: no finite logit here, the lowest index among equals as everywhere)
  if (__any(second > best - (1e-4f + 1e-5f * (fabsf(best) + 32.f)) || (cut == 0 && ibest == 0x7fffffff && b4 + (int)threadIdx.x < e4))) {
#pragma unroll 1
    for (int i4 = b4 + threadIdx.x; i4 < e4; i4 += blockDim.x) {
      const f32x4 x = group(i4);
      const u32x4 r = draw4(seed, stream, step, (uint32_t)i4);
#pragma unroll 1
      for (int e = 0; e < 4; ++e) {
        const float z = (e == 0 ? x[0] : e == 1 ? x[1] : e == 2 ? x[2] : x[3]) / temperature;
        const float score = z + gumbel_from_bits(e == 0 ? r.x : e == 1 ? r.y : e == 2 ? r.z : r.w);
        const int i = 4 * i4 + e;
        if (i < V && (score > a.best || (score == a.best && i < a.idx))) { a.best = score; a.zbest = z; a.idx = i; }
      }
    }
  } else if (ibest != 0x7fffffff) {
    a.zbest = xbest / temperature;
    a.best = a.zbest + gumbel_from_bits(wbest);
    a.idx = ibest;
  }
  for (int o = 32; o > 0; o >>= 1) { SampleAcc b = sample_acc_shfl_xor(a, o); sample_acc_merge(a, b); }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) sample_acc_merge(a, sh[w]);
    int64_t o = (int64_t)c * Mp + m, plane = (int64_t)TOPP_CHUNKS * Mp;
    sample_part_store(part, o, plane, a);
  }
}

size_t fast_topp_scratch_floats(int Mp) { return (size_t)5 * TOPP_CHUNKS * Mp + 2 * (size_t)Mp; }

void fast_topp_cut_and_draw(float *scratch, const float *logits, int64_t ld, int M, int Mp, int V, float temperature, float top_p,
                            uint64_t seed, DrawIds ids, hipStream_t st) {
  if (M <= 0) return;
  uint32_t *cut_key = (uint32_t *)(scratch + (size_t)5 * TOPP_CHUNKS * Mp);
  int32_t *cut_last = (int32_t *)cut_key + Mp;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void *)topp_cut_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, TOPP_LDS);
    attr_set = true;
  }
  hipLaunchKernelGGL(topp_cut_kernel, dim3(M), dim3(TOPP_THREADS), TOPP_LDS, st, cut_key, cut_last, logits, ld, V, temperature, top_p);
  hipLaunchKernelGGL(topp_draw_kernel, dim3(TOPP_CHUNKS, M), dim3(256), 0, st, scratch, Mp, cut_key, cut_last, logits, ld, V, temperature,
                     seed, ids);
}

}  // namespace echo
