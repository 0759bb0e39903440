// Debug path: plain fp32 kernels over row-major weights (fp32 or bf16 storage), fp32 activations and an
// fp32 KV cache.  One thread (or one small block) per output, sequential sums; no tiling.  This is the
// "fp32 debug mode" the fast kernels are cross-checked against on the GPU, and the path for fp32 models.
#include <type_traits>

#include "echo_device.h"
#include "echo_kernels.h"

namespace echo {

// Workgroups 0 .. M - 1: a row's embedding; the rest: the rotary table.
template <bool BF>
__global__ void dbg_embed_kernel(float *h, const void *embed, const int32_t *token, int M, int d, RopeTable rope) {
  if ((int)blockIdx.x >= M) {
    rope_entry((float2 *)rope.cs, rope.pos, (blockIdx.x - M) * blockDim.x + threadIdx.x, M, rope.hd / 2, rope.base);
    return;
  }
  int m = blockIdx.x, t = token[m];
  for (int i = threadIdx.x; i < d; i += blockDim.x) h[(int64_t)m * d + i] = t >= 0 ? load_w<BF>(embed, (int64_t)t * d + i) : 0.f;
}

void dbg_embed(float *h, const void *embed, int w_bf16, const int32_t *token, int M, int d, RopeTable rope, hipStream_t st) {
  const dim3 grid(M + (M * (rope.hd / 2) + 255) / 256);
  if (w_bf16) hipLaunchKernelGGL(dbg_embed_kernel<true>, grid, dim3(256), 0, st, h, embed, token, M, d, rope);
  else hipLaunchKernelGGL(dbg_embed_kernel<false>, grid, dim3(256), 0, st, h, embed, token, M, d, rope);
}

__device__ __forceinline__ float dbg_swiglu_of(float g, float u) { return g / (1.0f + expf(-g)) * u; }

__device__ float block_sum_256(float v, float *sh) {
  v = wave_sum(v);
  int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
  return t;
}

template <bool BF>
__global__ void dbg_rmsnorm_kernel(float *x, const float *h, const void *gain, int d, float eps) {
  __shared__ float sh[8];
  int m = blockIdx.x;
  float ss = 0.f;
  for (int i = threadIdx.x; i < d; i += blockDim.x) { float v = h[(int64_t)m * d + i]; ss += v * v; }
  ss = block_sum_256(ss, sh);
  float inv = 1.0f / sqrtf(ss / (float)d + eps);
  for (int i = threadIdx.x; i < d; i += blockDim.x) x[(int64_t)m * d + i] = h[(int64_t)m * d + i] * inv * load_w<BF>(gain, i);
}

void dbg_rmsnorm(float *x, const float *h, const void *gain, int w_bf16, int M, int d, float eps, hipStream_t st) {
  if (w_bf16) hipLaunchKernelGGL(dbg_rmsnorm_kernel<true>, dim3(M), dim3(256), 0, st, x, h, gain, d, eps);
  else hipLaunchKernelGGL(dbg_rmsnorm_kernel<false>, dim3(M), dim3(256), 0, st, x, h, gain, d, eps);
}

// One wavefront per output element: lanes stride over k, then a shuffle reduction.  VEC (K a multiple of 4, aligned
// rows): four elements per lane and load.  A product over a few hundred elements is bound by the latency of a lane's loads, one
// round trip per trip of the loop: MFMA-free and untiled as it is, the tiny model's launches
// (N 256 .. 1024, K 256 and 704, 8 rows) took 3.2 - 5.1 us and take 2.6 - 3.5, an empty launch 2 - 3.
// PRO: what makes the operand of X's rows: DBG_PLAIN the row itself; DBG_NORM its RMS norm, by the sums of dbg_rmsnorm_kernel, which every
// workgroup repeats; DBG_SWIGLU silu(gate) * up of a row [gate | up].  Repeated in every workgroup they cost more than a launch of their own
// once there are many rows, see dbg_fuses.
template <bool BF, bool VEC, int PRO>
__global__ void dbg_gemm_kernel(float *__restrict__ Y, const float *__restrict__ X, const void *__restrict__ W, int M, int N, int K, int accumulate,
                                const void *__restrict__ gain, float eps) {
  int n = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  int m = blockIdx.y, lane = threadIdx.x & 63;
  const float *x = X + (int64_t)m * K * (PRO == DBG_SWIGLU ? 2 : 1);
  float inv = 1.f;
  if (PRO == DBG_NORM) {
    __shared__ float sh[8];
    float ss = 0.f;
    for (int i = threadIdx.x; i < K; i += blockDim.x) ss += x[i] * x[i];
    inv = 1.0f / sqrtf(block_sum_256(ss, sh) / (float)K + eps);
  }
  if (n >= N) return;
  const int64_t o = (int64_t)m * N + n;
  const float y = accumulate && lane == 0 ? Y[o] : 0.f;
  auto four = [&](const void *p, int64_t k) {   // four values in the weights' type
    if (!BF) return *(const f32x4 *)((const float *)p + k);
    const uint2 b = *(const uint2 *)((const uint16_t *)p + k);
    return f32x4{__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u), __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xffff0000u)};
  };
  float acc = 0.f;
  if (VEC) {
    f32x4 a4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int k = lane * 4; k < K; k += 256) {
      const f32x4 w = four(W, (int64_t)n * K + k);
      f32x4 v = *(const f32x4 *)(x + k);
      if (PRO == DBG_NORM) {
        v = v * inv * four(gain, k);
      } else if (PRO == DBG_SWIGLU) {
        const f32x4 u = *(const f32x4 *)(x + K + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = dbg_swiglu_of(v[e], u[e]);
      }
      a4 += w * v;
    }
    acc = (a4[0] + a4[1]) + (a4[2] + a4[3]);
  } else {
    for (int k = lane; k < K; k += 64) {
      float v = x[k];
      if (PRO == DBG_NORM) v = v * inv * load_w<BF>(gain, k);
      else if (PRO == DBG_SWIGLU) v = dbg_swiglu_of(v, x[K + k]);
      acc += load_w<BF>(W, (int64_t)n * K + k) * v;
    }
  }
  acc = wave_sum(acc);
  if (lane == 0) Y[o] = y + acc;
}

void dbg_gemm(float *Y, const float *X, const void *W, int w_bf16, int M, int N, int K, int accumulate, hipStream_t st, DbgOperand pro, const void *gain,
              float eps) {
  dim3 grid((N + 3) / 4, M), block(256);
  const int unit = w_bf16 ? 8 : 16;
  const bool vec = K % 4 == 0 && (uintptr_t)W % unit == 0 && (uintptr_t)X % 16 == 0 && (uintptr_t)gain % unit == 0;
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, st, Y, X, W, M, N, K, accumulate, gain, eps); };
  auto pick = [&](auto tag) {
    constexpr int P = decltype(tag)::value;
    if (w_bf16) { if (vec) launch(dbg_gemm_kernel<true, true, P>); else launch(dbg_gemm_kernel<true, false, P>); }
    else { if (vec) launch(dbg_gemm_kernel<false, true, P>); else launch(dbg_gemm_kernel<false, false, P>); }
  };
  if (pro == DBG_NORM) pick(std::integral_constant<int, DBG_NORM>{});
  else if (pro == DBG_SWIGLU) pick(std::integral_constant<int, DBG_SWIGLU>{});
  else pick(std::integral_constant<int, DBG_PLAIN>{});
}

__device__ __forceinline__ float2 dbg_rotate(float a, float b, float2 cs) { return make_float2(a * cs.x - b * cs.y, a * cs.y + b * cs.x); }

// grid (M, Hq + 2*Hkv), block hd/2 threads (<= 128) rounded up to whole wavefronts (the norm's sum shuffles over all 64 lanes):
// optional per-head RMSNorm, rotary embedding on q and k, append k and v to the fp32 cache.
template <bool BF>
__global__ void dbg_qkv_post_kernel(float *qkv, const void *q_gain, const void *k_gain, int qk_norm, float eps,
                                    const float2 *rope_cs, RowState rows, KvGeom kv, int layer, int Hq, int Hkv) {
  __shared__ float sh[8];
  int m = blockIdx.x, j = blockIdx.y, hd = kv.head_dim, half = hd / 2, i = threadIdx.x;
  int width = (Hq + 2 * Hkv) * hd;
  float *v = qkv + (int64_t)m * width + (int64_t)j * hd;
  bool is_q = j < Hq, is_k = !is_q && j < Hq + Hkv;
  const bool on = i < half;
  float a = on ? v[i] : 0.f, b = on ? v[i + half] : 0.f;
  if (is_q || is_k) {
    if (qk_norm) {
      float ss = a * a + b * b;
      ss = wave_sum(ss);
      if (blockDim.x > 64) {  // hd > 128: two wavefronts
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
        __syncthreads();
        ss = sh[0] + sh[1];
      }
      float inv = 1.0f / sqrtf(ss / (float)hd + eps);
      if (!on) return;
      const void *g = is_q ? q_gain : k_gain;
      a = a * inv * load_w<BF>(g, i);
      b = b * inv * load_w<BF>(g, i + half);
    }
    if (!on) return;
    const float2 r = dbg_rotate(a, b, rope_cs[(int64_t)m * half + i]);
    a = r.x; b = r.y;
  }
  if (is_q) { v[i] = a; v[i + half] = b; return; }
  if (!on || !rows.active[m]) return;
  int kvh = is_k ? j - Hq : j - Hq - Hkv;
  float *dst = (float *)kv.base + (int64_t)rows.slot[m] * kv.slot_stride() + (int64_t)layer * kv.layer_stride() +
               (is_k ? 0 : kv.kv_stride()) + (int64_t)kvh * kv.head_stride() + (int64_t)rows.pos[m] * hd;
  dst[i] = a; dst[i + half] = b;
}

void dbg_qkv_post(float *qkv, const void *q_gain, const void *k_gain, int w_bf16, int qk_norm, float eps,
                  const float *rope_cs, RowState rows, KvGeom kv, int layer, int M, int Hq, int Hkv, hipStream_t st) {
  dim3 grid(M, Hq + 2 * Hkv), block((kv.head_dim / 2 + 63) / 64 * 64);
  if (w_bf16) hipLaunchKernelGGL(dbg_qkv_post_kernel<true>, grid, block, 0, st, qkv, q_gain, k_gain, qk_norm, eps,
                                 (const float2 *)rope_cs, rows, kv, layer, Hq, Hkv);
  else hipLaunchKernelGGL(dbg_qkv_post_kernel<false>, grid, block, 0, st, qkv, q_gain, k_gain, qk_norm, eps,
                          (const float2 *)rope_cs, rows, kv, layer, Hq, Hkv);
}

// grid (M, Hq), one wavefront: scores to LDS (dynamic, max_ctx floats), max, exp/sum, weighted sum of V.
// OWN: a decode pass, whose rows are different sequences and so read no key of one another's: the workgroup does dbg_qkv_post_kernel's work
// on its query head and on its KV head's new key and value, which it keeps for itself; the first query head of a KV head appends
// them to the cache.  One dependent launch less per layer: 8 rows, 4 heads of 64: 2.2 + 5.0 -> 5.7 us.
template <bool OWN, bool BF>
__global__ void dbg_attention_kernel(float *out, const float *qkv, RowState rows, KvGeom kv, int layer, int Hq, int Hkv, DbgHeads hp) {
  extern __shared__ float sc[];
  __shared__ __attribute__((aligned(16))) float own[2][256];   // OWN: the query, the new key
  int m = blockIdx.x, j = blockIdx.y, lane = threadIdx.x, hd = kv.head_dim;
  float *o = out + ((int64_t)m * Hq + j) * hd;
  if (!rows.active[m]) { for (int i = lane; i < hd; i += 64) o[i] = 0.f; return; }
  int width = (Hq + 2 * Hkv) * hd, n_keys = rows.pos[m] + 1, kvh = j / (Hq / Hkv);
  const float *q = qkv + (int64_t)m * width + (int64_t)j * hd, *v_new = qkv + (int64_t)m * width + (int64_t)(Hq + Hkv + kvh) * hd;
  const float *K = (const float *)kv.base + (int64_t)rows.slot[m] * kv.slot_stride() + (int64_t)layer * kv.layer_stride() +
                   (int64_t)kvh * kv.head_stride();
  const float *V = K + kv.kv_stride();
  if (OWN) {
    const float *k_raw = qkv + (int64_t)m * width + (int64_t)(Hq + kvh) * hd;
    for (int w = 0; w < 2; ++w) {
      const float *src = w ? k_raw : q;
      float ss = 0.f;
      if (hp.qk_norm) {
        for (int i0 = 0; i0 < hd / 2; i0 += 64) {
          const int i = i0 + lane;
          const float a = i < hd / 2 ? src[i] : 0.f, b = i < hd / 2 ? src[i + hd / 2] : 0.f;
          ss += wave_sum(a * a + b * b);
        }
      }
      const float inv = 1.0f / sqrtf(ss / (float)hd + hp.eps);
      for (int i = lane; i < hd / 2; i += 64) {
        float a = src[i], b = src[i + hd / 2];
        if (hp.qk_norm) {
          const void *g = w ? hp.k_gain : hp.q_gain;
          a = a * inv * load_w<BF>(g, i);
          b = b * inv * load_w<BF>(g, i + hd / 2);
        }
        const float2 r = dbg_rotate(a, b, hp.rope[(int64_t)m * (hd / 2) + i]);
        own[w][i] = r.x; own[w][i + hd / 2] = r.y;
      }
    }
    __syncthreads();
    if (j % (Hq / Hkv) == 0) {
      float *K_new = const_cast<float *>(K) + (int64_t)(n_keys - 1) * hd, *V_new = const_cast<float *>(V) + (int64_t)(n_keys - 1) * hd;
      for (int i = lane; i < hd; i += 64) { K_new[i] = own[1][i]; V_new[i] = v_new[i]; }
    }
    q = own[0];
  }
  float scale = 1.0f / sqrtf((float)hd), mx = -INFINITY;
  for (int t = lane; t < n_keys; t += 64) {
    float s = 0.f;
    const float *key = OWN && t == n_keys - 1 ? own[1] : K + (int64_t)t * hd;
    if (hd % 4 == 0) {   // a key's dims four at a time, several loads in flight (the sum keeps its order)
#pragma unroll 8
      for (int i = 0; i < hd; i += 4) {
        const f32x4 k4 = *(const f32x4 *)(key + i), q4 = *(const f32x4 *)(q + i);
        s += q4[0] * k4[0]; s += q4[1] * k4[1]; s += q4[2] * k4[2]; s += q4[3] * k4[3];
      }
    } else {
      for (int i = 0; i < hd; ++i) s += q[i] * key[i];
    }
    s *= scale;
    sc[t] = s;
    mx = fmaxf(mx, s);
  }
  mx = wave_max(mx);
  float den = 0.f;
  for (int t = lane; t < n_keys; t += 64) { float e = expf(sc[t] - mx); sc[t] = e; den += e; }
  den = wave_sum(den);
  __syncthreads();
  for (int i = lane; i < hd; i += 64) {
    float acc = 0.f;
#pragma unroll 16
    for (int t = 0; t < n_keys - (OWN ? 1 : 0); ++t) acc += sc[t] * V[(int64_t)t * hd + i];
    if (OWN) acc += sc[n_keys - 1] * v_new[i];
    o[i] = acc / den;
  }
}

void dbg_attention(float *out, const float *qkv, RowState rows, KvGeom kv, int layer, int M, int Hq, int Hkv, hipStream_t st, const DbgHeads *own, int w_bf16) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(M, Hq), dim3(64), (size_t)kv.max_ctx * sizeof(float), st, out, qkv, rows, kv, layer, Hq, Hkv, own ? *own : DbgHeads{});
  };
  if (!own) launch(dbg_attention_kernel<false, false>);
  else if (w_bf16) launch(dbg_attention_kernel<true, true>);
  else launch(dbg_attention_kernel<true, false>);
}

__global__ void dbg_swiglu_kernel(float *ff, const float *gu, int M, int F) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)M * F) return;
  int64_t m = idx / F, f = idx % F;
  ff[idx] = dbg_swiglu_of(gu[m * 2 * F + f], gu[m * 2 * F + F + f]);
}

void dbg_swiglu(float *ff, const float *gu, int M, int F, hipStream_t st) {
  int64_t n = (int64_t)M * F;
  hipLaunchKernelGGL(dbg_swiglu_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, ff, gu, M, F);
}

// grid (slices, M), block 256: Gumbel-max token and log softmax(z)[token] from materialised logits, every entry evaluated in
// full.  One slice per row: the token and its log-prob; more: the slice's running state, in the partial layout of the fused
// sampler.  The serial chain of a thread (two logf, an expf and a division per entry) bounds it, so a large vocabulary is cut into
// slices: 151936 entries, 6 rows: 245 -> 21 us, and 4 us for the merge.
__global__ void dbg_sample_kernel(int32_t *tok, float *lp, float *part, int Mp, const float *logits, int64_t ld, int V, float temperature,
                                  uint64_t seed, DrawIds ids, StepBook book) {
  __shared__ SampleAcc sh[4];
  const int c = blockIdx.x, slices = gridDim.x, m = blockIdx.y;
  const uint32_t s = draw_step(ids, m), stream = draw_stream(ids, m);
  const int v4 = (V + 3) / 4, per = (v4 + slices - 1) / slices, e4 = min(v4, (c + 1) * per);
  SampleAcc a = sample_acc_init();
  const float *lg = logits + (int64_t)m * ld;
  for (int i4 = c * per + threadIdx.x; i4 < e4; i4 += blockDim.x) {
    u32x4 r = draw4(seed, stream, s, (uint32_t)i4);
    uint32_t w[4] = {r.x, r.y, r.z, r.w};
    for (int e = 0; e < 4; ++e) {
      int i = i4 * 4 + e;
      if (i >= V) break;
      float z = lg[i] / temperature;
      sample_acc_add(a, z, z + gumbel_from_bits(w[e]), i);
    }
  }
  for (int o = 32; o > 0; o >>= 1) { SampleAcc b = sample_acc_shfl_xor(a, o); sample_acc_merge(a, b); }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) sample_acc_merge(a, sh[w]);
    if (slices == 1) {
      tok[m] = a.idx;
      lp[m] = a.zbest - (a.zmax + logf(a.zsum));
      if (book.d_step) book_row(book, m, a.idx, lp[m]);
    } else {
      const int64_t o = (int64_t)c * Mp + m, plane = (int64_t)slices * Mp;
      sample_part_store(part, o, plane, a);
    }
  }
}

void dbg_sample(int32_t *tok, float *lp, float *scratch, int Mp, const float *logits, int64_t ld, int M, int V, float temperature, uint64_t seed,
                DrawIds ids, const StepBook &book, hipStream_t st) {
  // a second launch (about 5 us) pays once a thread has more than a few entries (of 4) to itself
  const int slices = V > 8192 ? TOPP_CHUNKS_PER_ROW : 1;
  hipLaunchKernelGGL(dbg_sample_kernel, dim3(slices, M), dim3(256), 0, st, tok, lp, scratch, Mp, logits, ld, V, temperature, seed, ids, book);
  if (slices > 1) fast_sample_combine(tok, lp, scratch, slices, M, Mp, book, st);
}

__global__ void dbg_target_logprob_kernel(float *lp, const float *logits, int64_t ld, int V, float temperature,
                                          const int32_t *target) {
  __shared__ float sh[8];
  int m = blockIdx.x, t = target[m];
  if (t < 0) { if (threadIdx.x == 0) lp[m] = 0.f; return; }
  const float *lg = logits + (int64_t)m * ld;
  float mx = -INFINITY;
  for (int i = threadIdx.x; i < V; i += blockDim.x) mx = fmaxf(mx, lg[i] / temperature);
  mx = wave_max(mx);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
  float den = 0.f;
  for (int i = threadIdx.x; i < V; i += blockDim.x) den += expf(lg[i] / temperature - mx);
  den = block_sum_256(den, sh + 4);
  if (threadIdx.x == 0) lp[m] = lg[t] / temperature - (mx + logf(den));
}

void dbg_target_logprob(float *lp, const float *logits, int64_t ld, int M, int V, float temperature,
                        const int32_t *target, hipStream_t st) {
  hipLaunchKernelGGL(dbg_target_logprob_kernel, dim3(M), dim3(256), 0, st, lp, logits, ld, V, temperature, target);
}

}  // namespace echo
