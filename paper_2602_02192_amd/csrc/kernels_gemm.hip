// MFMA path, dense contractions: weight repacking, the weight-streaming GEMM (split-K over the
// wavefronts of a workgroup and over the grid) with its epilogues, and the lm_head GEMM whose epilogue
// is the sampler (temperature, Gumbel-max, running log-sum-exp), so logits never reach HBM.
//
// Operand roles of v_mfma_f32_32x32x16_f16 here: A = 32 weight rows x 16 k, B = 16 k x 32 batch rows.
// Lane l supplies A[row l%32][k 8*(l/32) .. +8] and B[k 8*(l/32) .. +8][col l%32]; it receives
// D[row 8*g + 4*(l/32) + i][col l%32] in accumulator register 4*g + i (g, i in 0..3).
#include <type_traits>

#include "echo_device.h"
#include "echo_kernels.h"

namespace echo {

// Packed weight addressing, in units of 16 bytes (8 halves): one 32-row block is contiguous over K, a k-step of it is 64 units.
__host__ __device__ __forceinline__ int64_t w_block_base(int nb, int Kp) { return (int64_t)nb * (Kp >> 3) * 32; }
constexpr int64_t W_KSTEP = 64;

// ---- weight repacking --------------------------------------------------------------------------------
// src: row-major bf16 [n_rows][K]; destination row of source row i is dst_row0 + i*dst_row_stride.
__global__ void pack_weight_kernel(uint4 *dst, const uint4 *src, int64_t dst_row0, int dst_row_stride, int64_t n_rows,
                                   int K8, int Kp8, int Np) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_rows * K8) return;
  int64_t i = idx / K8;
  int k8 = (int)(idx % K8);
  int64_t r = dst_row0 + i * dst_row_stride;
  uint4 v = src[idx];
  uint32_t w[4] = {v.x, v.y, v.z, v.w}, o[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)   // bf16 pair -> half pair, scaled by W_SCALE (exact)
    o[q] = (uint32_t)f32_to_h16_bits(__uint_as_float(w[q] << 16) * W_SCALE) |
           ((uint32_t)f32_to_h16_bits(__uint_as_float(w[q] & 0xffff0000u) * W_SCALE) << 16);
  dst[w_block_base((int)(r >> 5), Kp8 * 8) + (k8 >> 1) * W_KSTEP + (k8 & 1) * 32 + (r & 31)] = make_uint4(o[0], o[1], o[2], o[3]);
}

void fast_pack_weight(void *dst, const void *src, int64_t dst_row0, int dst_row_stride, int64_t n_rows, int K, int Kp,
                      int Np, hipStream_t st) {
  int64_t n = n_rows * (K / 8);
  if (n <= 0) return;
  hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (uint4 *)dst,
                     (const uint4 *)src, dst_row0, dst_row_stride, n_rows, K / 8, Kp / 8, Np);
}

// Re-pack a span of a matrix: elements [e0, e0 + n) of the row-major bf16 matrix [rows][K] (src holds just those n
// values) replace their places in the packed weight; source row i lives in destination row dst_row0 + i * stride.
// One thread per destination unit of 8 k that the span touches; a unit covered only in part keeps its other values.
__global__ void pack_span_kernel(uint16_t *dst, const uint16_t *src, int64_t e0, int64_t n, int64_t dst_row0, int dst_row_stride, int K,
                                 int Kp8, int Np) {
  const int64_t u0 = e0 >> 3, u = u0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // K % 8 == 0: units never straddle rows
  if (u * 8 >= e0 + n) return;
  const int K8 = K >> 3;
  const int64_t i = u / K8, r = dst_row0 + i * dst_row_stride;
  const int k8 = (int)(u % K8);
  uint16_t *d = dst + (w_block_base((int)(r >> 5), Kp8 * 8) + (k8 >> 1) * W_KSTEP + (k8 & 1) * 32 + (r & 31)) * 8;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int64_t e = u * 8 + q;
    if (e >= e0 && e < e0 + n) d[q] = f32_to_h16_bits(bf16_bits_to_f32(src[e - e0]) * W_SCALE);
  }
}

void fast_pack_span(void *dst, const void *src, int64_t e0, int64_t n, int64_t dst_row0, int dst_row_stride, int K, int Kp, int Np,
                    hipStream_t st) {
  if (n <= 0) return;
  const int64_t units = ((e0 + n + 7) >> 3) - (e0 >> 3);
  hipLaunchKernelGGL(pack_span_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, st, (uint16_t *)dst, (const uint16_t *)src, e0, n,
                     dst_row0, dst_row_stride, K, Kp / 8, Np);
}

// A quantised matrix (per-row fp32 scale, int8 codes) back to row-major bf16: the bf16 value nearest to float(code) * scale,
// computed as one fp32 product, ties to even.  One thread per code.
__global__ void dequant_q8_kernel(uint16_t *__restrict__ out, const int8_t *__restrict__ codes, const float *__restrict__ scales,
                                  int64_t n, int K) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  out[i] = f32_to_bf16_bits(__fmul_rn((float)codes[i], scales[i / K]));
}

void fast_dequant_q8(void *out_bf16, const void *codes, const void *scales, int64_t rows, int K, hipStream_t st) {
  const int64_t n = rows * K;
  if (n <= 0) return;
  hipLaunchKernelGGL(dequant_q8_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (uint16_t *)out_bf16, (const int8_t *)codes,
                     (const float *)scales, n, K);
}

// ---- weight-streaming GEMM with the activations staged through LDS -----------------------------------------
// Measured on MI355X: a compute unit sustains about 48 GB/s of vector-memory reads whether they come from HBM
// (weights) or from L2 (activations), so activation re-reads cost as much as weight bytes.  Here the WN wavefronts
// of a workgroup own WN consecutive 32-row weight blocks and walk the same k-range in chunks of KC k-steps; a
// chunk of activations (KC x MB KiB) is fetched once per workgroup, coalesced, and shared through LDS, which cuts
// the activation traffic per weight byte to MB/WN.  Weight loads run NSTAGE-1 chunks ahead in registers.  The
// activation loads of a chunk are issued before the weight loads of the same chunk: the memory counter retires in
// order, so waiting for them (to copy them into LDS) leaves every younger weight load in flight.
// grid (ceil(Np/32 / WN), nsplit); 32*MB batch rows, up to 128; block 64*WN; chunks_per_split chunks of KC k-steps per grid split.
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));

// The SwiGLU products of a 32 x 32 accumulator tile whose weight rows alternate gate_f, up_f: 16 features, of which a lane gets the eight of K8
// group `half` of its batch row.  (It holds features 4g + 2 half + {0, 1}: the two lanes of a row exchange what the other's group needs.)
// With the matrix cores idle this is time on top of the main loop, 2121 vector instructions per wavefront of a 256 x 256 ring tile while it was
// expf, a division and shuffles through LDS, 1477 now, same bits.  4096 rows, gate/up of the 4B / 8B / 32B shapes: 374 / 679 / 1735 -> 372 / 666 / 1711
// us, 1024 rows of the 4B shape 134.8 -> 130.7.
__device__ __forceinline__ u32x4v swiglu_unit(const f32x16 &acc) {
  uint32_t pk[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) pk[g] = f32_to_h16_pair(swiglu(acc[4 * g], acc[4 * g + 1]), swiglu(acc[4 * g + 2], acc[4 * g + 3]));
  const auto x0 = __builtin_amdgcn_permlane32_swap(pk[0], pk[2], false, false), x1 = __builtin_amdgcn_permlane32_swap(pk[1], pk[3], false, false);
  return u32x4v{x0[0], x0[1], x1[0], x1[1]};
}

constexpr int GEMM_KC = 8;   // k-steps per chunk
template <int MB, int WN> struct GemmLds {
  static constexpr int KC = GEMM_KC;
  static constexpr int CHUNK_UNITS = KC * 2 * 32 * MB;                  // 16-byte units of one activation chunk
  static constexpr int X_BYTES = 2 * CHUNK_UNITS * 16;                   // double buffer
  static constexpr int TILE_STRIDE = 36;                                 // floats per row of the transposed output tile, see transpose_in
  static constexpr int EPI_BYTES = WN * 32 * TILE_STRIDE * 4;            // one 32 x 32 tile per wavefront at a time
  static constexpr int BYTES = X_BYTES > EPI_BYTES ? X_BYTES : EPI_BYTES;
};

// A 32 x 32 accumulator tile to LDS as [batch row][weight row], scaled back, in 16-byte stores: with 36 floats per row the sixteen-byte
// slots of eight neighbouring lanes lie on all banks, here and in row-wise 16-byte reads.
template <int STRIDE> __device__ __forceinline__ void transpose_in(float *tile, const f32x16 &acc, int half, int col) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 v = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    *(f32x4 *)(tile + col * STRIDE + 8 * g + 4 * half) = v * W_UNSCALE;
  }
}

// The GEMM kernel's main loop as a function, for the lm_head (the GEMM kernel keeps its own inline copy: hipcc
// schedules the inlined function measurably worse there): accumulates, for weight block `nb` and the 32*MB batch rows,
// the k-range of `nchunks` chunks starting at chunk c_begin.  Ends with a workgroup barrier, after which the
// LDS buffers are free for the epilogue.
template <int MB, int WN, int NSTAGE>
__device__ __forceinline__ void gemm_lds_mainloop(f32x16 (&acc)[MB], char *lds_raw, const u32x4v *__restrict__ Xp,
                                                  const h16x8 *__restrict__ Wp, int Mp, int Np, int Kp, int nb, int c_begin,
                                                  int nchunks) {
  using L = GemmLds<MB, WN>;
  constexpr int KC = L::KC, T = WN * 64, XU = L::CHUNK_UNITS, XL = (XU + T - 1) / T, ROWS = 32 * MB;
  u32x4v *xs = (u32x4v *)lds_raw;
  const int lane = threadIdx.x & 63, tid = threadIdx.x;
  const h16x8 *a_ptr = Wp + w_block_base(nb, Kp) + (int64_t)c_begin * KC * W_KSTEP + (lane >> 5) * 32 + (lane & 31);
  const int64_t a_step = W_KSTEP;
#pragma unroll
  for (int j = 0; j < MB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  h16x8 a[NSTAGE][KC];
  u32x4v xr[NSTAGE][XL];
  auto load_a = [&](int st, int c) {
#pragma unroll
    for (int u = 0; u < KC; ++u) a[st][u] = __builtin_nontemporal_load(a_ptr + (int64_t)(c * KC + u) * a_step);
  };
  // unit i of a chunk: k8 group i / ROWS (two per k-step), batch row i % ROWS
  auto load_x = [&](int st, int c) {
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      int idx = min(i * T + tid, XU - 1);   // surplus threads repeat the last unit: no divergent branch around a load
      xr[st][i] = Xp[(int64_t)((c_begin + c) * KC * 2 + idx / ROWS) * Mp + idx % ROWS];
    }
  };
  auto store_x = [&](int st, int buf) {
#pragma unroll
    for (int i = 0; i < XL; ++i) xs[buf * XU + min(i * T + tid, XU - 1)] = xr[st][i];
  };
  // The B operands of GU k-steps are read from LDS in one batch ahead of their MFMAs: with one wavefront per SIMD
  // nothing else hides the LDS latency, and a read issued right before each MFMA would expose it every time.
  auto compute = [&](int st, int buf) {
    constexpr int GU = MB == 4 ? (WN > 4 ? 2 : 4) : KC;
    const u32x4v *bp = xs + buf * XU + (lane >> 5) * ROWS + (lane & 31);
#pragma unroll
    for (int u0 = 0; u0 < KC; u0 += GU) {
      u32x4v b[GU][MB];
#pragma unroll
      for (int u = 0; u < GU; ++u)
#pragma unroll
        for (int j = 0; j < MB; ++j) b[u][j] = bp[(u0 + u) * 2 * ROWS + j * 32];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < GU; ++u)
#pragma unroll
        for (int j = 0; j < MB; ++j) acc[j] = mfma_h16(a[st][u0 + u], __builtin_bit_cast(h16x8, b[u][j]), acc[j]);
    }
  };
  // Every load that the compiler sees behind a condition makes its wait counts assume the load was not issued, and
  // the waits that follow drain the queue.  So the pipeline is written without conditions around loads: prologue,
  // steady trips of NSTAGE chunks, and one straight-line tail per possible number of remaining chunks.
  auto tail = [&](auto r_tag) {
    constexpr int R = decltype(r_tag)::value;   // chunks left; chunk i of them sits in register stage i % NSTAGE
    const int cb = nchunks - R;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (i + NSTAGE - 1 < R) { load_x((i + NSTAGE - 1) % NSTAGE, cb + i + NSTAGE - 1); load_a((i + NSTAGE - 1) % NSTAGE, cb + i + NSTAGE - 1); }
      compute(i % NSTAGE, (cb + i) & 1);
      if (i + 1 < R) store_x((i + 1) % NSTAGE, (cb + i + 1) & 1);
      __syncthreads();
    }
  };
  if (nchunks >= NSTAGE - 1) {
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s) { load_x(s, s); load_a(s, s); }
    store_x(0, 0);
    __syncthreads();
    int c0 = 0;
    for (; c0 + 2 * NSTAGE - 2 < nchunks; c0 += NSTAGE) {
#pragma unroll
      for (int s = 0; s < NSTAGE; ++s) {
        const int c = c0 + s;
        load_x((s + NSTAGE - 1) % NSTAGE, c + NSTAGE - 1);
        load_a((s + NSTAGE - 1) % NSTAGE, c + NSTAGE - 1);
        compute(s, c & 1);
        store_x((s + 1) % NSTAGE, (c + 1) & 1);
        __syncthreads();
      }
    }
    // NSTAGE-1 .. 2*NSTAGE-2 chunks are left and c0 is a multiple of NSTAGE, so their register stages are static
    static_assert(NSTAGE == 2 || NSTAGE == 3, "one tail per remaining count");
    switch (nchunks - c0) {
      case 1: if (NSTAGE == 2) tail(std::integral_constant<int, 1>{}); break;
      case 2: tail(std::integral_constant<int, 2>{}); break;
      case 3: if (NSTAGE == 3) tail(std::integral_constant<int, 3>{}); break;
      case 4: if (NSTAGE == 3) tail(std::integral_constant<int, 4>{}); break;
      default: break;
    }
  } else if (nchunks > 0) {   // a K range shorter than the pipeline: guarded loads
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s)
      if (s < nchunks) { load_x(s, s); load_a(s, s); }
    store_x(0, 0);
    __syncthreads();
    for (int c0 = 0; c0 < nchunks; c0 += NSTAGE) {
#pragma unroll
      for (int s = 0; s < NSTAGE; ++s) {
        const int c = c0 + s;
        if (c < nchunks) {
          if (c + NSTAGE - 1 < nchunks) { load_x((s + NSTAGE - 1) % NSTAGE, c + NSTAGE - 1); load_a((s + NSTAGE - 1) % NSTAGE, c + NSTAGE - 1); }
          compute(s, c & 1);
          if (c + 1 < nchunks) store_x((s + 1) % NSTAGE, (c + 1) & 1);
          __syncthreads();
        }
      }
    }
  }
}

// The 64-row forms with the two-chunk weight pipeline are held to 256 registers per lane (the bound that would let two
// workgroups share a compute unit; these launches have at most one per unit): the code the compiler makes under that
// bound parks nothing in the accumulation half of the register file and measured 0.9 % faster per decode step of the 4B
// model, level on the 32B model.  At 32 rows the bound changes nothing, at 128 rows it forces spills.
template <int MB, int WN, int NSTAGE> constexpr int gemm_lds_min_wgs() { return MB == 2 && NSTAGE == 2 && WN <= 4 ? 2 : 1; }

template <int MB, int WN, int NSTAGE, int EPI>
__global__ __launch_bounds__(WN * 64, (gemm_lds_min_wgs<MB, WN, NSTAGE>())) void gemm_lds_kernel(void *out, const u32x4v *__restrict__ Xp, const h16x8 *__restrict__ Wp,
                                                           int Mp, int Np, int Kp, int chunks_per_split) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  using L = GemmLds<MB, WN>;
  constexpr int KC = L::KC, T = WN * 64, XU = L::CHUNK_UNITS, XL = (XU + T - 1) / T, ROWS = 32 * MB;
  u32x4v *xs = (u32x4v *)lds_raw;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, tid = threadIdx.x;
  const int nblocks = Np >> 5, total_chunks = (Kp >> 4) / KC;
  const int nb_own = blockIdx.x * WN + w, nb = min(nb_own, nblocks - 1);   // wavefronts past the end re-read the last block
  const int c_begin = blockIdx.y * chunks_per_split, nchunks = min(chunks_per_split, total_chunks - c_begin);
  const h16x8 *a_ptr = Wp + w_block_base(nb, Kp) + (int64_t)c_begin * KC * W_KSTEP + (lane >> 5) * 32 + (lane & 31);
  const int64_t a_step = W_KSTEP;
  f32x16 acc[MB];
#pragma unroll
  for (int j = 0; j < MB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  h16x8 a[NSTAGE][KC];
  u32x4v xr[NSTAGE][XL];
  auto load_a = [&](int st, int c) {
#pragma unroll
    for (int u = 0; u < KC; ++u) a[st][u] = __builtin_nontemporal_load(a_ptr + (int64_t)(c * KC + u) * a_step);
  };
  // unit i of a chunk: k8 group i / ROWS (two per k-step), batch row i % ROWS
  auto load_x = [&](int st, int c) {
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      int idx = min(i * T + tid, XU - 1);   // surplus threads repeat the last unit: no divergent branch around a load
      xr[st][i] = Xp[(int64_t)((c_begin + c) * KC * 2 + idx / ROWS) * Mp + idx % ROWS];
    }
  };
  auto store_x = [&](int st, int buf) {
#pragma unroll
    for (int i = 0; i < XL; ++i) xs[buf * XU + min(i * T + tid, XU - 1)] = xr[st][i];
  };
  // The B operands of GU k-steps are read from LDS in one batch ahead of their MFMAs: with one wavefront per SIMD
  // nothing else hides the LDS latency, and a read issued right before each MFMA would expose it every time.
  auto compute = [&](int st, int buf) {
    constexpr int GU = MB == 4 ? (WN > 4 ? 2 : 4) : KC;
    const u32x4v *bp = xs + buf * XU + (lane >> 5) * ROWS + (lane & 31);
#pragma unroll
    for (int u0 = 0; u0 < KC; u0 += GU) {
      u32x4v b[GU][MB];
#pragma unroll
      for (int u = 0; u < GU; ++u)
#pragma unroll
        for (int j = 0; j < MB; ++j) b[u][j] = bp[(u0 + u) * 2 * ROWS + j * 32];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < GU; ++u)
#pragma unroll
        for (int j = 0; j < MB; ++j) acc[j] = mfma_h16(a[st][u0 + u], __builtin_bit_cast(h16x8, b[u][j]), acc[j]);
    }
  };
  // Every load that the compiler sees behind a condition makes its wait counts assume the load was not issued, and
  // the waits that follow drain the queue.  So the pipeline is written without conditions around loads: prologue,
  // steady trips of NSTAGE chunks, and one straight-line tail per possible number of remaining chunks.
  auto tail = [&](auto r_tag) {
    constexpr int R = decltype(r_tag)::value;   // chunks left; chunk i of them sits in register stage i % NSTAGE
    const int cb = nchunks - R;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (i + NSTAGE - 1 < R) { load_x((i + NSTAGE - 1) % NSTAGE, cb + i + NSTAGE - 1); load_a((i + NSTAGE - 1) % NSTAGE, cb + i + NSTAGE - 1); }
      compute(i % NSTAGE, (cb + i) & 1);
      if (i + 1 < R) store_x((i + 1) % NSTAGE, (cb + i + 1) & 1);
      __syncthreads();
    }
  };
  if (nchunks >= NSTAGE - 1) {
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s) { load_x(s, s); load_a(s, s); }
    store_x(0, 0);
    __syncthreads();
    int c0 = 0;
    for (; c0 + 2 * NSTAGE - 2 < nchunks; c0 += NSTAGE) {
#pragma unroll
      for (int s = 0; s < NSTAGE; ++s) {
        const int c = c0 + s;
        load_x((s + NSTAGE - 1) % NSTAGE, c + NSTAGE - 1);
        load_a((s + NSTAGE - 1) % NSTAGE, c + NSTAGE - 1);
        compute(s, c & 1);
        store_x((s + 1) % NSTAGE, (c + 1) & 1);
        __syncthreads();
      }
    }
    // NSTAGE-1 .. 2*NSTAGE-2 chunks are left and c0 is a multiple of NSTAGE, so their register stages are static
    static_assert(NSTAGE == 2 || NSTAGE == 3, "one tail per remaining count");
    switch (nchunks - c0) {
      case 1: if (NSTAGE == 2) tail(std::integral_constant<int, 1>{}); break;
      case 2: tail(std::integral_constant<int, 2>{}); break;
      case 3: if (NSTAGE == 3) tail(std::integral_constant<int, 3>{}); break;
      case 4: if (NSTAGE == 3) tail(std::integral_constant<int, 4>{}); break;
      default: break;
    }
  } else if (nchunks > 0) {   // a K range shorter than the pipeline: guarded loads
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s)
      if (s < nchunks) { load_x(s, s); load_a(s, s); }
    store_x(0, 0);
    __syncthreads();
    for (int c0 = 0; c0 < nchunks; c0 += NSTAGE) {
#pragma unroll
      for (int s = 0; s < NSTAGE; ++s) {
        const int c = c0 + s;
        if (c < nchunks) {
          if (c + NSTAGE - 1 < nchunks) { load_x((s + NSTAGE - 1) % NSTAGE, c + NSTAGE - 1); load_a((s + NSTAGE - 1) % NSTAGE, c + NSTAGE - 1); }
          compute(s, c & 1);
          if (c + 1 < nchunks) store_x((s + 1) % NSTAGE, (c + 1) & 1);
          __syncthreads();
        }
      }
    }
  }
  const int half = lane >> 5, col = lane & 31;
  if (EPI == EPI_PARTIAL) {
    // transpose the wavefront's tile through LDS, 32 batch rows at a time, so that every store is a whole 128-byte
    // row segment (the LDS tile is private to the wavefront: only its own LDS traffic has to be waited for)
    float *tile = (float *)lds_raw + (size_t)w * 32 * L::TILE_STRIDE;
    float *P = (float *)out + (int64_t)blockIdx.y * Mp * Np + nb * 32;
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      transpose_in<L::TILE_STRIDE>(tile, acc[j], half, col);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (nb_own < nblocks) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          int r = q * 8 + (lane >> 3), n4 = (lane & 7) * 4;
          *(f32x4 *)(P + (int64_t)(j * 32 + r) * Np + n4) = *(const f32x4 *)(tile + r * L::TILE_STRIDE + n4);
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the reads are done before the next pass overwrites the tile
    }
  } else {  // EPI_SWIGLU: weight rows alternate gate_f, up_f; a block of 32 rows yields 16 features = two K8 groups
    if (nb_own >= nblocks) return;
#pragma unroll
    for (int j = 0; j < MB; ++j) *((u32x4v *)out + (int64_t)(nb * 2 + half) * Mp + j * 32 + col) = swiglu_unit(acc[j]);
  }
}

// ---- tiles with both operands in an LDS ring: batches of 256 rows and more ------------------------------
// What caps a large-tile GEMM here is what a compute unit can take in per cycle through its vector memory path, so a
// workgroup must fetch every operand byte once: 256 weight columns and 256 batch rows per k-step are 16 KB for 2 MFLOP.
// (A register-streaming form with two row halves fetched every weight block once per row half, 24 KB per k-step, and
// measured 12 - 25 % slower at 4096 rows.)  WR x WC wavefronts, each NBW weight blocks (32 NBW columns) x 32 MB rows.
// The weight blocks and the activation chunk of a k-step are fetched as 1 KB loads that land in LDS without passing
// through registers (buffer_load ... lds, the data of lane l at 16 l), shared out over the wavefronts; a stage of the ring is one
// k-step: [NB blocks x 64 units of A operands][2 k8 groups x ROWS rows of B operands], eight stages.
//
// Step c of the plain loop issues the loads of k-step c + LA, reads the operands of k-step c + 1 from the ring into the registers that k-step
// c - 1 has left, and runs the MFMAs of k-step c on the registers that the step before filled.  The scheduling barriers
// lay the operand reads behind the first MFMAs and the ring's loads behind the next: without them the compiler reads all operands and
// waits, and reads later in the step come too late for the next one.
// Every second step ends with a barrier, before which a wavefront waits until its own loads of the next three k-steps
// have landed (loads retire in order: all but the youngest LA - 3 k-steps' worth), so after the barrier of step c (odd) the
// stages c + 1 .. c + 3 are there, which are what steps c + 1 and c + 2 read ahead.  The stage that step c's loads overwrite
// held k-step c + LA - 8 <= c - 2, read in step c + LA - 9 <= c - 3 and used by the MFMAs of the step after that, and a barrier lies
// between any two steps that far apart.
// The wait is written by hand, together with the barrier: the compiler's own barrier sequence would wait for every
// outstanding load and empty the ring, and for the operand reads, which may stay in flight over the barrier.
//
// The loop by pairs of k-steps (PAIRS) has 16 x 16 x 32 MFMAs: half of the accumulator traffic per product for twice the operand reads
// from the register file (256 accumulators and 1024 operand halves for 8192 products, 1024 and 1024 for 16384 with 32 x 32 x 16 ones), and a
// 256 x 256 tile runs at the chip's power limit (1.5 GHz, the matrix cores busy 80 % of the cycles, with 32 x 32 x 16
// ones), so what a product costs in energy is what it costs in time.  A pair p issues the loads of pair p + 3, reads the operands of pair p + 1, runs
// its MFMAs and ends with the barrier, by which its wavefront's loads of the next four k-steps have landed; its loads overwrite pair p - 1's
// stages, whose reads the MFMAs of pair p - 1 have waited for.  Lane l supplies row l % 16 and k 8 (l / 16) .. + 8 of an operand and receives rows
// 4 (l / 16) + i of its column.  The weight rows of a tile are dealt to the A operand so that one lane swap per two registers turns two tiles into
// the halves of a 32 x 32 tile as the epilogues know it.  That one MFMA over 32 k sums in the bits of two over 16 is what the chip was seen to do, not
// something that its documents promise: tests/test_gpu_ring_forms.py holds the two loops against each other.
// 4096 rows, gate/up of the 4B / 8B / 32B shapes, launches back to back: 347 / 669 / 1736 us with global loads to LDS (a vector addition each, and the
// compiler waits for all operand reads at once behind them), 336 / 646 / 1675 with buffer loads and the reads behind the first MFMAs; on another card
// 344 / 654 / 1691 so, 329 / 605 / 1575 by pairs (1.24 / 1.36 / 1.36 PFLOP/s; inside scoring and prompt passes 320 - 327 / 596 - 633 / 1529 - 1570).
// Tiles of four wavefronts, bound by their loads, are 5 to 10 % slower by pairs and keep the plain loop; a 256 x 256 tile on four wavefronts is level in
// the plain loop and slower by pairs.
// Forms: 256 x 256 on eight wavefronts from 128 tiles on; 256 x 128 on four (12 KB per k-step) for batches of a few hundred rows (see fast_gemm_pick).
template <int WRv, int WCv, int MBv, int NBWv> struct GemmRingT {
  static constexpr int WR = WRv, WC = WCv, WN = WR * WC, MB = MBv, NBW = NBWv, NB = WC * NBW, ROWS = 32 * WR * MB, T = WN * 64;
  static constexpr int AU = NB * 64, XU = 2 * ROWS, SU = AU + XU;         // 16-byte units of a stage: A operands, B operands
  static constexpr int ALW = NB / WN, XLW = XU / T, LPS = ALW + XLW;      // weight, activation, all loads per wavefront and k-step
  static constexpr int NS = 8, LA = 6;                                    // stages, k-steps ahead
  static constexpr bool PAIRS = WN == 8;                                  // the loop by pairs of k-steps
  static constexpr int TILE_STRIDE = 36, BYTES = NS * SU * 16;            // 128 / 96 / 64 KB; the epilogue's WN x 32 x 36 floats reuse it
  static_assert(NB % WN == 0 && XU % T == 0 && WN * 32 * TILE_STRIDE * 4 <= BYTES, "whole loads per wavefront, room for the epilogue");
};
using Ring256x256 = GemmRingT<2, 4, 4, 2>;
using Ring256x128 = GemmRingT<2, 2, 4, 2>;   // 256 rows, 128 columns
using Ring128x128 = GemmRingT<2, 2, 2, 2>;   // two workgroups fit a compute unit; the lm_head only

// 16 bytes per lane from byte lane_off + off behind the buffer's base; l is the wavefront's base in LDS, lane l lands at l + 16 l.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t ring_buffer(const void *base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, -1, 0x00020000);
}
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t buf, int lane_off, int off, void *l) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (__attribute__((address_space(3))) void *)l, 16, lane_off, off, 0, 0);
}

// Which tile a workgroup takes: column strip bx, row block bz, run of k-steps by.  Workgroup i starts on XCD i % 8, so the
// tiles, numbered by runs of k-steps, then bands of four row blocks, then strips, are dealt to the XCDs in contiguous eighths: the 32
// tiles that are resident behind one L2 are four row blocks x eight strips, twelve operand blocks instead of up to 40.
constexpr int RING_BAND = 4;
__device__ __forceinline__ void ring_tile(int strips, int nz, int *bx, int *by, int *bz) {
  const int n = gridDim.x, id = blockIdx.x, x = id & 7;
  const int l = x * (n >> 3) + min(x, n & 7) + (id >> 3), per = strips * nz;
  *by = l / per;
  const int rem = l - *by * per, band = rem / (RING_BAND * strips), z0 = band * RING_BAND, in = rem - z0 * strips, nb = min(RING_BAND, nz - z0);
  *bx = in / nb;
  *bz = z0 + in % nb;
}

// Accumulates k-steps c_lo .. c_hi - 1 (a whole number of trips round the ring) of the tile whose first weight block is nbw
// and whose first row is mrow0.  Wavefront column wc holds the weight blocks ring_block<L, APART>(wc, 0 .. NBW - 1) of the
// tile.  Ends with a workgroup barrier, after which the ring is free for the epilogue.
template <class L, int APART = 1> __device__ __forceinline__ int ring_block(int wc, int n) {
  return wc / APART * APART * L::NBW + wc % APART + n * APART;
}

template <class L, int APART = 1>
__device__ __forceinline__ void ring_mainloop(f32x16 (&acc)[L::NBW][L::MB], u32x4v *ring, const u32x4v *__restrict__ Xp, const h16x8 *__restrict__ Wp,
                                              int Mp, int Kp, int nblocks, int nbw, int mrow0, int c_lo, int c_hi) {
  constexpr int MB = L::MB, NBW = L::NBW, ROWS = L::ROWS, NS = L::NS, LA = L::LA, SU = L::SU, AU = L::AU, WN = L::WN, WC = L::WC, LPS = L::LPS;
  static_assert((GEMM_K_PAD / 16) % NS == 0, "a run of k-steps is a whole number of trips round the ring");
  static_assert(NS == 8 && LA == 6, "the waits and the reuse of a stage are worked out above for these");
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, last = c_hi - 1;
  const int wrow = (w / WC) * 32 * MB;
  // what this wavefront fetches: weight blocks nbw + w, + WN .. (past the end: the last one again, never stored) and the
  // runs of 64 units i WN + w of the activation chunk (unit u: k8 group u / ROWS of the k-step, batch row u % ROWS)
  __amdgpu_buffer_rsrc_t a_src[L::ALW];
#pragma unroll
  for (int i = 0; i < L::ALW; ++i) a_src[i] = ring_buffer(Wp + w_block_base(min(nbw + i * WN + w, nblocks - 1), Kp));
  int x_off[L::XLW];
#pragma unroll
  for (int i = 0; i < L::XLW; ++i) {
    const int xi = (i * WN + w) * 64 + lane;
    x_off[i] = ((xi / ROWS) * Mp + xi % ROWS) * 16;
  }
  const int x_step = 2 * Mp * 16;
  // k-step c0 + i, or the last one (past the end: never used); the activations' offsets are from the trip's first k-step, a whole operand may pass 4 GB
  auto fetch = [&](int st, int c0, int i) {
    const __amdgpu_buffer_rsrc_t x_src = ring_buffer(Xp + mrow0 + (int64_t)(c0 * 2) * Mp);
    const int at = min(i, last - c0);
#pragma unroll
    for (int i = 0; i < L::XLW; ++i) load_to_lds(x_src, x_off[i], at * x_step, ring + st * SU + AU + (i * WN + w) * 64);
#pragma unroll
    for (int i = 0; i < L::ALW; ++i) load_to_lds(a_src[i], lane * 16, (c0 + at) * (int)(W_KSTEP * 16), ring + st * SU + (i * WN + w) * 64);
  };
#pragma unroll
  for (int j = 0; j < LA; ++j) fetch(j, c_lo, j);   // a run has at least NS k-steps
  if constexpr (L::PAIRS) {
    // what it reads: 16 rows of its weight blocks, and of its batch rows; k8 group lane / 16 of the pair
    const int s16 = lane & 15, k8 = lane >> 4, pair_at = (k8 >> 1) * SU;
    // (an LDS read reaches 64 KB from its base: one for either half of the ring, opaque, or the compiler keeps a register for every far address)
    int a_at[2], b_at[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      a_at[h] = h * (NS / 2) * SU + ring_block<L, APART>(w % WC, 0) * 64 + pair_at + (k8 & 1) * 32 + (s16 & 3) + 4 * (s16 >> 3) + 8 * (s16 >> 2 & 1);
      b_at[h] = h * (NS / 2) * SU + AU + pair_at + (k8 & 1) * ROWS + wrow + s16;
      asm("" : "+v"(a_at[h]), "+v"(b_at[h]));
    }
    u32x4v a[2][2 * NBW], b[2][2 * MB];
    auto read = [&](int set, int st) {
#pragma unroll
      for (int n = 0; n < 2 * NBW; ++n) a[set][n] = ring[a_at[st / (NS / 2)] + st % (NS / 2) * SU + (n >> 1) * APART * 64 + (n & 1) * 16];
#pragma unroll
      for (int j = 0; j < 2 * MB; ++j) b[set][j] = ring[b_at[st / (NS / 2)] + st % (NS / 2) * SU + j * 16];
    };
    f32x4 q[2 * NBW][2 * MB];
#pragma unroll
    for (int n = 0; n < 2 * NBW; ++n)
#pragma unroll
      for (int j = 0; j < 2 * MB; ++j) q[n][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LPS * (LA - 4)) : "memory");
    read(0, 0);
    for (int c0 = c_lo; c0 < c_hi; c0 += NS) {
#pragma unroll
      for (int s = 0; s < NS; s += 2) {
        read((s / 2 + 1) & 1, (s + 2) % NS);
        fetch((s + LA) % NS, c0, s + LA);
        fetch((s + 1 + LA) % NS, c0, s + 1 + LA);
#pragma unroll
        for (int j = 0; j < 2 * MB; ++j)
#pragma unroll
          for (int n = 0; n < 2 * NBW; ++n)
            q[n][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h16x8, a[s / 2 & 1][n]), __builtin_bit_cast(h16x8, b[s / 2 & 1][j]), q[n][j], 0, 0, 0);
        // MFMA, LDS read, four times; two MFMAs and a read (more reads at once and the registers of both pairs do not fit); two MFMAs and a load
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
#pragma unroll
        for (int i = 0; i < 2 * (NBW + MB) - 4; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
#pragma unroll
        for (int i = 0; i < 2 * LPS; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * NBW * MB, 0);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LPS * (LA - 4)) : "memory");
      }
    }
    // tiles 2j and 2j + 1 of a row hold columns 16 apart: exchanging the odd rows of 16 lanes of the first with the even ones of the second gives
    // every lane eight rows of the 16 for one of the 32 columns, the two results the rows 4 (l / 32) + i and 8 + 4 (l / 32) + i of the tile's half
#pragma unroll
    for (int n = 0; n < NBW; ++n)
#pragma unroll
      for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float u = q[2 * n + t][2 * j][i], v = q[2 * n + t][2 * j + 1][i];
            const auto x = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, u), __builtin_bit_cast(uint32_t, v), false, false);
            acc[n][j][8 * t + i] = __builtin_bit_cast(float, (uint32_t)x[0]);
            acc[n][j][8 * t + 4 + i] = __builtin_bit_cast(float, (uint32_t)x[1]);
          }
  } else {
    // what it reads: its NBW weight blocks, and its rows
    const u32x4v *a_lds = ring + ring_block<L, APART>(w % WC, 0) * 64 + lane;
    const u32x4v *b_lds = ring + AU + (lane >> 5) * ROWS + wrow + (lane & 31);
    u32x4v a[2][NBW], b[2][MB];
    auto read = [&](int set, int st) {
#pragma unroll
      for (int n = 0; n < NBW; ++n) a[set][n] = a_lds[st * SU + n * APART * 64];
#pragma unroll
      for (int j = 0; j < MB; ++j) b[set][j] = b_lds[st * SU + j * 32];
    };
#pragma unroll
    for (int n = 0; n < NBW; ++n)
#pragma unroll
      for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[n][j][r] = 0.f;
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LPS * (LA - 3)) : "memory");
    read(0, 0);
    for (int c0 = c_lo; c0 < c_hi; c0 += NS) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        read((s + 1) & 1, (s + 1) % NS);
        fetch((s + LA) % NS, c0, s + LA);
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
          for (int n = 0; n < NBW; ++n)
            acc[n][j] = mfma_h16(__builtin_bit_cast(h16x8, a[s & 1][n]), __builtin_bit_cast(h16x8, b[s & 1][j]), acc[n][j]);
#pragma unroll
        for (int i = 0; i < (NBW + MB) / 2; ++i) {   // MFMA, two LDS reads, ...
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
#pragma unroll
        for (int i = 0; i < LPS; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NBW * MB, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (s & 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LPS * (LA - 3)) : "memory");
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the loads past the end have landed before the ring is reused
  __syncthreads();
}

// grid strips * (Mp / ROWS) * runs of k-steps, see ring_tile; groups_per_split groups of eight k-steps per run.
template <class L, int EPI>
__global__ __launch_bounds__(L::T) void gemm_ring_kernel(void *out, const u32x4v *__restrict__ Xp, const h16x8 *__restrict__ Wp, int Mp, int Np, int Kp,
                                                         int groups_per_split, int strips) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  constexpr int MB = L::MB, NBW = L::NBW;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, nblocks = Np >> 5;
  int bx, by, bz;
  ring_tile(strips, Mp / L::ROWS, &bx, &by, &bz);
  const int c_lo = by * groups_per_split * L::NS, c_hi = min(Kp >> 4, c_lo + groups_per_split * L::NS);
  const int nbw = bx * L::NB, nb0 = nbw + (w % L::WC) * NBW, mrow0 = bz * L::ROWS, wrow = (w / L::WC) * 32 * MB;
  f32x16 acc[NBW][MB];
  ring_mainloop<L>(acc, (u32x4v *)lds_raw, Xp, Wp, Mp, Kp, nblocks, nbw, mrow0, c_lo, c_hi);
  const int half = lane >> 5, col = lane & 31;
  if (EPI == EPI_PARTIAL) {   // 32 x 32 tiles transposed through LDS so that every store is a whole 128-byte row segment
    float *tile = (float *)lds_raw + (size_t)w * 32 * L::TILE_STRIDE;
#pragma unroll
    for (int n = 0; n < NBW; ++n) {
      float *P = (float *)out + ((int64_t)by * Mp + mrow0 + wrow) * Np + (nb0 + n) * 32;
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        transpose_in<L::TILE_STRIDE>(tile, acc[n][j], half, col);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (nb0 + n < nblocks) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            int r = q * 8 + (lane >> 3), n4 = (lane & 7) * 4;
            *(f32x4 *)(P + (int64_t)(j * 32 + r) * Np + n4) = *(const f32x4 *)(tile + r * L::TILE_STRIDE + n4);
          }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
    }
  } else {  // EPI_SWIGLU
#pragma unroll
    for (int n = 0; n < NBW; ++n) {
      if (nb0 + n >= nblocks) break;
#pragma unroll
      for (int j = 0; j < MB; ++j) *((u32x4v *)out + (int64_t)((nb0 + n) * 2 + half) * Mp + mrow0 + wrow + j * 32 + col) = swiglu_unit(acc[n][j]);
    }
  }
}

template <class L, int EPI>
static void gemm_ring_launch(void *out, const void *Xp, const void *Wp, int Mp, int Np, int Kp, int nsplit, hipStream_t st) {
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void *)gemm_ring_kernel<L, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, L::BYTES);
    attr_set = true;
  }
  int strips = (Np / 32 + L::NB - 1) / L::NB, groups = (Kp / 16) / L::NS, gps = (groups + nsplit - 1) / nsplit, ny = (groups + gps - 1) / gps;
  hipLaunchKernelGGL((gemm_ring_kernel<L, EPI>), dim3(strips * (Mp / L::ROWS) * ny), dim3(L::T), L::BYTES, st, out, (const u32x4v *)Xp,
                     (const h16x8 *)Wp, Mp, Np, Kp, gps, strips);
}

// ---- QKV projection of large passes: per-head norm, rotary embedding and KV append in the epilogue --------------------------------
// The ring tile for a projection that is not split over K and has tiles enough (fast_gemm_qkv_fits).  A wavefront holds the two
// weight blocks whose dims are each other's rotation partners -- of a head of 128 blocks 0 and 2 or 1 and 3 (APART = 2), of a head of
// 64 both.  32 rows at a time it transposes its two 32 x 32 tiles through LDS, rotates four neighbouring dims and their partners per
// lane and stores q or the key tile; the per-head norm of a head of 128 adds the neighbouring wavefront's squares from its tiles.  A
// value unit holds eight keys of one dim, so there a lane takes a dim and gathers the eight rows of a unit (rows of a pass are runs of
// consecutive positions; the ends of a run, and rows in any other order -- a decode step's, each of another sequence -- are stored one by one).
// What it saves is the fp32 plane of the projection, written and read once: same products, same order, so q and the cache are
// bit-identical to qkv_post_wide_kernel's.  4096 rows, both kernels before against this one: 4B width 132 + 43 -> 138 us, 8B 208 + 46 ->
// 215, 32B 383 + 64 -> 404 (126 - 131 / 189 - 199 / 353 - 358 with the loop by pairs); whole scoring passes of 900 to 4096 rows 1 to 5 % faster at the three widths, none slower.
// Rollouts of 1000 rows, two layers, 31 steps: 4B width 27.7 -> 27.3 ms, 8B 39.4 -> 38.9.
struct QkvOut {
  uint16_t *q;              // half [M][Hq][hd]
  const float2 *rope;       // [M][hd / 2] (cos, sin)
  RowState rows;
  KvGeom kv;
  int layer, Hq, Hkv, M;
  const uint16_t *q_gain, *k_gain;   // bf16 [hd], with a per-head norm
  float eps;
};

template <class L, int HD, bool NORM>
__global__ __launch_bounds__(L::T) void gemm_ring_qkv_kernel(QkvOut out, const u32x4v *__restrict__ Xp, const h16x8 *__restrict__ Wp, int Mp, int Np, int Kp,
                                                             int strips) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  constexpr int MB = L::MB, NBW = L::NBW, APART = HD / 64, HALF = HD / 2, TS = L::TILE_STRIDE;
  static_assert(NBW == 2 && L::WC % APART == 0 && L::WN * 2 * 32 * TS * 4 <= L::BYTES, "whole heads per tile, room for the transposed tiles");
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31, nblocks = Np >> 5;
  int bx, by, bz;
  ring_tile(strips, Mp / L::ROWS, &bx, &by, &bz);
  const int nb0 = bx * L::NB + ring_block<L, APART>(w % L::WC, 0), mrow0 = bz * L::ROWS + (w / L::WC) * 32 * MB;
  f32x16 acc[NBW][MB];
  ring_mainloop<L, APART>(acc, (u32x4v *)lds_raw, Xp, Wp, Mp, Kp, nblocks, bx * L::NB, bz * L::ROWS, 0, Kp >> 4);
  // of batch row mrow0 + 32 j + col; requested here: held through the loop by pairs they spill 8 to 12 registers (4096 rows of the 4B / 8B / 32B shapes, kernel
  // medians 134 / 200 / 362 us, 131 / 199 / 358 so)
  int act[MB], pos[MB], slot[MB];
#pragma unroll
  for (int j = 0; j < MB; ++j) {
    const int m = min(mrow0 + j * 32 + col, out.M - 1);
    act[j] = out.rows.active[m]; pos[j] = out.rows.pos[m]; slot[j] = out.rows.slot[m];
  }
  const bool own = nb0 < nblocks;   // (heads are whole: both blocks lie past the end, or neither)
  if (!NORM && !own) return;
  const int head = nb0 / (HD / 32), d0 = (nb0 % (HD / 32)) * 32;   // dims d0 .. d0 + 31 and their partners HALF further
  const bool is_q = head < out.Hq, is_k = !is_q && head < out.Hq + out.Hkv, rotate = own && (is_q || is_k);
  const int kvh = is_q ? 0 : is_k ? head - out.Hq : head - out.Hq - out.Hkv;
  float *tile = (float *)lds_raw + (size_t)w * 2 * 32 * TS;   // [block][row][dim]
  // the rotation of rows 8 s + lane / 8 of 32, dims (lane % 8) * 4 .. + 3; requested 32 rows ahead of its use
  f32x4 cs[2][4][2];
  auto load_cs = [&](int j) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const f32x4 *p = (const f32x4 *)(out.rope + (int64_t)min(mrow0 + j * 32 + s * 8 + (lane >> 3), out.M - 1) * HALF + d0 + (lane & 7) * 4);
      cs[j & 1][s][0] = p[0]; cs[j & 1][s][1] = p[1];
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  float gain[2][4];   // of the lane's dims
  if (NORM && rotate) {
    const uint16_t *g = (is_q ? out.q_gain : out.k_gain) + d0 + (lane & 7) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) { gain[0][e] = bf16_bits_to_f32(g[e]); gain[1][e] = bf16_bits_to_f32(g[e + HALF]); }
  }
  const float *beside = tile + ((w % L::WC) % APART == 0 ? 1 : -1) * (APART - 1) * 2 * 32 * TS;   // the head's other wavefront's tiles, if it has one
  if (rotate) load_cs(0);
#pragma unroll
  for (int j = 0; j < MB; ++j) {
    const int m0 = mrow0 + j * 32;
    if (!NORM && m0 >= out.M) break;
    if (rotate && j + 1 < MB) load_cs(j + 1);
#pragma unroll
    for (int n = 0; n < 2; ++n) transpose_in<TS>(tile + n * 32 * TS, acc[n][j], half, col);
    const int on = m0 + col < out.M && act[j];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (NORM) __syncthreads();
    if (rotate) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = s * 8 + (lane >> 3), i = (lane & 7) * 4, m = m0 + r;
        const int r_act = __shfl(on, r, 64), r_pos = __shfl(pos[j], r, 64), r_slot = __shfl(slot[j], r, 64);
        f32x4 a = *(const f32x4 *)(tile + r * TS + i), b = *(const f32x4 *)(tile + (32 + r) * TS + i);
        if (NORM) {   // summed in the order of qkv_post_wide_kernel: dims 32 apart (a head of 128), then 16, 8, 4, 2 and 1
          float t[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) t[e] = fmaf(a[e], a[e], b[e] * b[e]);
          if (APART == 2) {
            const f32x4 oa = *(const f32x4 *)(beside + r * TS + i), ob = *(const f32x4 *)(beside + (32 + r) * TS + i);
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] += fmaf(oa[e], oa[e], ob[e] * ob[e]);
          }
#pragma unroll
          for (int off = 4; off > 0; off >>= 1)
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] += __shfl_xor(t[e], off);
          const float ss = (t[0] + t[2]) + (t[1] + t[3]), inv = 1.0f / sqrtf(ss / (float)HD + out.eps);
#pragma unroll
          for (int e = 0; e < 4; ++e) { a[e] = a[e] * inv * gain[0][e]; b[e] = b[e] * inv * gain[1][e]; }
        }
        if (m >= out.M) continue;
        const f32x4 c01 = cs[j & 1][s][0], c23 = cs[j & 1][s][1];
        const float cx[4] = {c01[0], c01[2], c23[0], c23[2]}, sy[4] = {c01[1], c01[3], c23[1], c23[3]};
        uint16_t ha[4], hb[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ha[e] = f32_to_h16_bits(fmaf(a[e], cx[e], -(b[e] * sy[e])));
          hb[e] = f32_to_h16_bits(fmaf(b[e], cx[e], a[e] * sy[e]));
        }
        const uint2 pa = {(uint32_t)ha[0] | (uint32_t)ha[1] << 16, (uint32_t)ha[2] | (uint32_t)ha[3] << 16};
        const uint2 pb = {(uint32_t)hb[0] | (uint32_t)hb[1] << 16, (uint32_t)hb[2] | (uint32_t)hb[3] << 16};
        if (is_q) {
          uint16_t *dst = out.q + ((int64_t)m * out.Hq + head) * HD + d0 + i;
          *(uint2 *)dst = pa;
          *(uint2 *)(dst + HALF) = pb;
        } else if (r_act) {
          uint16_t *dst = (uint16_t *)out.kv.base + out.kv.tiled_head_off(r_slot, out.layer, kvh);
          *(uint2 *)(dst + out.kv.tiled_k_off(r_pos, d0 + i)) = pa;
          *(uint2 *)(dst + out.kv.tiled_k_off(r_pos, d0 + HALF + i)) = pb;
        }
      }
    } else if (own) {
      const int pos0 = __builtin_amdgcn_readfirstlane(pos[j]), slot0 = __builtin_amdgcn_readfirstlane(slot[j]);
      uint16_t *cache = (uint16_t *)out.kv.base;
      const int dim = d0 + half * HALF + col;   // the lower half of the wavefront takes the first block's dims, the upper half their partners
      const float *t = tile + half * 32 * TS + col;
      if (__all(on && slot[j] == slot0 && pos[j] == pos0 + col)) {   // 32 consecutive keys
        uint16_t *dst = cache + out.kv.tiled_head_off(slot0, out.layer, kvh);
        for (int r = -(pos0 & 7); r < 32; r += 8) {
          uint16_t *unit = dst + out.kv.tiled_v_off(pos0 + r, dim);
          if (r >= 0 && r + 8 <= 32) {
            uint32_t p[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = (uint32_t)f32_to_h16_bits(t[(r + 2 * e) * TS]) | (uint32_t)f32_to_h16_bits(t[(r + 2 * e + 1) * TS]) << 16;
            *(uint4 *)unit = make_uint4(p[0], p[1], p[2], p[3]);
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (r + e >= 0 && r + e < 32) unit[e] = f32_to_h16_bits(t[(r + e) * TS]);
          }
        }
      } else {
        const int64_t mine = out.kv.tiled_head_off(slot[j], out.layer, kvh) + out.kv.tiled_v_off(pos[j], 0);   // where the row's dim 0 lies
        const int lo = (int)mine, hi = (int)(mine >> 32), of_dim = (int)out.kv.tiled_v_off(0, dim) - (int)out.kv.tiled_v_off(0, 0);
        for (int r = 0; r < 32; ++r) {
          if (!__builtin_amdgcn_readlane(on, r)) continue;
          const int64_t at = (int64_t)__builtin_amdgcn_readlane(hi, r) << 32 | (uint32_t)__builtin_amdgcn_readlane(lo, r);
          cache[at + of_dim] = f32_to_h16_bits(t[r * TS]);
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the reads are done before the next rows overwrite the tiles
    if (NORM) __syncthreads();
  }
}

template <class L, int HD, bool NORM>
static void gemm_ring_qkv_launch(const QkvOut &out, const void *Xp, const void *Wp, int Mp, int Np, int Kp, hipStream_t st) {
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void *)gemm_ring_qkv_kernel<L, HD, NORM>, hipFuncAttributeMaxDynamicSharedMemorySize, L::BYTES);
    attr_set = true;
  }
  const int strips = (Np / 32 + L::NB - 1) / L::NB;
  hipLaunchKernelGGL((gemm_ring_qkv_kernel<L, HD, NORM>), dim3(strips * (Mp / L::ROWS)), dim3(L::T), L::BYTES, st, out, (const u32x4v *)Xp, (const h16x8 *)Wp, Mp, Np,
                     Kp, strips);
}

// A tile's epilogue is as long as its 256 rows, however few tiles there are, where the kernel of its own deals the rows to the whole
// chip: below 48 tiles (narrow models, whose K is too short to be split) that one is the better.  This epilogue against it: rollouts of 48 steps,
// 10 tiles (200 rows, hidden 896) 33.7 / 31.2 ms, 24 tiles (256 rows, hidden 512) 15.8 / 15.0, 32 tiles (130 rows, hidden 1008) 33.2 / 33.1, 48
// tiles (512 rows, hidden 512) 18.7 / 18.7, 96 tiles (1000 rows) 24.0 / 24.8; scoring passes, 10 tiles 781 / 766 us, 24 tiles 660 / 656, 48 tiles
// 744 / 756, 96 tiles 783 / 826.
bool fast_gemm_qkv_fits(GemmShape g, int Mp, int Np) {
  if (g.form == GEMM_STREAM || g.nsplit != 1) return false;
  return g.form == GEMM_RING_256X256 || (Np / 32 + 3) / 4 * (Mp / 256) >= 48;   // (256 x 256 tiles: 128 or more, see fast_gemm_pick)
}

void fast_gemm_qkv(void *q_h16, const void *Xp, const void *Wp, int Mp, int Np, int Kp, GemmShape g, const void *q_gain, const void *k_gain, int qk_norm,
                   float eps, const float *rope_cs, RowState rows, KvGeom kv, int layer, int M, int Hq, int Hkv, hipStream_t st) {
  const QkvOut out{(uint16_t *)q_h16, (const float2 *)rope_cs, rows, kv, layer, Hq, Hkv, M, (const uint16_t *)q_gain, (const uint16_t *)k_gain, eps};
  auto tile = [&](auto l) {
    using L = decltype(l);
    if (kv.head_dim == 128) {
      if (qk_norm) gemm_ring_qkv_launch<L, 128, true>(out, Xp, Wp, Mp, Np, Kp, st); else gemm_ring_qkv_launch<L, 128, false>(out, Xp, Wp, Mp, Np, Kp, st);
    } else {
      if (qk_norm) gemm_ring_qkv_launch<L, 64, true>(out, Xp, Wp, Mp, Np, Kp, st); else gemm_ring_qkv_launch<L, 64, false>(out, Xp, Wp, Mp, Np, Kp, st);
    }
  };
  if (g.form == GEMM_RING_256X256) tile(Ring256x256{}); else tile(Ring256x128{});
}

// The largest split count <= nsplit that a ring kernel realises exactly: it cuts K into runs of ceil(groups / nsplit) groups of
// eight k-steps, which may come to fewer runs than asked for.
int fast_gemm_even_split(int Kp, int nsplit) {
  int groups = Kp / 16 / 8;
  for (;;) {
    int gps = (groups + nsplit - 1) / nsplit, ny = (groups + gps - 1) / gps;
    if (ny == nsplit) return nsplit;
    nsplit = ny;
  }
}

// Launch shape.  Up to 128 batch rows the LDS-staged kernel runs: three or four weight blocks per workgroup, and a
// grid split over K that brings the launch to about one workgroup per compute unit (partials cost HBM writes, so
// no more than that); a GEMM whose epilogue needs the whole K (SwiGLU) is not split and takes the workgroup width
// (three to eight blocks) that needs the fewest rounds of the chip.  Batches that are a multiple of 256 rows take the
// LDS-ring kernel (256 x 256 tiles from 128 of them on, 256 x 128 tiles with a split over K otherwise).  K is padded to
// GEMM_K_PAD and the rows to 32, 64, 128 or a multiple of 256, so there are no other shapes.
void fast_gemm_pick(int Np, int Kp, int Mp, int full_k, GemmShape *g) {
  const int nblocks = Np / 32, ksteps = Kp / 16;
  // 256 x 256 tiles against 256 x 128 at 512, 1024 and 4096 rows, no split, us: 112 tiles (224 of the smaller) 54 - 57 / 38 - 42 at K 2560, 80 - 89 / 57 - 63 at
  // K 4096, 183 - 196 / 128 - 136 at K 9728; 144 tiles (288: a second round) 57 - 60 / 64 - 79, 86 - 92 / 99 - 120, 188 - 197 / 240 - 252.  At 128 tiles exactly
  // the smaller ones are one round still and would be the better: 56 - 59 / 42 - 46, 83 - 92 / 63 - 70, 190 - 200 / 142 - 150.
  if (Mp % 256 == 0 && (nblocks + 7) / 8 * (Mp / 256) >= 128) {
    g->form = GEMM_RING_256X256; g->waves_n = 0; g->nsplit = 1;
    // One tile per compute unit at a time, so a tile count just above a multiple of 256 leaves most of the chip idle in
    // the last round (320 tiles take two rounds).  Splitting K in two runs makes the units of work half as long and the
    // rounds fill up (320 tiles: 1.5 rounds' worth), at the price of a second plane of fp32 partials written and read
    // again -- which pays once K is long.  4096 rows, the product with the norm that reads its planes, whole / in two runs, us: 320 tiles (N 5120) K 4096
    // 245 / 254, 5120 286 / 287, 6144 327 / 321, 8192 408 / 385 (344 / 297 the product alone), 25600 1100 / 950 (1036 / 875); 288 tiles K 4096 235 / 234,
    // 6144 317 / 303, 8192 397 / 367; 384 tiles K 4096 264 / 288, 6144 351 / 354, 8192 435 / 427.
    if (!full_k && Kp >= 6144) {
      const int tiles = (nblocks + 7) / 8 * (Mp / 256);
      if ((2 * tiles + 255) / 256 * 0.5 <= 0.8 * ((tiles + 255) / 256)) g->nsplit = 2;
    }
    return;
  }
  if (Mp % 256 == 0) {
    // 256 x 128 tiles (two row halves x two column pairs of wavefronts), K split until the launch has about one
    // workgroup per compute unit; a split keeps at least four groups of eight k-steps
    int strips = (nblocks + 3) / 4 * (Mp / 256), groups = ksteps / 8;
    int ns = full_k ? 1 : (240 + strips / 2) / strips;
    if (ns > groups / 4) ns = groups / 4;
    if (ns > 12) ns = 12;
    if (ns < 1) ns = 1;
    g->form = GEMM_RING_256X128; g->waves_n = 0; g->nsplit = fast_gemm_even_split(Kp, ns);
    return;
  }
  const int total_chunks = ksteps / GEMM_KC;
  g->form = GEMM_STREAM;
  if (full_k) {
    // No split over K (the SwiGLU epilogue needs whole sums), one workgroup per compute unit at a time: the launch takes
    // rounds x width, rounds = ceil(workgroups / 256).  The width with the smallest product wins, the wider one on a
    // tie (fewer rounds, fewer re-reads of the activations).  Measured at 64 rows: 608 blocks (4B) width 3, 203
    // workgroups, 21 us (width 4: 23); 768 blocks (8B) width 3, 256 workgroups, 34 us; 1600 blocks (32B) width 7,
    // 229 workgroups, 81 us -- width 3 (534 workgroups, three rounds) took 109 us there, width 4 (two rounds) 90.
    // At 128 rows the activations that every workgroup reads, as much as four blocks, are counted, and widths of five and six spill
    // registers (seven and eight do not, with half as many operands read ahead): 1600 blocks width 7, 92 us (width 4: 121); two layers of the 32B width
    // with 1100 blocks, 24 steps, width 7 14.1 ms (width 3: 15.7), 2040 blocks width 8 17.6 (width 4: 18.9); two layers of hidden 2560, 40 steps, 1030
    // to 1793 blocks 5 to 8 % faster than the best of widths three and four, up to 900 blocks the same form.
    int best = 3, best_cost = 1 << 30;
    for (int wn = 3; wn <= 8; ++wn) {
      if (Mp > 64 && (wn == 5 || wn == 6)) continue;
      int wgs = (nblocks + wn - 1) / wn, cost = (wgs + 255) / 256 * (Mp <= 64 ? wn : wn + 4);
      if (cost <= best_cost) { best = wn; best_cost = cost; }
    }
    g->waves_n = best; g->nsplit = 1;
    return;
  }
  // workgroups of a launch with wn weight blocks per workgroup once K is split to about one workgroup per compute unit
  auto split_for = [&](int wn, int *wgs) {
    int strips = (nblocks + wn - 1) / wn, ns = (240 + strips / 2) / strips;
    if (ns > total_chunks / 2) ns = total_chunks / 2;
    if (ns > 10) ns = 10;
    if (ns < 1) ns = 1;
    int cps = (total_chunks + ns - 1) / ns;
    ns = (total_chunks + cps - 1) / cps;
    *wgs = strips * ns;
    return ns;
  };
  g->waves_n = nblocks % 4 == 0 || nblocks > 96 ? 4 : 3;
  int wgs = 0;
  g->nsplit = split_for(g->waves_n, &wgs);
  // A narrow output with four blocks per workgroup can leave a third of the chip without a workgroup however K is split
  // (2560 columns: 20 strips x 8 runs = 160); three blocks give 27 strips and 216 workgroups (measured at 64 rows on the
  // 4B shape, output and down projection together: decode step 3.764 -> 3.741 ms; where the gain in workgroups is small --
  // 6144 columns, 240 -> 256 -- nothing moves).  Never past one workgroup per compute unit.
  if (Mp <= 64 && g->waves_n == 4) {
    int wgs3 = 0, ns3 = split_for(3, &wgs3);
    if (wgs3 <= 256 && wgs3 * 20 >= wgs * 23) { g->waves_n = 3; g->nsplit = ns3; }
  }
}

template <int MB, int WN, int NSTAGE, int EPI>
static void gemm_lds_launch(void *out, const void *Xp, const void *Wp, int Mp, int Np, int Kp, int nsplit, hipStream_t st) {
  using L = GemmLds<MB, WN>;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void *)gemm_lds_kernel<MB, WN, NSTAGE, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, L::BYTES);
    attr_set = true;
  }
  int nblocks = Np / 32, total_chunks = (Kp / 16) / L::KC, cps = (total_chunks + nsplit - 1) / nsplit;
  dim3 grid((nblocks + WN - 1) / WN, nsplit), block(64 * WN);
  hipLaunchKernelGGL((gemm_lds_kernel<MB, WN, NSTAGE, EPI>), grid, block, L::BYTES, st, out, (const u32x4v *)Xp, (const h16x8 *)Wp, Mp,
                     Np, Kp, cps);
}

// The instantiated forms: three blocks (the full-K projection at 32 and 128 rows with a three-chunk weight pipeline, all others with
// two chunks: deeper pipelines measured no faster for the split projections, and for 64 rows see gemm_lds_min_wgs), four blocks with two chunks, and for the full-K projection five to eight blocks with two chunks, at 128 rows seven or eight (see
// fast_gemm_pick).
template <int MB, int EPI>
static void gemm_lds_dispatch_rows(void *out, const void *Xp, const void *Wp, int Mp, int Np, int Kp, GemmShape g, hipStream_t st) {
  if constexpr (EPI == EPI_SWIGLU && MB != 2) {
    if (g.waves_n == 3) { gemm_lds_launch<MB, 3, 3, EPI>(out, Xp, Wp, Mp, Np, Kp, g.nsplit, st); return; }
  } else {
    if (g.waves_n == 3) { gemm_lds_launch<MB, 3, 2, EPI>(out, Xp, Wp, Mp, Np, Kp, g.nsplit, st); return; }
  }
  if constexpr (EPI == EPI_SWIGLU && MB <= 2) {
    if (g.waves_n == 5) { gemm_lds_launch<MB, 5, 2, EPI>(out, Xp, Wp, Mp, Np, Kp, g.nsplit, st); return; }
    if (g.waves_n == 6) { gemm_lds_launch<MB, 6, 2, EPI>(out, Xp, Wp, Mp, Np, Kp, g.nsplit, st); return; }
  }
  if constexpr (EPI == EPI_SWIGLU) {
    switch (g.waves_n) {
      case 7: gemm_lds_launch<MB, 7, 2, EPI>(out, Xp, Wp, Mp, Np, Kp, g.nsplit, st); return;
      case 8: gemm_lds_launch<MB, 8, 2, EPI>(out, Xp, Wp, Mp, Np, Kp, g.nsplit, st); return;
      default: break;
    }
  }
  gemm_lds_launch<MB, 4, 2, EPI>(out, Xp, Wp, Mp, Np, Kp, g.nsplit, st);
}

template <int EPI>
static void gemm_lds_dispatch(void *out, const void *Xp, const void *Wp, int Mp, int Np, int Kp, GemmShape g, hipStream_t st) {
  const int mb = Mp / 32;   // 1, 2 or 4
  if (mb == 1) gemm_lds_dispatch_rows<1, EPI>(out, Xp, Wp, Mp, Np, Kp, g, st);
  else if (mb == 2) gemm_lds_dispatch_rows<2, EPI>(out, Xp, Wp, Mp, Np, Kp, g, st);
  else gemm_lds_dispatch_rows<4, EPI>(out, Xp, Wp, Mp, Np, Kp, g, st);
}

template <int EPI>
static void gemm_dispatch(void *out, const void *Xp, const void *Wp, int Mp, int Np, int Kp, GemmShape g, hipStream_t st) {
  switch (g.form) {
    case GEMM_RING_256X256: gemm_ring_launch<Ring256x256, EPI>(out, Xp, Wp, Mp, Np, Kp, g.nsplit, st); return;
    case GEMM_RING_256X128: gemm_ring_launch<Ring256x128, EPI>(out, Xp, Wp, Mp, Np, Kp, g.nsplit, st); return;
    default: gemm_lds_dispatch<EPI>(out, Xp, Wp, Mp, Np, Kp, g, st);
  }
}

void fast_gemm(void *out, const void *Xp, const void *Wp, int Mp, int Np, int Kp, GemmShape g, GemmEpilogue epi,
               hipStream_t st) {
  if (epi == EPI_PARTIAL) gemm_dispatch<EPI_PARTIAL>(out, Xp, Wp, Mp, Np, Kp, g, st);
  else { g.nsplit = 1; gemm_dispatch<EPI_SWIGLU>(out, Xp, Wp, Mp, Np, Kp, g, st); }
}

// ---- lm_head ---------------------------------------------------------------------------------------------
// What a lane does with the logits it holds of one batch row: register 4g + i of accumulator x[n] is (times W_UNSCALE) the
// logit of vocabulary entry v0 + 32n + 8g + i, v0 = 32 * (first weight block) + 4 * (lane / 32).  Entries past V do not count.
constexpr float LOG2_E = 1.44269504088896341f;
template <int NBW>
__device__ __forceinline__ void mask_past_vocab(f32x16 (&x)[NBW], int v0, int V) {
  if (__any(v0 + 32 * NBW > V)) {
#pragma unroll
    for (int n = 0; n < NBW; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (v0 + 32 * n + 8 * (r >> 2) + (r & 3) >= V) x[n][r] = -INFINITY;
  }
}

// Sum of exp(z - max z) from the lane's largest accumulator value xm: the difference first, so that the sum is as exact at
// scores of thousands (low temperatures) as at small ones, then hardware exp2.
template <int NBW>
__device__ __forceinline__ float sum_exp_lane(const f32x16 (&x)[NBW], float c2, float xm) {
  float sum = 0.f;
  if (xm > -INFINITY) {
#pragma unroll
    for (int n = 0; n < NBW; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f((x[n][r] - xm) * c2);
  }
  return sum;
}

// Scoring: (max z, sum of exp(z - max z)); the target's z goes to *target_z if the lane holds it.
template <int NBW>
__device__ __forceinline__ SampleAcc score_lane(f32x16 (&x)[NBW], int v0, int V, float temperature, int target, float *target_z) {
  const float c2 = W_UNSCALE / temperature * LOG2_E;
  mask_past_vocab<NBW>(x, v0, V);
  if (__any(target >= v0 && target < v0 + 32 * NBW)) {
#pragma unroll
    for (int n = 0; n < NBW; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (target == v0 + 32 * n + 8 * (r >> 2) + (r & 3)) *target_z = x[n][r] * W_UNSCALE / temperature;
  }
  SampleAcc sa = sample_acc_init();
  float xm = -INFINITY;
#pragma unroll
  for (int n = 0; n < NBW; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) xm = fmaxf(xm, x[n][r]);
  sa.zsum = sum_exp_lane<NBW>(x, c2, xm);
  sa.zmax = xm * W_UNSCALE / temperature;
  return sa;
}

// Sampling: the same, and the best perturbed score z + g of the lane's entries (lowest index on exact ties).  The score that
// decides is the fp32 one (division by T, two logf), but it costs some sixty instructions per entry in a serial chain, more
// than the main loop at 256 rows.  So the entries are first compared by z/ln2 - log2(-log2 u), which orders them the same way up
// to the rounding of two hardware logarithms (relative 2^-22 each) and of z, and only the winner is evaluated in full.  The
// two orders can differ only where the lane's best two are closer than those errors: below 1e-5 plus 1e-6 of the score's
// magnitude together; within ten times that the lane's wavefront evaluates all entries in full, in index order (a percent of
// the wavefronts; through `dump`, 4 KB of LDS of its own, because a rolled loop cannot index registers).  So it does where a lane
// has entries but no score above -inf (logits of -inf): the lowest index among equals is an entry of the vocabulary there too.
template <int NBW>
__device__ __forceinline__ SampleAcc sample_lane(f32x16 (&x)[NBW], float *dump, int v0, int V, float temperature, uint64_t seed, uint32_t stream,
                                                 uint32_t step) {
  const float c2 = W_UNSCALE / temperature * LOG2_E;
  mask_past_vocab<NBW>(x, v0, V);
  SampleAcc sa = sample_acc_init();
  float xm = -INFINITY, best = -INFINITY, second = -INFINITY, xbest = 0.f;
  uint32_t wbest = 0;
  int kbest = -1;
#pragma unroll
  for (int n = 0; n < NBW; ++n)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const u32x4 d = draw4(seed, stream, step, (uint32_t)(v0 >> 2) + 8 * n + 2 * g);
      const uint32_t w[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float u = uniform_from_bits(w[i]);
        const float f = fmaf(x[n][4 * g + i], c2, -__builtin_amdgcn_logf(-__builtin_amdgcn_logf(u)));
        xm = fmaxf(xm, x[n][4 * g + i]);
        const bool better = f > best;
        second = __builtin_amdgcn_fmed3f(f, best, second);   // (the smaller of the two others where f is NaN)
        best = better ? f : best;
        xbest = better ? x[n][4 * g + i] : xbest;
        wbest = better ? w[i] : wbest;
        kbest = better ? 32 * n + 8 * g + i : kbest;
      }
    }
  sa.zsum = sum_exp_lane<NBW>(x, c2, xm);
  sa.zmax = xm * W_UNSCALE / temperature;
  if (__any(second > best - (1e-4f + 1e-5f * (fabsf(best) + 32.f)) || (kbest < 0 && v0 < V))) {
    float *mine = dump + (threadIdx.x & 63);
#pragma unroll
    for (int n = 0; n < NBW; ++n) {
#pragma unroll
      for (int r = 0; r < 16; ++r) mine[r * 64] = x[n][r];
#pragma unroll 1
      for (int g = 0; g < 4; ++g) {
        const u32x4 d = draw4(seed, stream, step, (uint32_t)(v0 >> 2) + 8 * n + 2 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int v = v0 + 32 * n + 8 * g + i;
          const float z = mine[(4 * g + i) * 64] * W_UNSCALE / temperature, score = z + gumbel_from_bits(i == 0 ? d.x : i == 1 ? d.y : i == 2 ? d.z : d.w);
          if (v < V && (score > sa.best || (score == sa.best && v < sa.idx))) { sa.best = score; sa.zbest = z; sa.idx = v; }
        }
      }
    }
  } else if (kbest >= 0) {
    sa.zbest = xbest * W_UNSCALE / temperature;
    sa.best = sa.zbest + gumbel_from_bits(wbest);
    sa.idx = v0 + kbest;
  }
  return sa;
}

// grid ceil(Np/32 / 4), block 256; 32*MB batch rows.  The GEMM main loop over the full K (four weight blocks per
// workgroup), then every lane's logits are folded into a running (max, sum-exp, best perturbed score, its index, its z) per
// batch row: per wavefront, then over the four wavefronts in wavefront order, one partial per workgroup.
constexpr int LM_WN = 4;
constexpr int LM_DUMP_FLOATS = 16 * 64;   // sample_lane's LDS, per wavefront

// The vocabulary takes several rounds of workgroups (1187 for 151936 rows on 256 compute units), and a workgroup's
// sampler epilogue moves no weights.  With two workgroups resident per compute unit one's epilogue and first loads run
// under the other's weight stream: 64 rows 199 -> 146 us, 32 rows 158 -> 133 us.  That needs the kernel inside 256 registers
// per lane, which a two-chunk weight pipeline allows (three chunks in flight fit only at 32 rows).  With only the winner
// of a lane's entries evaluated in full (sample_lane): 64 rows 137 -> 125 us, 32 rows 120.7 -> 117.5 us.  The logits form of 128
// rows has no long epilogue to hide and is alone on the unit.
template <int MB> constexpr int lm_wgs_per_cu() { return MB <= 2 ? 2 : 1; }

template <int MB, int NSTAGE, bool LOGITS, int WN = LM_WN>
__global__ __launch_bounds__(WN * 64, lm_wgs_per_cu<MB>()) void lmhead_kernel(const u32x4v *__restrict__ Xp, const h16x8 *__restrict__ Wp, int Mp,
                                                     int Np, int Kp, int V, float temperature, uint64_t seed,
                                                     DrawIds ids, const int32_t *target, float *target_z,
                                                     float *part, int n_wg, float *logits, int64_t ld) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  using L = GemmLds<MB, WN>;
  static_assert(LOGITS || WN == LM_WN, "the sampler's fold is over four wavefronts");
  int w = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int nblocks = Np >> 5;
  const int nb_own = blockIdx.x * WN + w, nb = min(nb_own, nblocks - 1);
  f32x16 acc[MB];
  gemm_lds_mainloop<MB, WN, NSTAGE>(acc, lds_raw, Xp, Wp, Mp, Np, Kp, nb, 0, (Kp >> 4) / L::KC);
  auto write_partial = [&](const SampleAcc &sa, int m) {
    int64_t o = (int64_t)blockIdx.x * Mp + m, plane = (int64_t)n_wg * Mp;
    if (target) score_part_store(part, o, sa);
    else sample_part_store(part, o, plane, sa);
  };
  if constexpr (LOGITS) {
    if (nb_own < nblocks) {
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        int m = j * 32 + col;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          int v0 = nb * 32 + 8 * g + 4 * half;
          f32x4 o = {acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]};
          if (v0 < V) *(f32x4 *)(logits + (int64_t)m * ld + v0) = o * W_UNSCALE;
        }
      }
    }
  } else {
    SampleAcc sa[MB];
    const int v0 = nb_own * 32 + 4 * half;
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      const int m = j * 32 + col;
      f32x16 x[1] = {acc[j]};
      if (target) sa[j] = score_lane<1>(x, v0, V, temperature, target[m], target_z + m);
      else sa[j] = sample_lane<1>(x, (float *)lds_raw + w * LM_DUMP_FLOATS, v0, V, temperature, seed, draw_stream(ids, m), draw_step(ids, m));
    }
    // lanes l and l^32 hold the same batch row; then fold the four wavefronts in wavefront order
    SampleAcc (*sh)[MB][32] = (SampleAcc (*)[MB][32])(lds_raw + LM_WN * LM_DUMP_FLOATS * 4);   // [3][MB][32]; the main loop's buffers are free by now
#pragma unroll
    for (int j = 0; j < MB; ++j) { SampleAcc b = sample_acc_shfl_xor(sa[j], 32); sample_acc_merge(sa[j], b); }
    if (w > 0 && half == 0)
#pragma unroll
      for (int j = 0; j < MB; ++j) sh[w - 1][j][col] = sa[j];
    __syncthreads();
    if (w == 0 && half == 0) {
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        for (int ww = 0; ww < 3; ++ww) sample_acc_merge(sa[j], sh[ww][j][col]);
        write_partial(sa[j], j * 32 + col);
      }
    }
  }
}

// ---- lm_head on the tiles of the LDS ring (128 rows and more) ----------------------------------------------------------------
// A wavefront holds 64 vocabulary entries of 32 MB batch rows; lanes l and l^32 hold the same rows.  One partial per (row, strip
// of 32 NB entries): max z, sum exp, best score, its z, its index (sample_part_store); scoring (SCORE) writes the first two and target_z.
// Scoring passes take 256 x 256 tiles, bound by the matrix cores: 4096 rows, vocabulary 151936: 2.32 - 2.47 ms at hidden 2560 (1.29 - 1.37
// PFLOP/s), 4.41 - 4.60 ms at 5120 (1.39 - 1.44; 2.63 and 5.10 before the loop by pairs), where the register-streaming tile it replaced (24 KB per k-step,
// accumulators parked in LDS for the epilogue) took 3.91 and 6.83.  Sampling takes 128 x 128 tiles: its epilogue keeps the vector unit busy for as long
// as the main loop keeps the loads and the matrix cores, and two workgroups per compute unit let one's epilogue run under the
// other's main loop: hidden 2560, 256 rows 267 us (256 x 256 tiles, one workgroup per unit: 298, 344 before the loop by pairs; 256 x 128: 338; the
// register-streaming tile with the full evaluation of every entry: 517), 128 rows 181 us (280).  The longer K, the less the epilogue counts: 128 x 128 against
// 256 x 256 tiles 408 / 427 us at hidden 4096, 504 / 485 at 5120; at 512 rows 457 / 489, 702 / 677, 873 / 793.
template <class L, bool SCORE>
__global__ __launch_bounds__(L::T) void lmhead_ring_kernel(const u32x4v *__restrict__ Xp, const h16x8 *__restrict__ Wp, int Mp, int Np, int Kp, int V,
                                                           float temperature, uint64_t seed, DrawIds ids, const int32_t *__restrict__ target,
                                                           float *__restrict__ target_z, float *__restrict__ part, int strips) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  constexpr int MB = L::MB, NBW = L::NBW;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31, nblocks = Np >> 5;
  int bx, by, bz;
  ring_tile(strips, Mp / L::ROWS, &bx, &by, &bz);
  const int nb0 = bx * L::NB + (w % L::WC) * NBW, mrow0 = bz * L::ROWS, wrow = (w / L::WC) * 32 * MB, v0 = nb0 * 32 + 4 * half;
  f32x16 acc[NBW][MB];
  ring_mainloop<L>(acc, (u32x4v *)lds_raw, Xp, Wp, Mp, Kp, nblocks, bx * L::NB, mrow0, 0, Kp >> 4);
  float *dump = (float *)lds_raw + w * LM_DUMP_FLOATS;   // the ring is free
  SampleAcc (*sh)[L::ROWS] = (SampleAcc (*)[L::ROWS])(lds_raw + L::WN * LM_DUMP_FLOATS * 4);   // [WC][ROWS]
  static_assert(L::WN * LM_DUMP_FLOATS * 4 + L::WC * L::ROWS * (int)sizeof(SampleAcc) <= L::BYTES, "the epilogue fits the ring");
#pragma unroll
  for (int j = 0; j < MB; ++j) {
    const int row = wrow + j * 32 + col, m = mrow0 + row;
    f32x16 x[NBW];
#pragma unroll
    for (int n = 0; n < NBW; ++n) x[n] = acc[n][j];
    SampleAcc sa;
    if (SCORE) sa = score_lane<NBW>(x, v0, V, temperature, target[m], target_z + m);
    else sa = sample_lane<NBW>(x, dump, v0, V, temperature, seed, draw_stream(ids, m), draw_step(ids, m));
    SampleAcc o = sample_acc_shfl_xor(sa, 32);
    sample_acc_merge(sa, o);
    if (half == 0) sh[w % L::WC][row] = sa;
  }
  __syncthreads();
  for (int r = threadIdx.x; r < L::ROWS; r += L::T) {   // the four column pairs of a row, lower indices first
    SampleAcc sa = sh[0][r];
#pragma unroll
    for (int c = 1; c < L::WC; ++c) sample_acc_merge(sa, sh[c][r]);
    const int64_t o = (int64_t)bx * Mp + mrow0 + r, plane = (int64_t)strips * Mp;
    if (SCORE) score_part_store(part, o, sa);
    else sample_part_store(part, o, plane, sa);
  }
}

template <class L, bool SCORE>
static void lmhead_ring_launch(const void *Xp, const void *Wp, int Mp, int Np, int Kp, int V, float temperature, uint64_t seed, DrawIds ids,
                               const int32_t *target, float *target_z, float *part, int strips, hipStream_t st) {
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void *)lmhead_ring_kernel<L, SCORE>, hipFuncAttributeMaxDynamicSharedMemorySize, L::BYTES);
    attr_set = true;
  }
  hipLaunchKernelGGL((lmhead_ring_kernel<L, SCORE>), dim3(strips * (Mp / L::ROWS)), dim3(L::T), L::BYTES, st, (const u32x4v *)Xp, (const h16x8 *)Wp,
                     Mp, Np, Kp, V, temperature, seed, ids, target, target_z, part, strips);
}

// grid M rows, block 256: fold the per-workgroup partials of one row in workgroup order.  sums_only: a scoring pass, whose partials are
// the maximum and the sum only; only target_lp is written.  Otherwise the row's bookkeeping follows, if the pass has any (a launch of its
// own before: 10.6 + 3.9 us at one row, 10.4 + 4.5 at 64; 12.3 together).  The lines that one compute unit can fetch bound it, 1187
// workgroups' times five while each value had a plane of its own, two with four of them side by side (sample_part_store): 12.3 -> 8.8 us
// at one row, 10.2 at 64, 17.2 -> 15.1 at 256, 4096 rows of a scoring pass 33 -> 28.5, and the lm_heads as before.  Requesting a thread's
// five partials at once changed nothing.
__global__ void sample_combine_kernel(int32_t *tok, float *lp, float *target_lp, const float *part, int n_wg, int Mp,
                                      const int32_t *target, const float *target_z, int sums_only, StepBook book) {
  __shared__ SampleAcc sh[4];
  int m = blockIdx.x;
  int64_t plane = (int64_t)n_wg * Mp;
  SampleAcc a = sample_acc_init();
  for (int g = threadIdx.x; g < n_wg; g += blockDim.x) {
    int64_t o = (int64_t)g * Mp + m;
    SampleAcc b;
    if (sums_only) { b = sample_acc_init(); b.zmax = part[2 * o]; b.zsum = part[2 * o + 1]; }
    else b = sample_part_load(part, o, plane);
    if (g == (int)threadIdx.x) a = b;   // (as it is: a row of NaN has no maximum, and a merge would drop its sum)
    else sample_acc_merge(a, b);
  }
  for (int o = 32; o > 0; o >>= 1) { SampleAcc b = sample_acc_shfl_xor(a, o); sample_acc_merge(a, b); }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) sample_acc_merge(a, sh[w]);
    float lse = a.zmax + logf(a.zsum);
    if (!sums_only) {
      tok[m] = a.idx; lp[m] = a.zbest - lse;
      if (book.d_step) book_row(book, m, a.idx, a.zbest - lse);
    }
    if (target_lp) target_lp[m] = (target && target[m] >= 0) ? target_z[m] - lse : 0.f;
  }
}

static int lm_wgs(int Np) { return (Np / 32 + LM_WN - 1) / LM_WN; }
size_t fast_lmhead_partial_floats(int Np, int Mp) { return (size_t)5 * lm_wgs(Np) * Mp + Mp; }

template <int MB, int NSTAGE, bool LOGITS, int WN = LM_WN>
static void lmhead_launch(const void *Xp, const void *Wp, int Mp, int Np, int Kp, int V, float temperature, uint64_t seed,
                          DrawIds ids, const int32_t *target, float *target_z, float *part, float *logits, int64_t ld,
                          hipStream_t st) {
  using L = GemmLds<MB, WN>;
  constexpr int SH = LOGITS ? 0 : LM_WN * LM_DUMP_FLOATS * 4 + 3 * MB * 32 * (int)sizeof(SampleAcc);
  constexpr int BYTES = L::X_BYTES > SH ? L::X_BYTES : SH;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void *)lmhead_kernel<MB, NSTAGE, LOGITS, WN>, hipFuncAttributeMaxDynamicSharedMemorySize, BYTES);
    attr_set = true;
  }
  const int n_wg = (Np / 32 + WN - 1) / WN;
  dim3 grid(n_wg), block(WN * 64);
  hipLaunchKernelGGL((lmhead_kernel<MB, NSTAGE, LOGITS, WN>), grid, block, BYTES, st, (const u32x4v *)Xp, (const h16x8 *)Wp, Mp, Np, Kp, V,
                     temperature, seed, ids, target, target_z, part, n_wg, logits, ld);
}

// 128 rows of logits: every workgroup reads all activations, 4 of its WN + 4 blocks' worth of loads per k-step, and a compute unit holds
// one workgroup.  Seven wavefronts (two per SIMD, inside 256 registers with two chunks of weights and half as many operands in flight; nothing
// spilled, where the form of four wavefronts spills 35) where rounds x (WN + 4) is less.  That count only orders the two forms: 151936 entries at hidden
// 4096, 3 x 11 against 5 x 8, take 256.7 us for 277.7 (4.8 TB/s of weights; a unit drains and fills again between its rounds).  Decode steps with
// nucleus sampling at hidden 2560 and 4096, wherever it takes seven: 1025 to 1280 blocks 8 % faster, 2049 blocks 1 to 2 %, 3073 blocks 8 to 10 %;
// at 1793 and 4096 blocks it stays with four.
static bool logits128_wide(int Np) {
  auto cost = [&](int wn) { return ((Np / 32 + wn - 1) / wn + 255) / 256 * (wn + 4); };
  return cost(7) < cost(LM_WN);
}

template <bool LOGITS>
static void lmhead_dispatch(const void *Xp, const void *Wp, int Mp, int Np, int Kp, int V, float temperature, uint64_t seed,
                            DrawIds ids, const int32_t *target, float *target_z, float *part, float *logits,
                            int64_t ld, hipStream_t st) {
  int mbt = Mp / 32;
#define LM_ARGS Xp, Wp, Mp, Np, Kp, V, temperature, seed, ids, target, target_z, part, logits, ld, st
  if constexpr (LOGITS) {
    if (mbt == 4) {
      if (logits128_wide(Np)) lmhead_launch<4, 2, LOGITS, 7>(LM_ARGS); else lmhead_launch<4, 3, LOGITS>(LM_ARGS);
      return;
    }
  }
  if (mbt == 2) lmhead_launch<2, 2, LOGITS>(LM_ARGS);
  else lmhead_launch<1, 3, LOGITS>(LM_ARGS);
#undef LM_ARGS
}

void fast_lmhead_sample(int32_t *tok, float *lp, float *target_lp, const void *Xp, const void *Wp, int Mp, int M, int V,
                        int Np, int Kp, float temperature, uint64_t seed, DrawIds ids,
                        const int32_t *target, const StepBook &book, float *partials, hipStream_t st) {
  const bool ring = Mp % 128 == 0, big = ring && target && Mp % 256 == 0;   // see lmhead_ring_kernel
  int n_wg = big ? (Np / 32 + Ring256x256::NB - 1) / Ring256x256::NB : lm_wgs(Np);
  float *target_z = partials + (size_t)5 * lm_wgs(Np) * Mp;   // behind the partials of either form
  if (big) lmhead_ring_launch<Ring256x256, true>(Xp, Wp, Mp, Np, Kp, V, temperature, seed, ids, target, target_z, partials, n_wg, st);
  else if (ring && target) lmhead_ring_launch<Ring128x128, true>(Xp, Wp, Mp, Np, Kp, V, temperature, seed, ids, target, target_z, partials, n_wg, st);
  else if (ring) lmhead_ring_launch<Ring128x128, false>(Xp, Wp, Mp, Np, Kp, V, temperature, seed, ids, target, target_z, partials, n_wg, st);
  else lmhead_dispatch<false>(Xp, Wp, Mp, Np, Kp, V, temperature, seed, ids, target, target_z, partials, nullptr, 0, st);
  hipLaunchKernelGGL(sample_combine_kernel, dim3(M), dim3(256), 0, st, tok, lp, target_lp, partials, n_wg, Mp, target,
                     target_z, target ? 1 : 0, book);
}

void fast_sample_combine(int32_t *tok, float *lp, const float *part, int n_parts, int M, int Mp, const StepBook &book, hipStream_t st) {
  hipLaunchKernelGGL(sample_combine_kernel, dim3(M), dim3(256), 0, st, tok, lp, (float *)nullptr, part, n_parts, Mp, (const int32_t *)nullptr,
                     (const float *)nullptr, 0, book);
}

void fast_lmhead_logits(float *logits, const void *Xp, const void *Wp, int Mp, int Np, int Kp, int V, hipStream_t st) {
  // 256 rows, vocabulary 151936, hidden 2560 / 4096 / 5120: 235 / 352 / 421 us on 256 x 256 ring tiles (256 x 128: 239 / 363 / 445, 128 x 128: 279 / 428 / 532, the
  // LDS-staged kernel at 2560: 296).  128 rows: 173 / 259 / 316 us by workgroups of seven blocks (see logits128_wide), 189 / 288 / 345 on 128 x 128 ring tiles.
  if (Mp % 256 == 0) { gemm_ring_launch<Ring256x256, EPI_PARTIAL>(logits, Xp, Wp, Mp, Np, Kp, 1, st); return; }
  lmhead_dispatch<true>(Xp, Wp, Mp, Np, Kp, V, 1.0f, 0, DrawIds{nullptr, nullptr, nullptr}, nullptr, nullptr, nullptr, logits, Np, st);
}

}  // namespace echo
