// Small kernels used by both the debug (fp32) and the MFMA (bf16) path: KV replication across a group, generator read-out, fills and row gathers.
#include <algorithm>

#include "echo_device.h"
#include "echo_kernels.h"

namespace echo {

// One key's row of a head is a whole number of 16-byte units, and every region starts on one, unless the all-fp32 path has a
// head_dim that is no multiple of 4.
__device__ __forceinline__ void copy_region(char *dst, const char *src, int64_t bytes, const KvGeom &kv) {
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  if (kv.head_dim * kv.elt_bytes % 16 == 0)
    for (int64_t i = first; i < bytes / 16; i += step) ((uint4 *)dst)[i] = ((const uint4 *)src)[i];
  else
    for (int64_t i = first; i < bytes / 4; i += step) ((uint32_t *)dst)[i] = ((const uint32_t *)src)[i];
}

// Copy the prompt part of slot p*G into slots p*G+1 .. p*G+G-1.  grid = (chunks, regions per slot, P*(G-1)).
// Plain form: a region is one head's K or V plane and the prompt is its first prompt_len rows.  Tiled form: a region
// is one head's K and V tiles and the prompt is its first ceil(prompt_len/32) tiles; with cut_only just the tile that the
// prompt fills in part, which every sequence goes on writing in its own slot -- the whole ones are read from slot p*G.
__global__ void kv_replicate_kernel(KvGeom kv, const int32_t *prompt_len, int G, int cut_only) {
  int p = blockIdx.z / (G - 1), g = blockIdx.z % (G - 1) + 1;
  int64_t region_bytes = kv.head_stride() * kv.elt_bytes * (kv.tiled ? 2 : 1), tile_bytes = (int64_t)64 * kv.head_dim * kv.elt_bytes;
  int64_t bytes = kv.tiled ? (prompt_len[p] + 31) / 32 * tile_bytes : (int64_t)prompt_len[p] * kv.head_dim * kv.elt_bytes;
  int64_t skip = cut_only ? prompt_len[p] / 32 * tile_bytes : 0;
  const char *src = (const char *)kv.base + ((int64_t)p * G) * kv.slot_stride() * kv.elt_bytes + blockIdx.y * region_bytes + skip;
  char *dst = (char *)kv.base + ((int64_t)p * G + g) * kv.slot_stride() * kv.elt_bytes + blockIdx.y * region_bytes + skip;
  copy_region(dst, src, bytes - skip, kv);
}

void launch_kv_replicate(KvGeom kv, const int32_t *prompt_len, int P, int G, int cut_only, hipStream_t st) {
  if (G <= 1 || P <= 0) return;
  int regions = kv.n_layers * kv.n_kv_heads * (kv.tiled ? 1 : 2), chunks = cut_only ? kv.head_dim / 32 : 8;   // cut_only: one tile, a unit per thread
  hipLaunchKernelGGL(kv_replicate_kernel, dim3(chunks, regions, P * (G - 1)), dim3(256), 0, st, kv, prompt_len, G, cut_only);
}

// Copy part of one cache slot's prompt into another slot, for a list of (src slot, dst slot, begin, end) quadruples.
// grid = (chunks, regions per slot, pairs).  Plain form: a region is one head's K or V plane and [begin, end) are rows
// (keys); tiled form: a region is one head's K and V tiles and [begin, end) are tiles of 32 keys.
__global__ void kv_copy_range_kernel(KvGeom kv, const int32_t *quads) {
  const int32_t *q = quads + 4 * blockIdx.z;
  int64_t unit_bytes = (kv.tiled ? 64 : 1) * (int64_t)kv.head_dim * kv.elt_bytes;
  int64_t region_bytes = kv.head_stride() * kv.elt_bytes * (kv.tiled ? 2 : 1);
  int64_t off = (int64_t)q[2] * unit_bytes, bytes = (int64_t)(q[3] - q[2]) * unit_bytes;
  if (bytes <= 0) return;
  const char *src = (const char *)kv.base + (int64_t)q[0] * kv.slot_stride() * kv.elt_bytes + blockIdx.y * region_bytes + off;
  char *dst = (char *)kv.base + (int64_t)q[1] * kv.slot_stride() * kv.elt_bytes + blockIdx.y * region_bytes + off;
  copy_region(dst, src, bytes, kv);
}

void launch_kv_copy_ranges(KvGeom kv, const int32_t *quads, int n_quads, hipStream_t st) {
  if (n_quads <= 0) return;
  int regions = kv.n_layers * kv.n_kv_heads * (kv.tiled ? 1 : 2);
  hipLaunchKernelGGL(kv_copy_range_kernel, dim3(8, regions, n_quads), dim3(256), 0, st, kv, quads);
}

// ---- row state and records between the device and pinned host memory ----------------------------------------------
// A continuous rollout reads the row state back, hands finished records over, opens new ones and uploads the row state at almost
// every step: each of these is one kernel that reads or writes pinned host memory itself, where a copy per array and per record
// cost the stream some 10 us each (4 + 3 per record + 4 per new sequence + 10 copies or fills).
// host [4][n]: token, position, active, generated length.
__global__ void rows_to_host_kernel(int32_t *host, RowState rows, const int32_t *gen_len, int n) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  host[r] = rows.token[r]; host[n + r] = rows.pos[r]; host[2 * n + r] = rows.active[r]; host[3 * n + r] = gen_len[r];
}

void launch_rows_to_host(int32_t *host, RowState rows, const int32_t *gen_len, int n, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(rows_to_host_kernel, dim3((n + 255) / 256), dim3(256), 0, st, host, rows, gen_len, n);
}

// host [10][n], in the order of the argument list.
__global__ void rows_from_host_kernel(const int32_t *host, RowState rows, SeqState seq, int n) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  int32_t *dst[10] = {rows.token, rows.pos, rows.active, rows.slot, rows.pslot, rows.ptiles, seq.prompt_len, seq.gen_len, seq.limit, seq.stream};
  int32_t v[10];
#pragma unroll
  for (int a = 0; a < 10; ++a) v[a] = host[(int64_t)a * n + r];   // all reads across the bus in flight together
#pragma unroll
  for (int a = 0; a < 10; ++a) dst[a][r] = v[a];
}

void launch_rows_from_host(const int32_t *host, RowState rows, SeqState seq, int n, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(rows_from_host_kernel, dim3((n + 255) / 256), dim3(256), 0, st, host, rows, seq, n);
}

// grid (chunks, records): record q, kept in cache slot slots[q], to host + q * 16 * max_new bytes as versions i64, tokens
// i32, log-probs f32, [max_new] each.
__global__ void records_to_host_kernel(char *host, const int32_t *slots, int max_new, const int32_t *tok, const float *lp, const int64_t *ver) {
  const int64_t r0 = (int64_t)slots[blockIdx.y] * max_new;
  char *rec = host + (int64_t)blockIdx.y * 16 * max_new;
  int64_t *hv = (int64_t *)rec;
  int32_t *ht = (int32_t *)(rec + (int64_t)8 * max_new);
  float *hl = (float *)(rec + (int64_t)12 * max_new);
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < max_new; t += gridDim.x * blockDim.x) { hv[t] = ver[r0 + t]; ht[t] = tok[r0 + t]; hl[t] = lp[r0 + t]; }
}

void launch_records_to_host(char *host, const int32_t *slots, int n, int max_new, const int32_t *tok, const float *lp, const int64_t *ver, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(records_to_host_kernel, dim3(std::min(16, (max_new + 255) / 256), n), dim3(256), 0, st, host, slots, max_new, tok, lp, ver);
}

// grid (chunks, records): the record of cache slot slots[q] starts empty; forced: its tokens to feed, host [n][max_new] (or null).
__global__ void records_begin_kernel(const int32_t *slots, int max_new, int32_t *tok, float *lp, int64_t *ver, int32_t *forced_dst, const int32_t *forced) {
  const int64_t r0 = (int64_t)slots[blockIdx.y] * max_new;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < max_new; t += gridDim.x * blockDim.x) {
    tok[r0 + t] = -1; lp[r0 + t] = 0.f; ver[r0 + t] = -1;
    if (forced) forced_dst[r0 + t] = forced[(int64_t)blockIdx.y * max_new + t];
  }
}

void launch_records_begin(const int32_t *slots, int n, int max_new, int32_t *tok, float *lp, int64_t *ver, int32_t *forced_dst, const int32_t *forced,
                          hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(records_begin_kernel, dim3(std::min(16, (max_new + 255) / 256), n), dim3(256), 0, st, slots, max_new, tok, lp, ver, forced_dst, forced);
}

__global__ void draw_bits_kernel(uint32_t *out, uint64_t seed, uint32_t n, uint32_t s, uint32_t i0, int count) {
  int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= count) return;
  uint32_t i = i0 + (uint32_t)j;
  u32x4 r = draw4(seed, n, s, i >> 2);
  uint32_t w[4] = {r.x, r.y, r.z, r.w};
  out[j] = w[i & 3u];
}

void launch_draw_bits(uint32_t *out, uint64_t seed, uint32_t n, uint32_t s, uint32_t i0, int count, hipStream_t st) {
  hipLaunchKernelGGL(draw_bits_kernel, dim3((count + 255) / 256), dim3(256), 0, st, out, seed, n, s, i0, count);
}

__global__ void fill_i32_kernel(int32_t *p, int32_t v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

void launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, v, n);
}

__global__ void gather_rows_kernel(float *dst, const float *src, const int32_t *src_row, int width) {
  int r = src_row[blockIdx.x];
  if (r < 0) return;
  for (int i = threadIdx.x; i < width; i += blockDim.x) dst[(int64_t)blockIdx.x * width + i] = src[(int64_t)r * width + i];
}

void launch_gather_rows_f32(float *dst, const float *src, const int32_t *src_row, int n_dst, int width, hipStream_t st) {
  if (n_dst <= 0) return;
  hipLaunchKernelGGL(gather_rows_kernel, dim3(n_dst), dim3(256), 0, st, dst, src, src_row, width);
}

// Group-wise normalised advantages (App. "Outcome-Based Returns and Group-wise Normalization"): one wave per group of
// G consecutive returns; mean and sample standard deviation (divisor G - 1) in double, A = (R - mean) / (std + eps).
__global__ void grpo_advantage_kernel(float *adv, const float *rewards, int G, float eps) {
  const float *r = rewards + (int64_t)blockIdx.x * G;
  int lane = threadIdx.x;
  double sum = 0;
  for (int j = lane; j < G; j += 64) sum += (double)r[j];
  for (int o = 32; o; o >>= 1) sum += __shfl_xor(sum, o);
  double mean = sum / G, ss = 0;
  for (int j = lane; j < G; j += 64) {
    double dv = (double)r[j] - mean;
    ss += dv * dv;
  }
  for (int o = 32; o; o >>= 1) ss += __shfl_xor(ss, o);
  double den = sqrt(ss / (G - 1)) + (double)eps;
  for (int j = lane; j < G; j += 64) adv[(int64_t)blockIdx.x * G + j] = (float)(((double)r[j] - mean) / den);
}

// Turn-aware response mask (App. "Turn-Aware Masking") and per-token advantages: one workgroup of 1024 threads per
// sequence walks the row in tiles of 4096 tokens, 4 consecutive tokens per thread; the turn index of a token is the
// carried count of turn starts plus a prefix sum over the tile (shuffles within a wave, LDS across the 16 waves).
// VEC: rows start 16-byte aligned (stride % 4 == 0), so the 4 tokens travel as one vector.
template <bool VEC>
__global__ void __launch_bounds__(1024) grpo_mask_kernel(uint8_t *mask, float *adv_tok, const int32_t *tokens, const int32_t *lens,
                                                        const float *adv, int stride, int32_t turn_start) {
  __shared__ int wave_tot[16];
  int n = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int32_t *row = tokens + (int64_t)n * stride;
  uint8_t *mrow = mask + (int64_t)n * stride;
  float *arow = adv_tok ? adv_tok + (int64_t)n * stride : nullptr;
  int len = lens[n];
  float a = adv[n];
  int carry = 0;
  for (int base = 0; base < stride; base += 4096) {
    int t0 = base + 4 * tid;
    int32_t tk[4];
    if (VEC && t0 + 3 < stride) {
      int4 v = *(const int4 *)(row + t0);
      tk[0] = v.x, tk[1] = v.y, tk[2] = v.z, tk[3] = v.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) tk[j] = t0 + j < stride ? row[t0 + j] : turn_start - 1;
    }
    int hit[4], cnt = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      hit[j] = (t0 + j < len && tk[j] == turn_start) ? 1 : 0;
      cnt += hit[j];
    }
    int inc = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      int up = __shfl_up(inc, o);
      if (lane >= o) inc += up;
    }
    if (lane == 63) wave_tot[w] = inc;
    __syncthreads();
    int before = carry + inc - cnt, total = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if (k < w) before += wave_tot[k];
      total += wave_tot[k];
    }
    carry += total;
    __syncthreads();
    int c = before;
    uint8_t m[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      c += hit[j];
      m[j] = (t0 + j < len && c > 1 && (c & 1)) ? 1 : 0;
    }
    if (VEC && t0 + 3 < stride) {
      *(uchar4 *)(mrow + t0) = make_uchar4(m[0], m[1], m[2], m[3]);
      if (arow) *(float4 *)(arow + t0) = make_float4(m[0] ? a : 0.f, m[1] ? a : 0.f, m[2] ? a : 0.f, m[3] ? a : 0.f);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (t0 + j < stride) {
          mrow[t0 + j] = m[j];
          if (arow) arow[t0 + j] = m[j] ? a : 0.f;
        }
    }
  }
}

void launch_grpo_tensors(uint8_t *mask, float *adv, float *adv_tok, const int32_t *tokens, const int32_t *lens, const float *rewards,
                         int n_seqs, int G, int stride, int32_t turn_start, float eps, hipStream_t st) {
  if (n_seqs <= 0) return;
  hipLaunchKernelGGL(grpo_advantage_kernel, dim3(n_seqs / G), dim3(64), 0, st, adv, rewards, G, eps);
  if (stride % 4 == 0)
    hipLaunchKernelGGL(grpo_mask_kernel<true>, dim3(n_seqs), dim3(1024), 0, st, mask, adv_tok, tokens, lens, adv, stride, turn_start);
  else
    hipLaunchKernelGGL(grpo_mask_kernel<false>, dim3(n_seqs), dim3(1024), 0, st, mask, adv_tok, tokens, lens, adv, stride, turn_start);
}

}  // namespace echo
