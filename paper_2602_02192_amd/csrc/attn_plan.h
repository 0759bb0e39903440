// The tile lists of the decode attention over several rows per workgroup (attn_rows_kernel in kernels_attn.hip), which the kernel
// that begins a step writes (step_begin_kernel in kernels_fast.hip).
#pragma once
#include "echo_device.h"
#include "echo_kernels.h"

namespace echo {

constexpr int ATT_TILE = 32;     // keys per tile
constexpr int ATT_ROWS_MAX = 8;            // rows per workgroup at most
constexpr int ATT_ROWS_WAVES = 8;
constexpr int ATT_ROWS_BATCH_MAX = 1024;   // rows of a batch that attn_rows_plan (one workgroup) deals
constexpr int ATT_SEG_MAX = 24;            // runs of rows with a common prompt (<= R/2) + two segments per row
constexpr int ATT_SEG_INTS = 8;            // cache slot, first tile, first and end position in the workgroup's tile list, first and end column, valid keys
constexpr int ATT_HDR_INTS = 16;           // number of rows, tiles in all, the rows
constexpr int ATT_PLAN_INTS = ATT_HDR_INTS + ATT_SEG_MAX * ATT_SEG_INTS;

// One workgroup of ATT_ROWS_BATCH_MAX threads, thread m for row m; NG row sets, each of at most ceil(M / NG) rows.
__device__ __forceinline__ void attn_rows_plan(int32_t *__restrict__ plan, const RowState &rows, int M, int grp, int NG) {
  __shared__ int32_t f[ATT_ROWS_BATCH_MAX][4];   // prompt slot, whole prompt tiles, keys, slot
  __shared__ int32_t order[ATT_ROWS_BATCH_MAX];  // the rows that are generating, in row order
  __shared__ int32_t wtot[ATT_ROWS_BATCH_MAX / 64 + 1];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const bool val = t < M && rows.active[t] != 0;
  if (val) { f[t][0] = rows.pslot[t]; f[t][1] = rows.ptiles[t] & ~ATT_PREFIX_DONE; f[t][2] = rows.pos[t] + 1; f[t][3] = rows.slot[t]; }
  const uint64_t bal = __ballot(val);
  if (lane == 0) wtot[w] = __popcll(bal);
  __syncthreads();
  int rank = __popcll(bal & ((1ull << lane) - 1)), n_act = 0;
  for (int i = 0; i < ATT_ROWS_BATCH_MAX / 64; ++i) { if (i < w) rank += wtot[i]; n_act += wtot[i]; }
  if (val) order[rank] = t;
  __syncthreads();
  // set t takes the generating rows of rank ceil(t n / NG) .. ceil((t + 1) n / NG) - 1: at most ceil(n / NG) of them
  const int first = (int)(((int64_t)t * n_act + NG - 1) / NG), end = (int)(((int64_t)(t + 1) * n_act + NG - 1) / NG), nr = t < NG ? end - first : 0;
  // The sets go into the list longest first (by tiles, shared ones counted per row): workgroups start in list order, so
  // when a launch has more workgroups than the chip holds at once the short ones fill in behind the long ones.
  int mine = 0;
  for (int r = 0; r < nr; ++r) mine += (f[order[first + r]][2] + ATT_TILE - 1) / ATT_TILE;
  __shared__ int32_t tot[ATT_ROWS_BATCH_MAX];
  if (t < NG) tot[t] = mine;
  __syncthreads();
  if (t >= NG) return;
  int place = 0;
  for (int u = 0; u < NG; ++u) place += tot[u] > mine || (tot[u] == mine && u < t);
  int32_t *hdr = plan + (int64_t)place * ATT_PLAN_INTS, *seg = hdr + ATT_HDR_INTS;
  int ns = 0, v = 0;
  auto emit = [&](int slot, int tile0, int n, int c0, int c1, int keys) {
    int32_t *s = seg + ns * ATT_SEG_INTS;
    s[0] = slot; s[1] = tile0; s[2] = v; s[3] = v + n; s[4] = c0; s[5] = c1; s[6] = keys; s[7] = 0;
    v += n;
    ++ns;
  };
  for (int r = 0; r < nr;) {
    const int32_t *a = f[order[first + r]];
    const int ps = a[0], pt = a[1];
    int r2 = r + 1, full = a[2] / ATT_TILE;
    while (r2 < nr) {
      const int32_t *b = f[order[first + r2]];
      if (b[0] != ps || b[1] != pt) break;
      full = min(full, b[2] / ATT_TILE);
      ++r2;
    }
    const int sh = r2 - r >= 2 ? min(pt, full) : 0;   // whole tiles that every row of the run reads from the same slot
    if (sh > 0) emit(ps, 0, sh, r * grp, r2 * grp, 0x7fffffff);
    for (int rr = r; rr < r2; ++rr) {
      const int32_t *b = f[order[first + rr]];
      const int nk = b[2], nt = (nk + ATT_TILE - 1) / ATT_TILE;
      int a0 = sh;
      const int e0 = min(pt, nt);
      if (e0 > a0) { emit(ps, a0, e0 - a0, rr * grp, (rr + 1) * grp, nk); a0 = e0; }   // prompt tiles the row reads alone
      if (nt > a0) emit(b[3], a0, nt - a0, rr * grp, (rr + 1) * grp, nk);
    }
    r = r2;
  }
  for (int i = ns; i < ATT_SEG_MAX; ++i) {   // unused entries lie beyond every tile
    int32_t *s = seg + i * ATT_SEG_INTS;
    s[0] = 0; s[1] = 0; s[2] = 0x7fffffff; s[3] = 0x7fffffff; s[4] = 0; s[5] = 0; s[6] = 0; s[7] = 0;
  }
  hdr[0] = nr; hdr[1] = v;
  for (int r = 0; r < ATT_ROWS_MAX; ++r) hdr[2 + r] = r < nr ? order[first + r] : -1;
}

}  // namespace echo
