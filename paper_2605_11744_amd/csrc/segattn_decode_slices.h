// Slice search shared by the two decode split kernels of libsegattn.
#pragma once
#include "segattn_internal.h"

namespace segattn {

// Rows [lo, hi) of window w = b * Hkv + kv that the step attends to.  a.pending: the newest row is not in
// the cache yet (the split kernel takes it from the caller's k_new / v_new and writes it there), and
// the counters do not count it.
__device__ inline void decode_window_rows(const Problem &p, const DecodeArgs &a, int w, int &lo, int &hi) {
  const int kv = w % p.Hkv;
  const int *meta = meta_ro(a.cache, a.geom, p, w / p.Hkv, kv);
  int seg_row0;
  window_of(p, a.geom, kv, meta, lo, seg_row0);
  hi = seg_row0 + meta[META_FILL] + a.pending;
}

// The windows of all (sequence, KV head) pairs laid end to end in the order b * Hkv + kv; workgroup
// i owns rows [i * rows_per_wg, (i + 1) * rows_per_wg) of that sequence -- or, a.per_window, every window is cut
// into slices of its own, the last one shorter, and workgroup i owns the i-th slice.  Finds the window
// that holds the workgroup's first row, the row's offset inside it and the slice's number among those of the
// window; w = -1 if the slices before this one cover every row.  A thread of the first four waves adds up a run of consecutive windows; then every wave scans
// the 256 sums, four a lane, and walks the run that holds the row.  (One thread walking the sums took up to
// 10 us; every wave reading all counters by itself made the step 10 % longer.)  Called by all threads of
// the workgroup (it synchronises).
__device__ inline void decode_slice_start(const Problem &p, const DecodeArgs &a, int &w_out, int &off_out, int &split_out) {
  __shared__ __attribute__((aligned(16))) int sm_run[256];
  const int tid = threadIdx.x, lane = tid & 63;
  const int n_win = p.B * p.Hkv, run = (n_win + 255) / 256;
  const int per = a.rows_per_wg, start = (int)blockIdx.x * (a.per_window ? 1 : per);  // all rows fit the card: below 2^31
  auto units = [&](int rows) { return a.per_window ? (rows + per - 1) / per : rows; };
  if (tid < 256) {
    int sum = 0;
    for (int j = 0; j < run; ++j) {
      const int w = tid * run + j;
      if (w < n_win) {
        int lo, hi;
        decode_window_rows(p, a, w, lo, hi);
        sum += units(hi - lo);
      }
    }
    sm_run[tid] = sum;
  }
  __syncthreads();
  int part[4], incl = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    part[j] = sm_run[4 * lane + j];
    incl += part[j];
  }
  const int mine = incl;
#pragma unroll
  for (int sh = 1; sh < 64; sh <<= 1) {
    const int up = __shfl_up(incl, sh);
    if (lane >= sh) incl += up;
  }
  const unsigned long long reach = __builtin_amdgcn_ballot_w64(incl > start);
  w_out = -1;
  off_out = split_out = 0;
  if (reach == 0) return;
  const int L = (int)__builtin_ctzll(reach);
  int before = __builtin_amdgcn_readlane(incl - mine, L), t = 4 * L;
#pragma unroll
  for (int j = 0; j < 3; ++j) {  // the last of the four needs no look
    const int n = __builtin_amdgcn_readlane(part[j], L);
    if (t == 4 * L + j && before + n <= start) {
      before += n;
      ++t;
    }
  }
  int w = t * run;
  for (int j = 0; j + 1 < run; ++j) {
    int lo, hi;
    decode_window_rows(p, a, w, lo, hi);
    if (before + units(hi - lo) > start) break;
    before += units(hi - lo);
    ++w;
  }
  w_out = __builtin_amdgcn_readfirstlane(w);
  const int off = __builtin_amdgcn_readfirstlane(start - before);
  off_out = a.per_window ? off * per : off;
  // (the window's first row lies off rows before the slice's: the slices in between are whole ones)
  split_out = a.per_window ? off : (int)blockIdx.x - (start - off) / per;
}

// The same for a numbered launch: the workgroup's number gives the window and the slice, no counter
// is read.  A slice beyond the window's last row is empty; the caller finds that out from the rows.
__device__ inline void decode_slice_numbered(const Problem &p, const DecodeArgs &a, int &w_out, int &off_out, int &split_out) {
  const bool past = (int)blockIdx.x < a.wgs_past;
  const int i = (int)blockIdx.x - (past ? 0 : a.wgs_past);
  const FastDiv slots = past ? a.slots_past : a.slots_other, heads = past ? a.heads_past : a.heads_other;
  const int win = fast_div(i, slots), b = fast_div(win, heads);
  split_out = i - win * (int)slots.d;
  off_out = split_out * a.rows_per_wg;
  w_out = b * p.Hkv + p.order[(past ? 0 : p.n_past) + win - b * (int)heads.d];
}

}  // namespace segattn
