// RoPE for segmented execution (Sec. 3.4 "RoPE Re-indexing for Prefix Concatenation",
// Appendix E).  The paper gives a prefix of length P the key positions 0..P-1 and the segment's
// queries and keys the positions P..P+m-1.  Standard RoPE scores depend on position differences
// only, so for a prefix that is a contiguous run of tokens ending at the segment start (the
// carried tail, the whole history) this is the same as rotating every token once by its
// absolute position -- which is what rope_apply_kernel does, in place, before the rows are
// attended to and committed.  A retrieved prefix is not contiguous: its rows are turned to the
// positions s-R .. s-1 just before the segment when they are gathered (cache_select_kernel).
//
// Channel pair (i, i + D/2) is turned by position * theta^(-2i/D).  The angle is formed and
// reduced to [-pi, pi] in double precision (a float product is off by up to 0.01 rad at
// position 10^5), sine and cosine are single precision.  HBM-bound: every element is read and
// written once.
#include <math.h>

#include "segattn_internal.h"

namespace segattn {

// sine and cosine of pos * inv_freq, the angle reduced to [-pi, pi] in double precision
__device__ inline void rope_sincos(double pos, double inv_freq, float &sn, float &cs) {
  const double a = pos * inv_freq;
  const double two_pi = 6.283185307179586476925286766559, inv_two_pi = 0.15915494309189533576888376337251;
  const float r = (float)(a - two_pi * rint(a * inv_two_pi));
  sincosf(r, &sn, &cs);
}

// Rotate 8 consecutive channels (lo) with their partners D/2 further on (hi).
__device__ inline void rope_rotate8(uint4 &lo, uint4 &hi, const float (&sn)[8], const float (&cs)[8]) {
  unsigned *lw = (unsigned *)&lo, *hw = (unsigned *)&hi;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    unsigned lo_out = 0, hi_out = 0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float a = __uint_as_float(e ? (lw[w] & 0xffff0000u) : (lw[w] << 16));
      const float b = __uint_as_float(e ? (hw[w] & 0xffff0000u) : (hw[w] << 16));
      const __bf16 ya = (__bf16)(a * cs[2 * w + e] - b * sn[2 * w + e]);
      const __bf16 yb = (__bf16)(a * sn[2 * w + e] + b * cs[2 * w + e]);
      lo_out |= (unsigned)__builtin_bit_cast(unsigned short, ya) << (16 * e);
      hi_out |= (unsigned)__builtin_bit_cast(unsigned short, yb) << (16 * e);
    }
    lw[w] = lo_out;
    hw[w] = hi_out;
  }
}

// A workgroup rotates up to kRopeRows consecutive token rows: its threads form the sines and cosines of
// their D/2 channel pairs once, in LDS, and then walk over the rows' q and over their k in memory order, a
// thread taking 8 channel pairs of one head at a time (16 bytes and their partners D/2 further on).
// Bound by HBM, each element read and written in place; what counts is the order of the accesses: with a
// thread per (row, 8 channel pairs) that walked over all heads of its row, all waves were at the same head
// of different rows (the same few addresses modulo the row size) and formed sines first, and 32K rows of
// 32 + 8 heads took 152 us; in memory order 135 (5.0 TB/s), 500 rows 4.7 instead of 11.8.  One 16-byte pair in flight per
// thread: the in-place probe is fastest so (5.7 TB/s; eight pieces: 4.0).  A thread's first piece of q is requested
// before the sines are formed, so that the two waits do not add up: 28K rows of 4 + 4 heads of 64 9.0 -> 8.7 us (a
// thread per row 8.8), 32K rows of 32 + 8 heads of 128 122.6 -> 121.1 in a loop over one buffer.
constexpr int kRopeRows = 16;
template <int D>
__global__ __launch_bounds__(256) void rope_apply_kernel(const Problem p, const RopeArgs a, const int rows_per_wg) {
  constexpr int LPH = D / 16, kPairs = D / 2;  // threads per head; channel pairs
  __shared__ __attribute__((aligned(16))) float sm_sn[kRopeRows][kPairs], sm_cs[kRopeRows][kPairs];
  const int tid = threadIdx.x;
  const long long total = (long long)p.B * a.rows, row0 = (long long)blockIdx.x * rows_per_wg;
  const int n_rows = total - row0 < rows_per_wg ? (int)(total - row0) : rows_per_wg;
  const int li = tid % LPH;
  uint4 lo, hi;  // the piece in hand
  auto load = [&](const unsigned short *at) __attribute__((always_inline)) {
    lo = *(const uint4 *)at;
    hi = *(const uint4 *)(at + kPairs);
  };
  const int r_q = tid / (p.Hq * LPH);
  if (r_q < n_rows) load(a.q + ((row0 + r_q) * p.Hq + (tid - r_q * p.Hq * LPH) / LPH) * D + 8 * li);
  for (int i = tid; i < n_rows * kPairs; i += 256) {
    const int r = i / kPairs, c = i % kPairs;
    const long long br = row0 + r, b = br / a.rows;
    const double pos = (double)((a.pos0 ? a.pos0[b] : 0) + (br - b * a.rows));
    float sn, cs;
    rope_sincos(pos, a.inv_freq[c], sn, cs);
    sm_sn[r][c] = sn;
    sm_cs[r][c] = cs;
  }
  __syncthreads();
  auto walk = [&](unsigned short *base, int heads, bool held) __attribute__((always_inline)) {
    const int per_row = heads * LPH;  // pieces of 8 channel pairs in a row
    unsigned short *const x = base + row0 * heads * D;
    int r = tid / per_row, u = tid - r * per_row;  // this thread's piece: row r, piece u of the row
    const int dr = 256 / per_row, du = 256 - dr * per_row;
    for (; r < n_rows; held = false) {
      unsigned short *const at = x + ((long long)r * heads + u / LPH) * D + 8 * li;
      if (!held) load(at);
      float sn[8], cs[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sn[e] = sm_sn[r][8 * li + e];
        cs[e] = sm_cs[r][8 * li + e];
      }
      rope_rotate8(lo, hi, sn, cs);
      *(uint4 *)at = lo;
      *(uint4 *)(at + kPairs) = hi;
      r += dr;
      u += du;
      if (u >= per_row) {
        u -= per_row;
        ++r;
      }
    }
  };
  walk(a.q, p.Hq, true);
  walk(a.k, p.Hkv, false);
}

hipError_t launch_rope_apply(const Problem &p, const RopeArgs &a, hipStream_t st) {
  // fewer rows per workgroup where sixteen would leave CUs idle
  const long long total = (long long)p.B * a.rows;
  long long rows = total / 1024;
  rows = rows < 1 ? 1 : rows > kRopeRows ? kRopeRows : rows;
  const long long blocks = (total + rows - 1) / rows;
  if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  if (p.D == 128) hipLaunchKernelGGL(rope_apply_kernel<128>, dim3((unsigned)blocks), dim3(256), 0, st, p, a, (int)rows);
  else hipLaunchKernelGGL(rope_apply_kernel<64>, dim3((unsigned)blocks), dim3(256), 0, st, p, a, (int)rows);
  return hipGetLastError();
}

}  // namespace segattn
