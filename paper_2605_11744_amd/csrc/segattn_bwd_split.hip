// Backward kernels for small training windows: short sequences, few heads.
//
// The kernels in segattn_bwd_dq.hip and segattn_bwd_mfma.hip walk everything a workgroup's rows or
// keys meet in one chain of steps: a 128-key workgroup of the dK/dV kernel all query heads of its
// group and all their query steps, 0.5 us (D = 64) to 1 us a step.  With few workgroups the launch is
// as long as the longest of these chains.  Here the steps are what a workgroup's waves share out:
//
//   bwd_dkv_split_kernel   a workgroup owns 32 keys of one KV head; wave w takes the (query head, query
//                          step) pairs w, w + NW, ... of the group; the waves' dK, dV meet in LDS
//   bwd_dq_split_kernel    a workgroup owns 32 query columns (32/HS rows of HS heads of a group); wave w
//                          takes the key steps w, w + NW, ...; the waves' dQ meet in LDS
//
// Sums in a fixed order, no atomics: deterministic.  Arithmetic and layouts are those of the other
// kernels (score accumulators that start at -LSE/scale, dP at delta, V negated; 32x32x16 bf16
// products, P and dS rounded to bf16).  The price is that every wave stages its own tiles (16 KB a
// step at D = 128) where the other kernels share one among four waves, and that nothing is scheduled by
// hand; the launchers take these forms only where the chain is what bounds the other one.
#include <math.h>
#include <string.h>

#include <atomic>

#include "segattn_bwd_tiles.h"

namespace segattn {

constexpr int kDqSplitWaves = 8;

// A wave's two [32 x D] tiles, HBM/L2 -> registers: load i covers rows RPL i + lane / chunks.
template <int D>
struct TilePair {
  static constexpr int kRPL = 1024 / (2 * D), kLoads = kBwdStep / kRPL;
  u32x4 a[kLoads], b[kLoads];
  // rows r0 .. r0 + 31 of two tensors of the same row stride; rows beyond `last` repeat it.  (Global pointers
  // by name: a load through a generic one counts as an LDS access too, and every LDS wait of a step would
  // wait for the next step's tiles.)
  __device__ __forceinline__ void fetch(const GLB_AS unsigned char *pa, const GLB_AS unsigned char *pb, unsigned row_bytes, int last, int lane) {
    const int lrow = lane / BwdTile<D>::kChunks;
    const unsigned lchunk = (unsigned)(lane % BwdTile<D>::kChunks) * 16;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int r = kRPL * i + lrow < last ? kRPL * i + lrow : last;
      const unsigned o = (unsigned)r * row_bytes + lchunk;
      a[i] = *(const GLB_AS u32x4 *)(pa + o);
      b[i] = *(const GLB_AS u32x4 *)(pb + o);
    }
  }
  __device__ __forceinline__ void store(unsigned char *ta, unsigned char *tb, int lane) const {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int at = BwdTile<D>::at(kRPL * i + lane / BwdTile<D>::kChunks, lane % BwdTile<D>::kChunks);
      *(u32x4 *)(ta + at) = a[i];
      *(u32x4 *)(tb + at) = b[i];
    }
  }
};

// A wave's [D x 32] accumulators (lane = column) at [wave][column][D] fp32, 16-byte chunks swizzled by
// the column; then the sum over the waves, in order, of one 16-byte chunk of a column.
template <int D>
__device__ __forceinline__ void merge_store(unsigned char *smem, int wave, int lane, const f32x16 (&acc)[D / 32]) {
  const int hi = lane >> 5, col = lane & 31;
  unsigned char *const dst = smem + (wave * 32 + col) * (D * 4);
#pragma unroll
  for (int nb = 0; nb < D / 32; ++nb)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const f32x4 o = {acc[nb][4 * g4], acc[nb][4 * g4 + 1], acc[nb][4 * g4 + 2], acc[nb][4 * g4 + 3]};
      *(f32x4 *)(dst + (((8 * nb + 2 * g4 + hi) ^ (col & (D / 4 - 1))) << 4)) = o;
    }
}
template <int D, int NW>
__device__ __forceinline__ f32x4 merge_sum(const unsigned char *smem, int col, int chunk) {
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < NW; ++w) s += *(const f32x4 *)(smem + (w * 32 + col) * (D * 4) + ((chunk ^ (col & (D / 4 - 1))) << 4));
  return s;
}
__device__ __forceinline__ void store4(void *base, bool wide, long long at, const f32x4 x) {
  if (wide) *(f32x4 *)((float *)base + at) = x;
  else *(uint2 *)((unsigned short *)base + at) = __builtin_bit_cast(uint2, __builtin_convertvector(x, bf16x4));
}

// ---------------------------------------------------------------------------------------------
// dK, dV
// ---------------------------------------------------------------------------------------------
// NW waves per workgroup.  D = 128 holds 128 accumulator registers and 64 of K and V operands: one wave per
// SIMD, four waves.  D = 64: eight waves, or four with two workgroups per CU where there are enough
// workgroups (one's prologue and merge then run under the other's steps).
template <int D, int NW>
struct DkvSplitGeom {
  static constexpr int kWave = 2 * BwdTile<D>::kBytes;          // [Q tile][dO tile]
  static constexpr int kMerge = NW * 32 * D * 4;                // one of dK, dV at a time
  static constexpr int kTiles = NW * kWave > kMerge ? NW * kWave : kMerge;
  static constexpr int kStats = kTiles;                         // [wave][-LSE/scale x 32 | delta x 32]
  static constexpr int kBytes = kStats + NW * 64 * 4;
};

template <int D, int NW>
__global__ __launch_bounds__(64 * NW, D == 128 ? 1 : 2) void bwd_dkv_split_kernel(const Problem p, const BwdArgs a,
                                                                                 const int blocks_per_seg, const int n_seg,
                                                                                 const int packed) {
  using T = BwdTile<D>;
  using G = DkvSplitGeom<D, NW>;
  constexpr int NC = D / 16, NB = D / 32;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  // blockIdx -> (key block, segment, KV head, sequence), longest first: the key blocks that reach into the
  // carried tail (they also see the whole next segment), then the others from the segment's start on.
  // packed (number_packed): the key blocks of the batch are numbered, the heads of a block side by side.
  int kb, seg, kv, b;
  if (packed) {
    kv = (int)blockIdx.x % p.Hkv;
    packed_block(p, a.cu_seqlens, (int)blockIdx.x / p.Hkv, kBwdStep, b, seg, kb);
  } else {
    const int per = n_seg * p.Hkv * p.B;
    const int ord = blockIdx.x / per;
    const int kb_tail = (p.S - p.T) / kBwdStep;  // first key block with keys in the tail
    const int n_tail = p.T > 0 && kb_tail < blocks_per_seg ? blocks_per_seg - kb_tail : 0;
    kb = ord < n_tail ? kb_tail + ord : ord - n_tail;
    int rest = (blockIdx.x % per + ord) % per;
    seg = rest % n_seg;
    rest /= n_seg;
    kv = rest % p.Hkv;
    b = rest / p.Hkv;
  }
  const int pol = p.policy[kv];
  SeqSpan sq = seq_span(p, a, b);
  sq.row0 = uniform_i64(sq.row0);
  sq.n = uniform_i64(sq.n);
  sq.stat0 = uniform_i64(sq.stat0);
  sq.stat_stride = uniform_i64(sq.stat_stride);
  const long long s0 = (long long)seg * p.S;
  const long long seg_end = s0 + p.S < sq.n ? s0 + p.S : sq.n;
  const long long j0 = s0 + (long long)kb * kBwdStep;
  if (j0 >= seg_end) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hi = lane >> 5, col = lane & 31;
  const float c = p.scale_log2e;
  const int keys = (int)(seg_end - j0 < kBwdStep ? seg_end - j0 : kBwdStep);
  const long long koff = ((sq.row0 + j0 + (col < keys ? col : keys - 1)) * p.Hkv + kv) * D;
  bf16x8 Kr[NC], Vr[NC];  // K^T and (negated) V^T operands of the lane's key, matrix operands only
#pragma unroll
  for (int kc = 0; kc < NC; ++kc) {
    uint4 vv = *(const uint4 *)(a.v + koff + 16 * kc + 8 * hi);
    vv.x ^= 0x80008000u;
    vv.y ^= 0x80008000u;
    vv.z ^= 0x80008000u;
    vv.w ^= 0x80008000u;
    const uint4 kk = *(const uint4 *)(a.k + koff + 16 * kc + 8 * hi);
    if constexpr (D == 128) {
      Kr[kc] = park(kk);
      Vr[kc] = park(vv);
    } else {
      Kr[kc] = __builtin_bit_cast(bf16x8, kk);
      Vr[kc] = __builtin_bit_cast(bf16x8, vv);
    }
  }
  f32x16 dKa[NB], dVa[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      dKa[nb][r] = 0.f;
      dVa[nb][r] = 0.f;
    }

  // queries: own segment from row j0 on; then, for keys in the carried tail of the next segment, all
  // rows of that segment (one contiguous row range)
  const long long tail_lo = seg_end - p.T;
  long long next_end = seg_end;
  if ((pol & SEGATTN_TAIL) && seg_end == s0 + p.S && j0 + keys > tail_lo && seg_end < sq.n)
    next_end = seg_end + p.S < sq.n ? seg_end + p.S : sq.n;
  const int n_q = (int)(next_end - j0);
  const int steps_per_head = (n_q + kBwdStep - 1) / kBwdStep;
  const int n = steps_per_head * p.g;
  // the lane's differentiable queries, relative to j0: [col, q_lim)
  const int q_lim = col < keys ? (int)((j0 + col >= tail_lo ? next_end : seg_end) - j0) : 0;

  unsigned char *const tq = smem + wave * G::kWave, *const tg = tq + T::kBytes;
  float *const st = (float *)(smem + G::kStats) + wave * 64;
  const unsigned row_bytes = (unsigned)(p.Hq * D * 2);
  const long long head0 = ((sq.row0 + j0) * p.Hq + (long long)kv * p.g) * D;
  const long long stat0 = sq.stat0 + (long long)kv * p.g * sq.stat_stride + j0;
  const float *const stat_src = lane < kBwdStep ? a.nls : a.delta;
  TilePair<D> next;
  float next_stat = 0.f;
  auto fetch = [&](int it) __attribute__((always_inline)) {
    const int h = it / steps_per_head, q0 = (it - h * steps_per_head) * kBwdStep;
    const long long o = (head0 + (long long)h * D) * 2 + (long long)q0 * row_bytes;
    next.fetch((const GLB_AS unsigned char *)a.q + o, (const GLB_AS unsigned char *)a.dout + o, row_bytes, n_q - 1 - q0, lane);
    const int r = q0 + col < n_q ? q0 + col : n_q - 1;
    next_stat = stat_src[stat0 + h * sq.stat_stride + r];
  };
  if (wave < n) fetch(wave);
  for (int it = wave; it < n; it += NW) {
    const int q0 = (it % steps_per_head) * kBwdStep;
    next.store(tq, tg, lane);
    st[lane] = next_stat;
    if (it + NW < n) fetch(it + NW);
    f32x16 S, dP;  // register r of the lane: query 8 (r/4) + 4 hi + r%4 of the step
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const f32x4 x = *(const f32x4 *)(st + 8 * g4 + 4 * hi), y = *(const f32x4 *)(st + 32 + 8 * g4 + 4 * hi);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        S[4 * g4 + e] = x[e];
        dP[4 * g4 + e] = y[e];
      }
    }
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) mma_acc(S, read_row<D>(tq, lane, kc), Kr[kc]);
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) mma_acc(dP, read_row<D>(tg, lane, kc), Vr[kc]);
    // pairs that carry no gradient get weight 0: the diagonal, the end of the queries, a short key block
    if (q0 < kBwdStep || q0 + kBwdStep > (int)(seg_end - j0) || keys < kBwdStep) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = q0 + 8 * (r / 4) + 4 * hi + r % 4;
        S[r] = ((i >= col) & (i < q_lim)) ? S[r] : -INFINITY;
      }
    }
    bf16x8 P[2], dS[2];
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      f32x8 e, ds;
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        e[x] = __builtin_amdgcn_exp2f(S[8 * h2 + x] * c);
        ds[x] = e[x] * dP[8 * h2 + x];
      }
      P[h2] = __builtin_convertvector(e, bf16x8);
      dS[h2] = __builtin_convertvector(ds, bf16x8);
    }
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        mma_acc(dVa[nb], read_transposed<D>(tg, lane, nb, h2), P[h2]);
        mma_acc(dKa[nb], read_transposed<D>(tq, lane, nb, h2), dS[h2]);
      }
  }

  // the waves meet: dV, then dK (whose sign comes back with the scale: V was negated)
  constexpr int kQ = D / 4;
  const long long out0 = ((sq.row0 + j0) * p.Hkv + kv) * D;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
    merge_store<D>(smem, wave, lane, which ? dKa : dVa);
    __syncthreads();
    for (int idx = tid; idx < 32 * kQ; idx += 64 * NW) {
      const int cc = idx / kQ, ch = idx % kQ;
      if (cc >= keys) continue;
      f32x4 s = merge_sum<D, NW>(smem, cc, ch);
      if (which) s *= -p.scale;
      store4(which ? a.dk : a.dv, p.out_fp32 != 0, out0 + (long long)cc * p.Hkv * D + 4 * ch, s);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// dQ
// ---------------------------------------------------------------------------------------------
template <int D>
struct DqSplitGeom {
  static constexpr int kWave = 2 * BwdTile<D>::kBytes;  // [K tile][V tile]
  static constexpr int kMerge = kDqSplitWaves * 32 * D * 4;
  static constexpr int kBytes = kDqSplitWaves * kWave > kMerge ? kDqSplitWaves * kWave : kMerge;
};

template <int D, int HS, bool PK>
__global__ __launch_bounds__(64 * kDqSplitWaves, 2) void bwd_dq_split_kernel(const Problem p, const PrefillArgs pa, const BwdArgs a) {
  using T = BwdTile<D>;
  using G = DqSplitGeom<D>;
  constexpr int NC = D / 16, NB = D / 32, R = 32 / HS;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  WorkItem w = resolve<PK, false>(p, pa, (int)blockIdx.x, R, HS);
  if (!w.valid) return;
  pin_uniform(w);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hi = lane >> 5, col = lane & 31;
  const float c = p.scale_log2e;
  const int last_row = w.n1 - 1;
  const long long seg_row = (w.q - a.q) / ((long long)p.Hq * D);  // global row of the segment's first token
  const int head0 = w.kv * p.g + w.hsub * HS;
  int t = w.t0 + col / HS;  // this lane's query column: row t, head head0 + col % HS
  t = t < last_row ? t : last_row;
  const long long qoff = ((seg_row + t) * p.Hq + head0 + col % HS) * D;
  const long long stat = (w.lse - a.lse) + (long long)(head0 + col % HS) * w.lse_head_stride + t;
  const float lse = a.lse[stat], lse2 = lse * kLog2e;
  bf16x8 Qr[NC], Gr[NC];
#pragma unroll
  for (int kc = 0; kc < NC; ++kc) {
    Qr[kc] = *(const bf16x8 *)(a.q + qoff + 16 * kc + 8 * hi);
    Gr[kc] = *(const bf16x8 *)(a.dout + qoff + 16 * kc + 8 * hi);
  }
  const float delta = row_delta<NC>(a.out, p.out_fp32 != 0, qoff, hi, Gr);
  if (wave == 0 && hi == 0 && w.t0 + col / HS <= last_row) {  // for the dK/dV kernel; the eight waves hold the same columns
    a.delta[stat] = delta;
    a.nls[stat] = -lse / p.scale;
  }
  f32x16 acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nb][r] = 0.f;
  const int n1_needed = w.t0 + R < w.n1 ? w.t0 + R : w.n1;
  const int nst0 = (w.n0 + kBwdStep - 1) / kBwdStep;
  const int n = nst0 + (n1_needed + kBwdStep - 1) / kBwdStep;
  unsigned char *const tk = smem + wave * G::kWave, *const tv = tk + T::kBytes;
  const unsigned row_bytes = (unsigned)(w.stride1 * 2);  // both spans: the backward pass reads K/V by absolute position
  TilePair<D> next;
  auto fetch = [&](int j) __attribute__((always_inline)) {
    const bool own = j >= nst0;
    const int r0 = (own ? j - nst0 : j) * kBwdStep;
    const unsigned long long o = (unsigned long long)r0 * row_bytes;
    next.fetch((const GLB_AS unsigned char *)(own ? w.k1 : w.k0) + o, (const GLB_AS unsigned char *)(own ? w.v1 : w.v0) + o, row_bytes,
               (own ? w.n1 : w.n0) - 1 - r0, lane);
  };
  if (wave < n) fetch(wave);
  for (int j = wave; j < n; j += kDqSplitWaves) {
    next.store(tk, tv, lane);
    if (j + kDqSplitWaves < n) fetch(j + kDqSplitWaves);
    f32x16 S = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 dP = S;
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) {
      mma_acc(S, read_row<D>(tk, lane, kc), Qr[kc]);
      mma_acc(dP, read_row<D>(tv, lane, kc), Gr[kc]);
    }
    const bool own = j >= nst0;
    const int k0 = (own ? j - nst0 : j) * kBwdStep;
    if (own ? k0 + kBwdStep - 1 > w.t0 : k0 + kBwdStep > w.n0) {  // keys the lane's row may not see: weight 0
      const int lim = (own ? t + 1 : w.n0) - k0 - 4 * hi;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + (r & 3) >= lim) S[r] = -INFINITY;
    }
    bf16x8 dS[2];
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      f32x8 e;
#pragma unroll
      for (int x = 0; x < 8; ++x) e[x] = __builtin_amdgcn_exp2f(fmaf(S[8 * h2 + x], c, -lse2)) * (dP[8 * h2 + x] - delta);
      dS[h2] = __builtin_convertvector(e, bf16x8);
    }
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) mma_acc(acc[nb], read_transposed<D>(tk, lane, nb, h2), dS[h2]);
  }
  __syncthreads();
  merge_store<D>(smem, wave, lane, acc);
  __syncthreads();
  constexpr int kQ = D / 4;
  for (int idx = tid; idx < 32 * kQ; idx += 64 * kDqSplitWaves) {
    const int cc = idx / kQ, ch = idx % kQ, row = w.t0 + cc / HS;
    if (row > last_row) continue;
    const f32x4 s = merge_sum<D, kDqSplitWaves>(smem, cc, ch) * p.scale;
    store4(a.dq, p.out_fp32 != 0, ((seg_row + row) * p.Hq + head0 + cc % HS) * D + 4 * ch, s);
  }
}

// ---------------------------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------------------------
template <typename K>
static hipError_t allow_lds(K kern, int bytes, std::atomic<bool> &ready) {
  if (ready.load(std::memory_order_acquire)) return hipSuccess;  // the same answer whoever asks first
  const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) ready.store(true, std::memory_order_release);
  return e;
}

// Which form?  Estimates in microseconds from the longest chain of steps of a workgroup, the wave-steps in all and
// the rounds of workgroups, fitted to 11,123 windows and packed batches of 360 to 65,000 rows (eight numbers of
// heads, segments of 64 to 4096, every form of each timed): 0.6 % (D = 64) and 0.8 % (D = 128) slower than the best
// form on average; against the forms for large launches alone 13 of them more than 3 % slower, none more than 7 %.
// The split forms pay where those leave the chip waiting for a chain: 1024 rows, 32/8 heads of 64, 100 -> 48 us;
// 445 rows, 16/2 heads of 128, 76 -> 48.  They don't where waves that stage tiles of their own are bound by L2 (8192
// rows, 32/8 heads of 128, would lose 580 us), or by a further round of workgroups, however few they are (packed
// sequences of 10 to 60 rows, 8/8 heads of 128, 340 workgroups: 30 -> 41).  A forced launch shape keeps the other forms.
bool bwd_dq_split_pays(const Problem &p, const BwdArgs &a) {
  if (p.tune_waves != 0 || p.tune_queue != 0) return false;
  const long long total = a.cu_seqlens ? a.total : 0;
  const StepCount c = count_steps(p, a.n, total, 0);
  const double rounds = more_rounds(p.Hq * row_blocks(p, a.n, total, 32), device_cus());
  if (p.D == 64)
    return 9.48 - 0.22 * c.longest + 5.93e-4 * c.steps + 4.84 * rounds < 0.967 * (8 + fmax(0.349 * c.longest, 4.43e-4 * c.steps));
  return 11.1 - 0.066 * c.longest + 9.37e-4 * c.steps + 8.08 * rounds < 0.982 * (8 + fmax(0.487 * c.longest, 6.95e-4 * c.steps));
}
// dK/dV: waves of a workgroup of the split form (D = 64: eight, or four with two workgroups per CU), 0: the other form.
int bwd_dkv_split_waves(const Problem &p, const BwdArgs &a) {
  if (p.tune_waves != 0 || p.tune_queue != 0) return 0;
  const long long total = a.cu_seqlens ? a.total : 0;
  const double n = a.n, seqs = total > 0 ? total / n : p.B, cus = device_cus();
  const double seg = n < p.S ? n : p.S, segs = n / seg, per_seg = ceil(seg / 32), last = ceil(a.n % p.S / 32.);
  int n_tail = 0;
  for (int h = 0; h < p.Hkv; ++h) n_tail += p.policy[h] & SEGATTN_TAIL ? 1 : 0;
  const bool tails = n_tail > 0 && segs > 1 && p.T > 0;
  const double next = segs < 2 ? n - seg : seg;  // rows of a following segment
  // wave-steps of either form (the other one's in 128-key blocks of four waves); steps of the longest block of
  // either, all query heads of the group
  auto own128 = [](double steps) {
    const double blocks = ceil(steps / 4);
    return 4 * (blocks * steps - 2 * blocks * (blocks - 1));
  };
  const double whole = a.n / p.S, tail_segs = tails ? (segs > 2 ? segs - 1 : 1) * next / 32 : 0;
  const double steps = seqs * p.g * (p.Hkv * (whole * per_seg * (per_seg + 1) + last * (last + 1)) / 2 + n_tail * tail_segs * ceil(p.T / 32.));
  const double steps128 = seqs * p.g * (p.Hkv * (whole * own128(per_seg) + own128(last)) + n_tail * tail_segs * 4 * ceil(p.T / 128.));
  const double chain = p.g * fmax(per_seg, tails ? (p.T + next) / 32 : 0);
  const double chain128 = p.g * fmax(per_seg, tails ? (fmax(p.T, 128) + next) / 32 : 0);
  // workgroups; the other form's grid pads a packed batch: `empty` of them a CU find no keys
  const double blocks = p.Hkv * row_blocks(p, a.n, total, 32);
  double blocks128 = p.Hkv * row_blocks(p, a.n, 0, 128);
  if (total > 0) blocks128 = fmin(blocks128, p.Hkv * (total * ceil(p.S / 128.) / p.S + p.B / 2.));
  const double empty = fmax(p.Hkv * p.B * ceil(n / p.S) * ceil(seg / 128) - blocks128, 0) / cus;
  const double rounds = more_rounds(blocks, cus), rounds128 = more_rounds(blocks128, cus);
  if (p.D == 128) {
    const double split = 6.14 + 0.109 * chain + 1.3e-3 * steps + 4.4 * rounds;
    return split < 0.97 * (8 + fmax(0.5 * chain128, 9.28e-4 * steps128) + 1.96 * empty + 2.16 * rounds128) ? 4 : 0;
  }
  const double four = 6.34 + 0.335 * chain + 5.21e-4 * steps + 2.2 * more_rounds(blocks, 2 * cus);
  const double eight = 7.81 + 0.209 * chain + 7.45e-4 * steps + 2.84 * rounds;
  if (fmin(four, eight) >= 0.988 * (8 + fmax(0.709 * chain128, 5.15e-4 * steps128) + 9.82 * empty + 3.59 * rounds128)) return 0;
  return four <= eight ? 4 : 8;
}

template <int D, int NW>
static hipError_t launch_dkv_split_d(const Problem &p, const BwdArgs &a, hipStream_t st) {
  constexpr int lds = DkvSplitGeom<D, NW>::kBytes;
  static std::atomic<bool> ready{false};
  const hipError_t e = allow_lds(bwd_dkv_split_kernel<D, NW>, lds, ready);
  if (e != hipSuccess) return e;
  const int n_seg = (a.n + p.S - 1) / p.S;
  const long long seg_rows = a.n < p.S ? a.n : p.S;
  const int blocks_per_seg = (int)((seg_rows + kBwdStep - 1) / kBwdStep);
  const bool packed = a.cu_seqlens && number_packed(p, a.total, n_seg, blocks_per_seg, kBwdStep);
  const long long grid = packed ? (packed_units(a.total, p.S, kBwdStep) + p.B) * p.Hkv
                                : (long long)p.B * p.Hkv * n_seg * blocks_per_seg;
  if (grid <= 0 || grid > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((bwd_dkv_split_kernel<D, NW>), dim3((unsigned)grid), dim3(64 * NW), lds, st, p, a, blocks_per_seg, n_seg, (int)packed);
  return hipGetLastError();
}
hipError_t launch_bwd_dkv_split(const Problem &p, const BwdArgs &a, int waves, hipStream_t st) {
  if (p.D == 128) return launch_dkv_split_d<128, 4>(p, a, st);
  return waves == 4 ? launch_dkv_split_d<64, 4>(p, a, st) : launch_dkv_split_d<64, 8>(p, a, st);
}

template <int D, int HS, bool PK>
static hipError_t launch_dq_split_pk(const Problem &p, const PrefillArgs &pa, const BwdArgs &a, long long grid, hipStream_t st) {
  static std::atomic<bool> ready{false};
  const hipError_t e = allow_lds(bwd_dq_split_kernel<D, HS, PK>, DqSplitGeom<D>::kBytes, ready);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((bwd_dq_split_kernel<D, HS, PK>), dim3((unsigned)grid), dim3(64 * kDqSplitWaves), DqSplitGeom<D>::kBytes, st, p, pa, a);
  return hipGetLastError();
}
template <int D, int HS>
static hipError_t launch_dq_split_d(const Problem &p, const PrefillArgs &pa, const BwdArgs &a, long long grid, hipStream_t st) {
  return pa.packed ? launch_dq_split_pk<D, HS, true>(p, pa, a, grid, st) : launch_dq_split_pk<D, HS, false>(p, pa, a, grid, st);
}
hipError_t launch_bwd_dq_split(const Problem &p, const PrefillArgs &pa, const BwdArgs &a, int hs, long long grid, hipStream_t st) {
  if (p.D == 128) {
    if (hs == 4) return launch_dq_split_d<128, 4>(p, pa, a, grid, st);
    if (hs == 2) return launch_dq_split_d<128, 2>(p, pa, a, grid, st);
    return launch_dq_split_d<128, 1>(p, pa, a, grid, st);
  }
  if (hs == 4) return launch_dq_split_d<64, 4>(p, pa, a, grid, st);
  if (hs == 2) return launch_dq_split_d<64, 2>(p, pa, a, grid, st);
  return launch_dq_split_d<64, 1>(p, pa, a, grid, st);
}

}  // namespace segattn
