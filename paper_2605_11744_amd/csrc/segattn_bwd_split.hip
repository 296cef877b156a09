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
// The dK/dV item itself is in segattn_bwd_dkv_split.h: where its chains are long against the work it shares one launch
// with the dQ items (bwd_both_kernel in segattn_bwd_dq.hip, rule below).
//
// Sums in a fixed order, no atomics: deterministic.  Arithmetic and layouts are those of the other
// kernels (score accumulators that start at -LSE/scale, dP at delta, V negated; 32x32x16 bf16
// products, P and dS rounded to bf16).  The price is that every wave stages its own tiles (16 KB a
// step at D = 128) where the other kernels share one among four waves, and that nothing is scheduled by
// hand; the launchers take these forms only where the chain is what bounds the other one.
#include <math.h>
#include <string.h>

#include <atomic>

#include "segattn_bwd_dkv_split.h"

namespace segattn {

constexpr int kDqSplitWaves = 8;

// ---------------------------------------------------------------------------------------------
// dK, dV
// ---------------------------------------------------------------------------------------------
template <int D, int NW>
__global__ __launch_bounds__(64 * NW, D == 128 ? 1 : 2) void bwd_dkv_split_kernel(const Problem p, const BwdArgs a,
                                                                                 const int blocks_per_seg, const int n_seg,
                                                                                 const int packed) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  bwd_dkv_split_item<D, NW>(p, a, blocks_per_seg, n_seg, packed, (int)blockIdx.x, smem);
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
// The split forms pay where those leave the chip waiting for a chain (groups of several heads where the two passes don't share
// one launch, bwd_both_pays): backward of 1024 rows, own segment and tail, 8/8 heads of 64 49.5 -> 22.1 us, 12/4 heads 87 -> 38,
// 16/1 heads 220 -> 75; 445 rows, 8/8 heads of 128, 39.7 -> 29.1; 4942 rows, 4/1 heads of 128, S = 163, 149 -> 103.  They don't where waves that stage tiles of their own are bound by L2 (8192
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
// What the dK/dV pass has to do: wave-steps of the split form (32-key blocks) and of the other one (in 128-key blocks of four
// waves); steps of the longest block of either, all query heads of the group.
struct DkvSteps {
  double steps, steps128, chain, chain128;
};
static DkvSteps dkv_steps(const Problem &p, const BwdArgs &a) {
  const long long total = a.cu_seqlens ? a.total : 0;
  const double n = a.n, seqs = total > 0 ? total / n : p.B;
  const double seg = n < p.S ? n : p.S, segs = n / seg, per_seg = ceil(seg / 32), last = ceil(a.n % p.S / 32.);
  int n_tail = 0;
  for (int h = 0; h < p.Hkv; ++h) n_tail += p.policy[h] & SEGATTN_TAIL ? 1 : 0;
  const bool tails = n_tail > 0 && segs > 1 && p.T > 0;
  const double next = segs < 2 ? n - seg : seg;  // rows of a following segment
  auto own128 = [](double steps) {
    const double blocks = ceil(steps / 4);
    return 4 * (blocks * steps - 2 * blocks * (blocks - 1));
  };
  const double whole = a.n / p.S, tail_segs = tails ? (segs > 2 ? segs - 1 : 1) * next / 32 : 0;
  DkvSteps d;
  d.steps = seqs * p.g * (p.Hkv * (whole * per_seg * (per_seg + 1) + last * (last + 1)) / 2 + n_tail * tail_segs * ceil(p.T / 32.));
  d.steps128 = seqs * p.g * (p.Hkv * (whole * own128(per_seg) + own128(last)) + n_tail * tail_segs * 4 * ceil(p.T / 128.));
  d.chain = p.g * fmax(per_seg, tails ? (p.T + next) / 32 : 0);
  d.chain128 = p.g * fmax(per_seg, tails ? (fmax(p.T, 128) + next) / 32 : 0);
  return d;
}
// dQ and dK/dV in one launch (bwd_both_kernel)?  It pays where the longest chain of the dK/dV items (1.5 us a step of
// four waves) is long against the work of all items spread over the chip's waves.  Of 450 drawn windows and packed
// batches of 1000 to 16,000 rows (backward alone, one launch against the better forms of two), D = 128 beyond a ratio
// of 1.0 gained 1.3x in the mean of those taken, one lost 2 %; below, the one wave per SIMD that the dK/dV item leaves
// the dQ items costs more than the idle end of a launch did (0.6x for a window of 5000 rows of 32/8 heads).  D = 64, two
// workgroups per CU either way, beyond 0.22: 1.14x, none lost (beyond 600,000 wave-steps some did, 0.87 to 1.05x).
// Groups of one head, and at D = 64 those that are no multiple of four, keep the split form of dQ, which is the faster one
// there (0.85x).  At D = 64 two launches also share a long chain out among eight waves, in this one the dQ items walk theirs
// alone and the dK/dV items with four.  That costs more than the second launch where there are few items and dQ's chain is
// the longer one (3678 rows of 4/1 heads, all of the past, S = 128: 35 us in two launches, 69 in one), and where the dK/dV
// items have a CU each and a chain far beyond dQ's, groups of eight heads and more (1024 rows of 16/1 heads, S = 512, 75
// and 88; 1024 of 8/1 43 and 48; but 4096 of 8/1 with the past, S = 512, 92 and 77).  Of 2343 drawn windows (1, 2, 4 and 8 KV
// heads, groups of 4 to 16) 2054 went beyond 0.22, 207 of them more than 3 % slower than in two launches; without these two kinds 60 of 1748
// (1.26x at worst), and of the 306 that they take out 62 had gained more than 3 % (8 % in the mean).
bool bwd_both_pays(const Problem &p, const BwdArgs &a) {
  if (p.tune_waves != 0 || p.tune_queue != 0) return false;
  if (p.g == 1 || (p.D == 64 && p.g % 4 != 0)) return false;
  const long long total = a.cu_seqlens ? a.total : 0;
  const DkvSteps d = dkv_steps(p, a);
  const StepCount q = count_steps(p, a.n, total, 0);
  const double cus = device_cus(), waves = 4 * cus, steps = d.steps + q.steps;
  if (p.D == 64) {
    if (steps > 600 * waves) return false;
    const double dq_items = p.Hkv * (p.g / 4) * row_blocks(p, a.n, total, 32), dkv_items = p.Hkv * row_blocks(p, a.n, total, 32);
    if (q.longest > 1.2 * d.chain && dq_items <= 0.83 * cus) return false;
    if (d.chain > 150 && ((q.longest <= 0.125 * d.chain && dkv_items <= cus) || (q.longest <= 0.15 * d.chain && dkv_items <= cus / 4)))
      return false;
  }
  return d.chain * (1.5 / 4) > (p.D == 64 ? 0.22 : 1.0) * steps / waves;
}
// dK/dV: waves of a workgroup of the split form (D = 64: eight, or four with two workgroups per CU), 0: the other form.
int bwd_dkv_split_waves(const Problem &p, const BwdArgs &a) {
  if (p.tune_waves != 0 || p.tune_queue != 0) return 0;
  const long long total = a.cu_seqlens ? a.total : 0;
  const double n = a.n, seg = n < p.S ? n : p.S, cus = device_cus();
  const auto [steps, steps128, chain, chain128] = dkv_steps(p, a);
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

DkvSplitGrid dkv_split_grid(const Problem &p, const BwdArgs &a) {
  DkvSplitGrid g;
  g.n_seg = (a.n + p.S - 1) / p.S;
  const long long seg_rows = a.n < p.S ? a.n : p.S;
  g.blocks_per_seg = (int)((seg_rows + kBwdStep - 1) / kBwdStep);
  g.packed = a.cu_seqlens && number_packed(p, a.total, g.n_seg, g.blocks_per_seg, kBwdStep);
  g.items = g.packed ? (packed_units(a.total, p.S, kBwdStep) + p.B) * p.Hkv
                     : (long long)p.B * p.Hkv * g.n_seg * g.blocks_per_seg;
  return g;
}

template <int D, int NW>
static hipError_t launch_dkv_split_d(const Problem &p, const BwdArgs &a, hipStream_t st) {
  constexpr int lds = DkvSplitGeom<D, NW>::kBytes;
  static std::atomic<bool> ready{false};
  const hipError_t e = allow_lds(bwd_dkv_split_kernel<D, NW>, lds, ready);
  if (e != hipSuccess) return e;
  const DkvSplitGrid g = dkv_split_grid(p, a);
  if (g.items <= 0 || g.items > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((bwd_dkv_split_kernel<D, NW>), dim3((unsigned)g.items), dim3(64 * NW), lds, st, p, a, g.blocks_per_seg, g.n_seg, g.packed);
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
