// The dK/dV work item of short training windows (scheme and reasons: segattn_bwd_split.hip), with the helpers that
// the split kernels share.
#pragma once
#include "segattn_bwd_tiles.h"

namespace segattn {

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
__device__ __forceinline__ void bwd_dkv_split_item(const Problem &p, const BwdArgs &a, const int blocks_per_seg, const int n_seg,
                                                   const int packed, const int bid, unsigned char *const smem) {
  using T = BwdTile<D>;
  using G = DkvSplitGeom<D, NW>;
  constexpr int NC = D / 16, NB = D / 32;

  // bid -> (key block, segment, KV head, sequence), longest first: the key blocks that reach into the
  // carried tail (they also see the whole next segment), then the others from the segment's start on.
  // packed (number_packed): the key blocks of the batch are numbered, the heads of a block side by side.
  int kb, seg, kv, b;
  if (packed) {
    kv = bid % p.Hkv;
    packed_block(p, a.cu_seqlens, bid / p.Hkv, kBwdStep, b, seg, kb);
  } else {
    const int per = n_seg * p.Hkv * p.B;
    const int ord = bid / per;
    const int kb_tail = (p.S - p.T) / kBwdStep;  // first key block with keys in the tail
    const int n_tail = p.T > 0 && kb_tail < blocks_per_seg ? blocks_per_seg - kb_tail : 0;
    kb = ord < n_tail ? kb_tail + ord : ord - n_tail;
    int rest = (bid % per + ord) % per;
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

}  // namespace segattn
