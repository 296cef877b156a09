// Forward kernel for launches with few query rows: a prompt of a few hundred to a few thousand
// tokens, short sequences packed together, a handful of rows behind a filled cache.
//
// With few rows the hand-pipelined kernel (segattn_prefill_mfma.hip) is bound by its longest
// workgroup: one workgroup walks all keys of its rows in order, 0.5 us per step of 32 keys with one
// wave per SIMD, while most of the chip idles.  Here the keys are what a workgroup shares out: its
// eight (or sixteen) waves hold the same 32 query columns (32/HS rows of HS heads of one GQA group) and wave w
// takes the key steps w, w + 8, ...; at the end the partial results meet in LDS.  The chain of
// dependent steps is an eighth, and there are as many workgroups as 32-column blocks.  The price: every
// wave stages its own K/V tile (16 KB of L2 traffic per wave and step, where the other kernel's
// eight waves share one) and nothing is scheduled by hand -- so it is chosen only where the
// other form leaves the chip waiting (choose_prefill in segattn_prefill_mfma.hip).  The form also takes the pieces
// of a prefix behind which a chunk has few rows (plan_pieces there).
//
// Products and layouts as in segattn_prefill_mfma.hip: S^T = K . Q^T, O^T += V^T . P^T with 32x32x16 bf16
// products, P straight from the S^T accumulators, weights rounded to bf16 and summed as rounded, a
// lazy reference maximum.  Tiles go HBM/L2 -> registers (one tile ahead) -> a wave-private LDS tile ->
// operands: no barrier before the merge.
#include <atomic>

#include "segattn_work.h"

namespace segattn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
#define LDS_AS __attribute__((address_space(3)))
#define GLB_AS __attribute__((address_space(1)))

constexpr int kSplitStep = 32;  // keys per step
constexpr int kSplitCols = 32;  // query columns per workgroup

template <int D, int NW>
struct SplitGeom {
  static constexpr int kRowBytes = 2 * D, kChunks = D / 8;
  static constexpr int kTensorBytes = kSplitStep * kRowBytes;
  static constexpr int kTileBytes = 2 * kTensorBytes;                    // [K rows][V rows] of one step
  static constexpr int kMerge = NW * kSplitCols * D * 4;        // the waves' O^T, fp32
  static constexpr int kTiles = NW * kTileBytes;
  static constexpr int kStats = kTiles > kMerge ? kTiles : kMerge;       // then [wave][column] m, l
  static constexpr int kBytes = kStats + NW * kSplitCols * 2 * 4;
  static constexpr int kRowsPer256 = 256 / kRowBytes;
  // 16-byte chunks of a row XOR-swizzled as in the other forward kernel (row reads and transposing
  // reads free of bank conflicts)
  __device__ static constexpr int swz_k(int row) { return (row / kRowsPer256) & (kChunks - 1) & 15; }
  __device__ static constexpr int swz_v(int row) { return 4 * ((row / kRowsPer256) % (kChunks / 4)); }
};

// Items: of whole sequences or an uncut chunk; of a packed batch; pieces (see resolve in segattn_work.h).  NW: waves.
enum { kPlainItems, kPackedItems, kPieceItems };
template <int D, int HS, int NW, int Items>
__global__ __launch_bounds__(64 * NW, D == 64 ? 4 : 2) void prefill_keysplit_kernel(const Problem p, const PrefillArgs a) {
  using G = SplitGeom<D, NW>;
  constexpr int NC = D / 16, NB = D / 32;
  constexpr int R = kSplitCols / HS;           // query rows per workgroup
  constexpr int RPL = 1024 / G::kRowBytes;     // rows per 1 KB wave load
  constexpr int NL = kSplitStep / RPL;         // loads per tile and tensor
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  WorkItem w = resolve<Items == kPackedItems, Items == kPieceItems>(p, a, (int)blockIdx.x, R, HS);
  if (!w.valid) return;
  pin_uniform(w);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hi = lane >> 5, col = lane & 31, i16 = lane & 15, g16 = (lane >> 4) & 1;
  const float c = p.scale_log2e;
  const int last_row = w.nq - 1;
  // this lane's query column: row t of the segment, head hcol of the sub-group
  const int hcol = col % HS;
  int t = w.t0 + col / HS;
  t = t < last_row ? t : last_row;

  const int n1_needed = w.t0 + R < w.n1 ? w.t0 + R : w.n1;
  const int nst0 = (w.n0 + kSplitStep - 1) / kSplitStep;
  const int n = nst0 + (n1_needed + kSplitStep - 1) / kSplitStep;

  bf16x8 Qr[NC];
  {
    const unsigned short *qrow = w.q + ((long long)t * p.Hq + w.kv * p.g + w.hsub * HS + hcol) * D + 8 * hi;
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) Qr[kc] = *(const bf16x8 *)(qrow + 16 * kc);
  }

  unsigned char *const tile = smem + wave * G::kTileBytes;
  int koff[NC];
#pragma unroll
  for (int kc = 0; kc < NC; ++kc) koff[kc] = col * G::kRowBytes + (((2 * kc + hi) ^ G::swz_k(col)) << 4);
  int voff[NB];
  {
    const int vrow = 4 * hi + (i16 >> 2);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int chunk = 4 * nb + 2 * g16 + ((i16 & 3) >> 1);
      voff[nb] = G::kTensorBytes + vrow * G::kRowBytes + ((chunk ^ G::swz_v(vrow)) << 4) + 8 * (i16 & 1);
    }
  }
  // Load i of a tile: row RPL i + lane / chunks, chunk lane % chunks.
  u32x4 nk[NL], nv[NL];
  const int lrow = lane / G::kChunks;
  const unsigned lchunk = (unsigned)(lane % G::kChunks) * 16;
  auto fetch = [&](int j) __attribute__((always_inline)) {
    const bool own = j >= nst0;
    const int r0 = (own ? j - nst0 : j) * kSplitStep, rows = own ? w.n1 : w.n0;
    const unsigned stride = (unsigned)(own ? w.stride1 : w.stride0) * 2;  // bytes between rows
    // (global pointers by name: they come out of scalar registers, and a load through a generic one counts as an
    // LDS access too, so that every LDS wait of a step waited for the next step's tile as well -- no prefetch)
    const GLB_AS unsigned char *kp = (const GLB_AS unsigned char *)(own ? w.k1 : w.k0) + (unsigned long long)r0 * stride;
    const GLB_AS unsigned char *vp = (const GLB_AS unsigned char *)(own ? w.v1 : w.v0) + (unsigned long long)r0 * stride;
    const int last = rows - 1 - r0;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = RPL * i + lrow < last ? RPL * i + lrow : last;  // the ragged end of a span: repeat its last row (masked below)
      const unsigned o = (unsigned)r * stride + lchunk;
      nk[i] = *(const GLB_AS u32x4 *)(kp + o);
      nv[i] = *(const GLB_AS u32x4 *)(vp + o);
    }
  };

  f32x16 O[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) O[nb][r] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;

  if (wave < n) fetch(wave);
  for (int j = wave; j < n; j += NW) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = RPL * i + lrow, ch = lane % G::kChunks;
      *(u32x4 *)(tile + r * G::kRowBytes + ((ch ^ G::swz_k(r)) << 4)) = nk[i];
      *(u32x4 *)(tile + G::kTensorBytes + r * G::kRowBytes + ((ch ^ G::swz_v(r)) << 4)) = nv[i];
    }
    if (j + NW < n) fetch(j + NW);
    f32x16 S = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < NC; ++kc)
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)(tile + koff[kc]), Qr[kc], S, 0, 0, 0);
    // register r of the lane is key 8 (r/4) + 4 hi + r%4 of the step; keys the lane's row may not see get -inf
    const bool own = j >= nst0;
    const int j0 = (own ? j - nst0 : j) * kSplitStep;
    if (own ? j0 + kSplitStep - 1 > w.t0 : j0 + kSplitStep > w.n0) {
      const int lim = (own ? t + 1 : w.n0) - j0 - 4 * hi;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + (r & 3) >= lim) S[r] = -INFINITY;
    }
    float mx = fmaxf(S[0], S[1]);
#pragma unroll
    for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, S[r]), S[r + 1]);
    {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_int(mx), __float_as_int(mx), false, false);
      mx = fmaxf(__int_as_float(sw[0]), __int_as_float(sw[1]));
    }
    // The reference maximum is raised (and what has been summed is scaled down) only where a weight
    // would exceed 2^8.  A column that has seen no key yet has none (-inf): the first key raises it.
    if (__builtin_amdgcn_ballot_w64((mx - m_ref) * c > 8.f)) {
      const float m_new = fmaxf(m_ref, mx);
      const float alpha = m_ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_ref - m_new) * c);
      m_ref = m_new;
      l_run *= alpha;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[nb][r] *= alpha;
    }
    const float mc = m_ref == -INFINITY ? 0.f : m_ref * c;
    bf16x8 P[2];
    float ps = 0.f;
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      f32x8 e;
#pragma unroll
      for (int x = 0; x < 8; ++x) e[x] = __builtin_amdgcn_exp2f(fmaf(S[8 * h2 + x], c, -mc));
      P[h2] = __builtin_convertvector(e, bf16x8);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const bf16x2 pr = {P[h2][2 * x], P[h2][2 * x + 1]};
        ps = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, ps, false);
      }
    }
    l_run += ps;
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const LDS_AS s16x4 *p0 = (const LDS_AS s16x4 *)(tile + voff[nb] + 16 * h2 * G::kRowBytes);
        const LDS_AS s16x4 *p1 = (const LDS_AS s16x4 *)(tile + voff[nb] + (16 * h2 + 8) * G::kRowBytes);
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4 *)p0);
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4 *)p1);
        const bf16x8 va = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
        O[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, P[h2], O[nb], 0, 0, 0);
      }
  }
  {  // the row sum of a column is split over the two half-waves
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_int(l_run), __float_as_int(l_run), false, false);
    l_run = __int_as_float(sw[0]) + __int_as_float(sw[1]);
  }

  // ---- the waves meet: O^T of wave w, column col at [w][col][D] fp32, 16-byte chunks swizzled by the column
  __syncthreads();  // every wave is done with its tile
  constexpr int kQ = D / 4;  // 16-byte chunks per column
  float *const stats = (float *)(smem + G::kStats);
  {
    unsigned char *const dst = smem + (wave * kSplitCols + col) * (D * 4);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int ch = 8 * nb + 2 * g4 + hi;
        const f32x4 o = {O[nb][4 * g4], O[nb][4 * g4 + 1], O[nb][4 * g4 + 2], O[nb][4 * g4 + 3]};
        *(f32x4 *)(dst + ((ch ^ (col & (kQ - 1))) << 4)) = o;
      }
    if (hi == 0) {
      stats[2 * (wave * kSplitCols + col)] = m_ref;
      stats[2 * (wave * kSplitCols + col) + 1] = l_run;
    }
  }
  __syncthreads();
  for (int idx = tid; idx < kSplitCols * kQ; idx += 64 * NW) {
    const int cc = idx / kQ, ch = idx % kQ;
    const int row = w.t0 + cc / HS;
    if (row > last_row) continue;
    float mx = -INFINITY;
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) mx = fmaxf(mx, stats[2 * (wv * kSplitCols + cc)]);
    float l = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
      const float wgt = __builtin_amdgcn_exp2f((stats[2 * (wv * kSplitCols + cc)] - mx) * c);  // a wave without keys: 0
      l = fmaf(stats[2 * (wv * kSplitCols + cc) + 1], wgt, l);
      const f32x4 x = *(const f32x4 *)(smem + (wv * kSplitCols + cc) * (D * 4) + ((ch ^ (cc & (kQ - 1))) << 4));
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = fmaf(x[e], wgt, o[e]);
    }
    const float inv = 1.f / l;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] *= inv;
    const int oh = w.ohead0 + cc % HS;
    const long long at = ((long long)row * w.out_heads + oh) * D + 4 * ch;
    if (w.wide) *(f32x4 *)((float *)w.out + at) = o;
    else *(uint2 *)((unsigned short *)w.out + at) = __builtin_bit_cast(uint2, __builtin_convertvector(o, bf16x4));
    if (ch == 0) w.lse[(long long)oh * w.lse_head_stride + row] = mx * p.scale + __logf(l);
  }
}

template <int D, int HS, int NW, int Items>
static hipError_t launch_split_d(const Problem &p, const PrefillArgs &a, long long grid, hipStream_t st) {
  auto kern = prefill_keysplit_kernel<D, HS, NW, Items>;
  constexpr int lds = SplitGeom<D, NW>::kBytes;
  static std::atomic<bool> ready{false};  // the same answer whoever asks first
  if (!ready.load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    ready.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * NW), lds, st, p, a);
  return hipGetLastError();
}

template <int D, int HS, int NW>
static hipError_t launch_split(const Problem &p, const PrefillArgs &a, long long grid, hipStream_t st) {
  if constexpr (NW == 8) {
    if (a.packed) return launch_split_d<D, HS, NW, kPackedItems>(p, a, grid, st);
    if (a.piece_rows.d != 0) return launch_split_d<D, HS, NW, kPieceItems>(p, a, grid, st);
  }
  return launch_split_d<D, HS, NW, kPlainItems>(p, a, grid, st);
}

template <int D, int NW>
static hipError_t launch_split_hs(const Problem &p, const PrefillArgs &a, int hs, long long grid, hipStream_t st) {
  if (hs == 4) return launch_split<D, 4, NW>(p, a, grid, st);
  if (hs == 2) return launch_split<D, 2, NW>(p, a, grid, st);
  return launch_split<D, 1, NW>(p, a, grid, st);
}

// Sixteen waves share out long chains of head dimension 64 where every workgroup has a CU to itself, eight -> sixteen: 68 rows
// behind 33K, 16/4 heads, with the commit 122 -> 101 us, 3 x 114 rows of 4/4 heads 109 -> 93, a prompt of 7953 rows, one
// head, 31.9 -> 28.5.  Of 1466 drawn chunks that stay uncut 1.2x in the mean from 256 steps on, 1.04x with 96 to
// 128 (none lost); not worth the larger merge where a chain is shorter (64 to 96 steps 0.97 to 1.04x, below 0.84 to 0.97x),
// nor with more workgroups than CUs (two of eight waves fit one).
int keysplit_waves(const Problem &p, const PrefillArgs &a, long long grid) {
  return p.D == 64 && grid <= device_cus() && !a.packed && a.piece_rows.d == 0 && a.longest_steps >= 96 ? 16 : 8;
}

hipError_t launch_prefill_keysplit(const Problem &p, const PrefillArgs &a, int hs, long long grid, hipStream_t st) {
  if (p.D == 128) return launch_split_hs<128, 8>(p, a, hs, grid, st);
  if (keysplit_waves(p, a, grid) == 16) return launch_split_hs<64, 16>(p, a, hs, grid, st);
  return launch_split_hs<64, 8>(p, a, hs, grid, st);
}

}  // namespace segattn
