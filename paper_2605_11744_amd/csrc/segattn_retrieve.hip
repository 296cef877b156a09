// Top-k retrieval operator (Appendix D) for the long-range channel of libsegattn: from the
// previous segment's queries and a long-range head's past pool to the R pool rows that become
// the retrieved prefix.  The paper names the steps but none of their sizes; the sizes are
// parameters here (segattn_retrieval) and the steps are read as follows:
//
//   query construction   last L_q query rows of the previous segment, every query head of the
//                        group: means of consecutive windows of `pool_window` rows, plus the mean
//                        of the last `tail_avg` rows; rounded to bf16 (MFMA operands)
//   scoring              score(row) = max over the summaries of summary . key(row): one pass over
//                        the pool's K rows, HBM-bound (each row read once); the products are a
//                        dense [summaries x 128] x [128 x rows] contraction and run on the
//                        matrix cores so that the scan stays bandwidth-bound
//   top-k / anchors      the n_anchors rows with the highest scores, ties to the lower row.  (For
//                        any k >= n_anchors these are the anchors that "per-summary top-k,
//                        de-duplicate, keep the best" yields.)  Two levels: every chunk of 1024
//                        or 4096 rows (small chunks when few heads have to fill the chip)
//                        keeps its own best n_anchors next to the scores in LDS -- scores never
//                        go to HBM -- and one workgroup per head merges the candidates.  Both
//                        levels place a row by counting the rows that are better (64-bit keys from
//                        LDS, no chain of rounds): of the 256 threads' best rows those that at
//                        least n_anchors others beat rule out their threads, of the chunks' best
//                        rows likewise their chunks, and what is left is counted once more
//   window expansion     anchors in descending score order add rows a - win_before .. a + win_after
//                        (clipped to the visible pool, ascending, rows already in skipped) until
//                        R rows are in; then the earliest visible rows pad to R; sorted output
#include "segattn_internal.h"

namespace segattn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxAnchors = 32;

// (value, row) pairs ordered by value descending, then row ascending, as one number: the larger key is the
// better row.  0: no row (an invisible row's -inf).
__device__ inline unsigned long long row_key(float v, int row) {
  if (v == -INFINITY) return 0ull;
  const unsigned bits = __float_as_uint(v + 0.f);  // -0 and 0 are the same score
  const unsigned up = bits ^ ((bits >> 31) ? 0xffffffffu : 0x80000000u);
  return ((unsigned long long)up << 32) | (unsigned)~row;
}
__device__ inline int key_row(unsigned long long key) { return (int)~(unsigned)key; }
// Keys of list[0 .. n) (LDS, 16-byte aligned, n even) that are better than `key`; *some: those that are a row.
__device__ inline int count_better(const unsigned long long *list, int n, unsigned long long key, int *some = nullptr) {
  typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
  int better = 0, rows = 0;
#pragma unroll 8
  for (int i = 0; i < n; i += 2) {
    const u64x2 two = *(const u64x2 *)(list + i);
    better += (two[0] > key) + (two[1] > key);
    if (some) rows += (two[0] != 0) + (two[1] != 0);
  }
  if (some) *some = rows;
  return better;
}

// ---- query summaries: [B, n_past, NSP, D] bf16, NSP = g * n_sum rounded up to 32 (the padding
//      repeats summary 0, which cannot change a maximum).  One workgroup per (b, PAST head).
template <int D>
__global__ __launch_bounds__(256) void retrieve_summaries_kernel(const Problem p, const RetrieveArgs a) {
  constexpr int CH = D / 8;  // a thread forms 8 channels of one summary
  const int b = blockIdx.x / p.n_past, np = blockIdx.x % p.n_past;  // b: sequence, or (sequence, segment)
  const int kv = p.order[np];
  const PoolView pv = pool_view(p, a, b, kv);
  const int L = a.n_queries < a.m ? a.n_queries : a.m;
  const int n_win = (L + a.pool_window - 1) / a.pool_window;
  const int n_sum = n_win + 1;
  unsigned short *dst = a.summaries + ((long long)b * p.n_past + np) * a.nsp * D;
  for (int item = threadIdx.x; item < a.nsp * CH; item += 256) {
    const int s = item / CH, c = item % CH;
    const int sr = s < p.g * n_sum ? s : 0;           // padding rows repeat summary 0
    const int hq = kv * p.g + sr / n_sum, w = sr % n_sum;
    int r0, r1;                                        // rows [r0, r1) of the last L rows
    if (w < n_win) {
      r0 = w * a.pool_window;
      r1 = r0 + a.pool_window < L ? r0 + a.pool_window : L;
    } else {
      r0 = L - (a.tail_avg < L ? a.tail_avg : L);
      r1 = L;
    }
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const unsigned short *src = pv.q + ((long long)(a.m - L) * p.Hq + hq) * D + 8 * c;
    const long long stride = (long long)p.Hq * D;
#pragma unroll 4
    for (int r = r0; r < r1; ++r) {
      const uint4 x = *(const uint4 *)(src + r * stride);
      const unsigned xw[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] += __uint_as_float(xw[e] << 16);
        acc[2 * e + 1] += __uint_as_float(xw[e] & 0xffff0000u);
      }
    }
    const float inv_n = (float)(r1 - r0);
    unsigned o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const __bf16 lo16 = (__bf16)(acc[2 * e] / inv_n), hi16 = (__bf16)(acc[2 * e + 1] / inv_n);
      o[e] = (unsigned)__builtin_bit_cast(unsigned short, lo16) | ((unsigned)__builtin_bit_cast(unsigned short, hi16) << 16);
    }
    *(uint4 *)(dst + (long long)s * D + 8 * c) = uint4{o[0], o[1], o[2], o[3]};
  }
}

// ---- scoring + per-chunk candidates.  grid (chunks, B * n_past), 4 waves; a wave scores 32 rows
//      at a time: S[summary][row] = Sigma . K^T, A = summaries (registers), B = K rows in operand
//      layout (lane = row); the lane's 16 accumulator registers are 16 summaries of its row, so
//      the maximum over summaries is local.
template <int D, int NT, int kChunkRows>  // NT = NSP / 32 summary tiles; pool rows per workgroup
__global__ __launch_bounds__(256) void retrieve_score_kernel(const Problem p, const RetrieveArgs a) {
  constexpr int NC = D / 16;
  __shared__ float sc[kChunkRows];
  __shared__ __attribute__((aligned(16))) unsigned char stage[4][32 * 2 * D];  // one K tile per wave
  const int b = blockIdx.y / p.n_past, np = blockIdx.y % p.n_past;
  const int kv = p.order[np];
  const PoolView pv = pool_view(p, a, b, kv);
  const int pool = pv.pool, lo = pv.lo;
  const int c0 = blockIdx.x * kChunkRows;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, hi = lane >> 5, col = lane & 31;
  unsigned long long *cand = a.cand + (((long long)b * p.n_past + np) * a.n_chunks + blockIdx.x) * kMaxAnchors;
  if (c0 >= pool || c0 + kChunkRows <= lo) {  // nothing visible in this chunk
    if (tid < kMaxAnchors) cand[tid] = 0ull;
    return;
  }
  const unsigned short *sg = a.summaries + ((long long)b * p.n_past + np) * a.nsp * D;
  bf16x8 A[NT][NC];  // summary (32 t + col), channels 16 kc + 8 hi .. +7
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) A[t][kc] = *(const bf16x8 *)(sg + (long long)(32 * t + col) * D + 16 * kc + 8 * hi);
  // K rows travel HBM -> registers with coalesced wave loads (a pool in the cache arena is
  // contiguous: 1 KB per load; rows of a token-major prompt are 2 D contiguous bytes each), are dropped into a wave-private LDS tile with the 16-byte chunks of
  // a row XOR-swizzled by the row, and come back in operand layout (lane = row).  The loads of
  // the next tile are in flight while the current one is scored.
  constexpr int RPL = 1024 / (2 * D);        // rows per 1 KB load
  constexpr int NL = 32 / RPL;               // loads per tile
  constexpr int CH = D / 8;                  // 16-byte chunks per row
  const unsigned char *kb = pv.k;
  const long long row_bytes = pv.row_bytes;
  auto swz = [](int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); };
  const long long last_byte_row = (long long)(pool - 1);
  u32x4 cur[NL], nxt[NL];
  auto fetch = [&](u32x4(&dst)[NL], int t0) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      long long row = (long long)c0 + t0 + RPL * i + lane / CH;
      row = row < last_byte_row ? row : last_byte_row;  // clamp: stays inside the pool
      dst[i] = __builtin_nontemporal_load((const u32x4 *)(kb + row * row_bytes + (lane % CH) * 16));  // read once
    }
  };
  unsigned char *tile = stage[wave];
  fetch(cur, wave * 32);
  for (int t0 = wave * 32; t0 < kChunkRows; t0 += 128) {
    if (t0 + 128 < kChunkRows) fetch(nxt, t0 + 128);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = RPL * i + lane / CH, c = lane % CH;
      *(u32x4 *)(tile + r * (2 * D) + ((c ^ swz(r)) << 4)) = cur[i];
    }
    bf16x8 K[NC];
#pragma unroll
    for (int kc = 0; kc < NC; ++kc)
      K[kc] = *(const bf16x8 *)(tile + col * (2 * D) + (((2 * kc + hi) ^ swz(col)) << 4));
    const int row = c0 + t0 + col;
    float best = -INFINITY;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      f32x16 S = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < NC; ++kc) S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[t][kc], K[kc], S, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) best = fmaxf(best, S[r]);
    }
    best = fmaxf(best, __shfl_xor(best, 32));  // the other 16 summaries of each tile
    if (hi == 0) sc[t0 + col] = (row >= lo && row < pool) ? best : -INFINITY;
#pragma unroll
    for (int i = 0; i < NL; ++i) cur[i] = nxt[i];
  }
  __syncthreads();
  // The chunk's best n_anchors rows, in order.  A thread holds E scores; only threads whose best row fewer than
  // n_anchors other threads' best rows beat can hold one of them, and their rows are ranked once more.
  // (Rounds of a wave-wide arg-max and a merge of the four waves' lists took 10.5 us of a 512-row
  // chunk's 21; the scan of four pools of 61K rows: 26.0 -> 19.6 us, of a 64K prompt: 85 -> 71.)
  constexpr int E = kChunkRows / 256;
  unsigned long long *const best_of = (unsigned long long *)&stage[0][0];  // [256], over the tiles
  unsigned long long *const left = best_of + 256;                         // [n_anchors][E]
  static_assert((256 + kMaxAnchors * E) * 8 <= 4 * 32 * 2 * D, "fits the tiles");
  unsigned long long key[E], top = 0ull;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    key[e] = row_key(sc[tid + 256 * e], c0 + tid + 256 * e);
    top = key[e] > top ? key[e] : top;
  }
  best_of[tid] = top;
  const int n_left = a.n_anchors * E;  // even: E is
  for (int i = tid; i < n_left; i += 256) left[i] = 0ull;
  __syncthreads();
  const int place = count_better(best_of, 256, top);
  if (top != 0ull && place < a.n_anchors) {
#pragma unroll
    for (int e = 0; e < E; ++e) left[place * E + e] = key[e];
  }
  __syncthreads();
  for (int i = tid; i < n_left; i += 256) {
    int rows;
    const unsigned long long mine = left[i];
    const int rank = count_better(left, n_left, mine, &rows);
    if (mine != 0ull && rank < a.n_anchors) cand[rank] = mine;
    if (i < a.n_anchors && i >= rows) cand[i] = 0ull;
  }
}

// ---- merge the candidates of all chunks, expand, pad, emit.  One workgroup per (b, PAST head); every step a
// constant number of passes over all anchors at once (a merge of the chunks' lists in n_anchors rounds and
// an expansion anchor by anchor on a sorted list of ranges took 15 us of 20; the kernel: 22.6 -> 10.8 us for 120 chunks a pool).
// 2^20 pool rows in chunks of 512: those are chosen by the longest pool with visible rows, and the grid covers
// the longest pool of all.
constexpr int kMaxChunks = 2048;

__global__ __launch_bounds__(256) void retrieve_select_kernel(const Problem p, const RetrieveArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned long long heads[kMaxChunks];  // best candidate of every chunk
  __shared__ __attribute__((aligned(16))) unsigned long long cand[kMaxAnchors * (kMaxAnchors + 1) / 2 + 2];
  __shared__ int src[kMaxAnchors], anchors[kMaxAnchors];
  __shared__ int q_lo[kMaxAnchors], q_len[kMaxAnchors];
  __shared__ int p_lo[2 * kMaxAnchors + 2], p_before[2 * kMaxAnchors + 2];
  __shared__ int n_found, n_pieces;
  const int b = blockIdx.x / p.n_past, np = blockIdx.x % p.n_past;
  const int kv = p.order[np];
  const PoolView pv = pool_view(p, a, b, kv);
  const int pool = pv.pool, lo = pv.lo;
  const int tid = threadIdx.x, n = a.n_anchors;
  const unsigned long long *lists = a.cand + ((long long)b * p.n_past + np) * a.n_chunks * kMaxAnchors;
  // Chunk lists are in order, so the n best candidates are among the first n - k of the chunk with the k-th
  // best head, k < n.
  const int n_heads = (a.n_chunks + 1) & ~1;
  for (int c = tid; c < n_heads; c += 256) heads[c] = c < a.n_chunks ? lists[(long long)c * kMaxAnchors] : 0ull;
  const int n_cand = (n * (n + 1) / 2 + 1) & ~1;
  for (int i = tid; i < n_cand; i += 256) cand[i] = 0ull;
  if (tid < n) src[tid] = -1;
  __syncthreads();
  for (int c = tid; c < a.n_chunks; c += 256) {
    const unsigned long long head = heads[c];
    const int k = count_better(heads, n_heads, head);
    if (head != 0ull && k < n) src[k] = c;
  }
  __syncthreads();
  for (int i = tid; i < n * n; i += 256) {
    const int k = i / n, e = i - k * n;
    if (e < n - k && src[k] >= 0) cand[k * n - k * (k - 1) / 2 + e] = lists[(long long)src[k] * kMaxAnchors + e];
  }
  __syncthreads();
  for (int i = tid; i < n_cand; i += 256) {
    int rows;
    const unsigned long long mine = cand[i];
    const int rank = count_better(cand, n_cand, mine, &rows);
    if (mine != 0ull && rank < n) anchors[rank] = key_row(mine);
    if (i == 0) n_found = rows < n ? rows : n;
  }
  __syncthreads();
  const int n_anch = n_found;
  const int visible = pool - lo;
  const int want = a.R < visible ? a.R : visible;
  if (tid < 64) {
    // Lane r: the anchor of rank r and its window, clipped to the visible pool.  Windows start and end in the
    // order of their anchors (they are equally long but for the clipping), so what better anchors have taken
    // of this one is a piece at its start (from anchors below) and one at its end (from anchors above):
    // the rows it adds are one range [from, to).
    const int lane = tid;
    const bool live = lane < n_anch;
    const int an = live ? anchors[lane] : 0;
    const int s = an - a.win_before > lo ? an - a.win_before : lo;
    const int e = an + a.win_after + 1 < pool ? an + a.win_after + 1 : pool;
    int from = s, to = e;
    for (int j = 0; j + 1 < n_anch; ++j) {
      const int aj = __builtin_amdgcn_readlane(an, j), sj = __builtin_amdgcn_readlane(s, j), ej = __builtin_amdgcn_readlane(e, j);
      if (j < lane) {
        if (aj < an) from = from > ej ? from : ej;
        else to = to < sj ? to : sj;
      }
    }
    auto prefix = [&](int x) {  // exclusive prefix sum over the lanes
      int incl = x;
#pragma unroll
      for (int sh = 1; sh < 64; sh <<= 1) {
        const int up = __shfl_up(incl, sh);
        if (lane >= sh) incl += up;
      }
      return incl - x;
    };
    const int adds = live && to > from ? to - from : 0;
    const int room = want - prefix(adds);  // rows still wanted when this anchor's turn comes
    const int take = room < 0 ? 0 : room < adds ? room : adds;
    // the ranges in row order
    const unsigned long long used = __builtin_amdgcn_ballot_w64(take > 0);
    const int k_used = (int)__builtin_popcountll(used);
    int pos = 0;
    for (int j = 0; j < n_anch; ++j) {
      const int fj = __builtin_amdgcn_readlane(from, j), tj = __builtin_amdgcn_readlane(take, j);
      pos += (tj > 0 && fj < from) ? 1 : 0;
    }
    if (take > 0) {
      q_lo[pos] = from;
      q_len[pos] = take;
    }
    // (one wave: LDS operations are in order)  padding: the earliest visible rows, i.e. the gaps in front of the
    // ranges from the first on; lane k_used has the gap behind the last range
    const int r_lo = lane < k_used ? q_lo[lane] : pool, r_len = lane < k_used ? q_len[lane] : 0;
    int prev_end = __shfl_up(r_lo + r_len, 1);
    if (lane == 0) prev_end = lo;
    const int gap = lane <= k_used ? r_lo - prev_end : 0;
    const int chosen = prefix(take) + take;  // lane 63: all rows the windows gave
    const int missing = want - __builtin_amdgcn_readlane(chosen, 63) - prefix(gap);
    const int pad = missing < 0 ? 0 : missing < gap ? missing : gap;
    const int before = prefix(pad + r_len);
    if (lane <= k_used) {
      p_lo[2 * lane] = prev_end;
      p_before[2 * lane] = before;
      p_lo[2 * lane + 1] = r_lo;
      p_before[2 * lane + 1] = before + pad;
    }
    if (lane == 0) n_pieces = 2 * k_used + 1;
  }
  __syncthreads();
  int *out = a.idx_out + ((long long)b * p.n_past + np) * a.R;
  for (int o = tid; o < a.R; o += 256) {
    int val = visible > 0 ? pool - 1 : 0;  // beyond the visible rows: refused on the host (an empty pool's list is not meaningful)
    if (o < want) {
      int l = 0, h = n_pieces;  // the last piece that starts at or before o
      while (h - l > 1) {
        const int mid = (l + h) >> 1;
        if (p_before[mid] <= o) l = mid;
        else h = mid;
      }
      val = p_lo[l] + (o - p_before[l]);
    }
    out[o] = val;
  }
}

hipError_t launch_retrieve(const Problem &p, const RetrieveArgs &a, hipStream_t st) {
  const int seqs = a.k_seq ? p.B * a.n_seg : p.B;  // whole-prompt form: one "sequence" per (b, segment)
  const dim3 heads(seqs * p.n_past);
  if (p.D == 128) hipLaunchKernelGGL(retrieve_summaries_kernel<128>, heads, dim3(256), 0, st, p, a);
  else hipLaunchKernelGGL(retrieve_summaries_kernel<64>, heads, dim3(256), 0, st, p, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid(a.n_chunks, seqs * p.n_past);
  const int nt = a.nsp / 32;
#define SEGATTN_SCORE(DD, NTT)                                                                            \
  do {                                                                                                    \
    if (a.chunk_rows == 512) hipLaunchKernelGGL((retrieve_score_kernel<DD, NTT, 512>), grid, dim3(256), 0, st, p, a); \
    else if (a.chunk_rows == 1024) hipLaunchKernelGGL((retrieve_score_kernel<DD, NTT, 1024>), grid, dim3(256), 0, st, p, a); \
    else hipLaunchKernelGGL((retrieve_score_kernel<DD, NTT, 4096>), grid, dim3(256), 0, st, p, a);         \
  } while (0)
  if (p.D == 128) {
    if (nt == 1) SEGATTN_SCORE(128, 1);
    else SEGATTN_SCORE(128, 2);
  } else {
    if (nt == 1) SEGATTN_SCORE(64, 1);
    else SEGATTN_SCORE(64, 2);
  }
#undef SEGATTN_SCORE
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(retrieve_select_kernel, heads, dim3(256), 0, st, p, a);
  return hipGetLastError();
}

}  // namespace segattn
