// Work decomposition shared by the prefill kernels of libsegattn: which workgroup handles
// which (sequence, KV head, head sub-group, segment, query block), and where its keys live.
//
// A workgroup's keys form two spans: span 0 = the prefix the head's policy grants (carried
// tail and/or past rows -- the whole pool or, in retrieval mode, the gathered rows of the
// head's attention view -- Eq. 13; every row visible to every query of the workgroup) and
// span 1 = the rows of the query's own segment (causal, Eq. 12's mask).
#pragma once
#include "segattn_internal.h"

namespace segattn {

// One workgroup's share of the problem.
struct WorkItem {
  const unsigned short *k0, *v0, *k1, *v1;  // first row of span 0 / span 1 for this KV head
  long long stride0, stride1;               // elements between consecutive rows
  int n0, n1;                               // rows in span 0; rows of the segment present
  const unsigned short *q;                  // row 0 of the segment's queries, head 0
  unsigned char *out;                       // row 0 of the segment's outputs, head 0
  float *lse;                               // lse of (b, head 0, segment row 0)
  long long lse_head_stride;                // floats between heads in lse
  int t0;                                   // first in-segment query row of the workgroup
  int kv, hsub, b;
  // Where the MFMA prefill kernel writes: rows of `out_heads` heads, this workgroup's first head
  // at `ohead0`, fp32 if `wide`.  Normally the caller's tensor; the workspace for a split prefix.
  int nq;                                   // query rows of the segment present (n1, except for a prefix piece)
  int out_heads, ohead0;
  bool wide;
  bool valid;
};

// Workgroup barrier for data handed over in LDS: waits for this wave's LDS accesses only.  __syncthreads()
// also waits for every global store of the wave to have been written, 1 to 2 us when the output of an
// item has just been stored.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ---- work items from queues (kernels that run as a resident grid)
// Queue y (counter at queue[kQueueStride * y]) holds the items y, y+8, ... of a launch of
// `n_items`, in order: what XCD y would be dealt if every item were a workgroup of its own.  A
// workgroup (on XCD blockIdx.x % 8) takes from its XCD's queue first; once that is empty, from the
// queue with the most items left (the XCD furthest behind); -1 when all are empty.  Thread 0 does
// the work, `slot` (shared memory) carries the answer to the others; two workgroup barriers.
// drawn / ticket: thread 0 may already hold a position drawn from the own queue (by atomicAdd,
// while the previous item was finishing), so that the round trip is over by now.
__device__ __forceinline__ int take_item(unsigned *queue, int n_items, bool drawn, unsigned ticket, int *slot) {
  if (threadIdx.x == 0) {
    auto items_of = [&](int y) { return y < n_items ? (unsigned)(n_items - y + 7) >> 3 : 0u; };
    const int x = (int)blockIdx.x & 7;
    int got = -1;
    const unsigned j0 = drawn ? ticket : atomicAdd(queue + kQueueStride * x, 1u);
    if (j0 < items_of(x)) {
      got = 8 * (int)j0 + x;
    } else {
      // Counters only grow, so a queue seen empty stays empty; a failed attempt marks its queue
      // empty: at most eight attempts.
      unsigned left[8];
#pragma unroll
      for (int y = 0; y < 8; ++y) {
        const unsigned at = __hip_atomic_load(queue + kQueueStride * y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        left[y] = at < items_of(y) ? items_of(y) - at : 0u;
      }
#pragma unroll 1
      for (int t = 0; t < 8 && got < 0; ++t) {
        unsigned most = 0;
        int y = -1;
#pragma unroll
        for (int z = 0; z < 8; ++z)
          if (left[z] > most) {
            most = left[z];
            y = z;
          }
        if (y < 0) break;
        const unsigned j = atomicAdd(queue + kQueueStride * y, 1u);
        if (j < items_of(y)) got = 8 * (int)j + y;
#pragma unroll
        for (int z = 0; z < 8; ++z)
          if (z == y) left[z] = 0;
      }
    }
    *slot = got;
  }
  lds_barrier();
  const int bid = __builtin_amdgcn_readfirstlane(*slot);
  lds_barrier();  // everyone has read it before thread 0 writes the next one
  return bid;
}

// A workgroup that got no item leaves; the last one of the launch puts the counters back to zero for
// the next launch on this stream, which starts only after this one has ended.  (Each workgroup
// counts itself after its own last access to the counters, so nobody uses them any more then.  A
// one-wave kernel in front of every queued launch did this before: a forward and a backward pass of
// 6.4K packed tokens, two queued launches, 183.3 -> 181.9 us without it.)
__device__ __forceinline__ void leave_queues(unsigned *queue) {
  if (threadIdx.x != 0) return;
  if (atomicAdd(queue + 8 * kQueueStride, 1u) + 1u == gridDim.x)
    for (int y = 0; y < 9; ++y)
      __hip_atomic_store(queue + kQueueStride * y, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Item index -> (segment, query block, head list position, sequence, head sub-group, prefix piece):
// all PAST items by descending absolute query block (longest work first), then the others grouped
// so that the query blocks sharing K/V rows run together on one XCD.  Pure integer arithmetic, the
// same on the host (where it is tested for being a one-to-one map) and on the device.
// total_items: items of the launch (PrefillArgs::grid_items, or the grid size).
struct ItemCoords {
  int seg, qblk, hidx, b, hs, part;
};
__host__ __device__ inline ItemCoords item_coords(const Problem &p, const PrefillArgs &a, int bid, int total_items,
                                                  int heads_per_wg) {
  const int nhs = p.g / heads_per_wg;
  const int nqb = a.q_blocks_per_seg;
  const int n_first = heads_listed_first(p, a);
  const int n_other = p.Hkv - n_first;
  const int parts = (a.cache != nullptr && a.parts > 1) ? a.parts : 1;
  const int parts_other = (a.cache != nullptr && a.parts_other > 1) ? a.parts_other : 1;
  const long long past_items = (long long)p.B * n_first * nhs * a.n_seg * nqb * parts;
  int seg, qblk, hidx, b, hs, part = 0;
  if (a.dv.ok) {
    // the same arithmetic as the branches below with the launch's divisors prepared by the host
    // (every quantity is below 2^31 then): a few scalar multiplies instead of a dozen divisions
    const ResolveDivs &dv = a.dv;
    if (bid < past_items) {
      const int row = fast_div(bid, dv.per);
      const int gq = a.n_seg * nqb - 1 - row;
      int rest = bid - row * (int)dv.per.d;
      if (a.cu_seqlens) rest = fast_mod(rest + row, dv.per);
      part = fast_mod(rest, dv.parts);
      rest = fast_div(rest, dv.parts);
      seg = fast_div(gq, dv.nqb);
      qblk = gq - seg * nqb;
      hs = fast_mod(rest, dv.nhs);
      rest = fast_div(rest, dv.nhs);
      b = fast_div(rest, dv.n_first);
      hidx = rest - b * (int)dv.n_first.d;
    } else {
      const int pi = (int)past_items;
      const int items = total_items - pi;
      const int x = bid & 7;
      int start = 0, first = 0;
#pragma unroll
      for (int xx = 0; xx < 8; ++xx) {
        const int o = (xx - pi) & 7;
        const int cnt = o < items ? (items - o + 7) >> 3 : 0;
        if (xx < x) start += cnt;
        if (xx == x) first = pi + o;
      }
      const int L = start + ((bid - first) >> 3);
      const int d = (int)dv.sub.d;
      const int sg = fast_div(L, dv.per_sub);
      const int grp = fast_div(sg, dv.sub);
      qblk = nqb - 1 - ((sg - grp * d) + d * (L - sg * (int)dv.per_sub.d));
      const long long shuffled = (long long)grp * (a.pair_stride > 0 ? a.pair_stride : 1);  // < 2^31 (host check)
      int rest = fast_mod((int)shuffled, dv.groups);
      if (parts_other > 1) {
        part = fast_mod(rest, dv.parts_other);
        rest = fast_div(rest, dv.parts_other);
      }
      hs = fast_mod(rest, dv.nhs);
      rest = fast_div(rest, dv.nhs);
      const int r2 = fast_div(rest, dv.n_other);
      hidx = n_first + (rest - r2 * (int)dv.n_other.d);
      seg = fast_div(r2, dv.batch);
      b = r2 - seg * (int)dv.batch.d;
    }
  } else if (bid < past_items) {
    const int per = p.B * n_first * nhs * parts;
    const int gq = a.n_seg * nqb - 1 - bid / per;
    int rest = bid % per;
    // Packed batch of unequal sequences: the workgroups of one query block index are `per` in a
    // row, and where `per` is a multiple of 8 a given (sequence, head) would meet the same XCD at
    // every index -- the long sequences' XCDs would work on while the others idle.  Rotate.
    if (a.cu_seqlens) rest = (rest + bid / per) % per;
    part = rest % parts;
    rest /= parts;
    seg = gq / nqb;
    qblk = gq % nqb;
    hs = rest % nhs;
    rest /= nhs;
    hidx = rest % n_first;
    b = rest / n_first;
  } else {
    // Heads without the PAST bit: the query blocks of one (sequence, head, segment) read the same
    // few MB of K/V, so they should run at the same time behind the same L2.  Workgroups go to the
    // 8 XCDs (one L2 each) round-robin by index: XCD x = bid % 8 takes the bids x, x+8, ... in
    // order.  Give each XCD a contiguous range of the list ordered by (segment, sequence, head,
    // head sub-group) and, inside one of those, by descending query block.
    const long long items = (long long)total_items - past_items;
    const int x = bid & 7;
    long long start = 0, first = 0;
#pragma unroll
    for (int xx = 0; xx < 8; ++xx) {
      const long long o = (xx - past_items) & 7;  // first list position served by XCD xx
      const long long cnt = o < items ? (items - o + 7) >> 3 : 0;
      if (xx < x) start += cnt;
      if (xx == x) first = past_items + o;
    }
    long long L = start + ((bid - first) >> 3);
    // Position L of the list -> (group, query block).  Every XCD takes its workgroups in index
    // order, so at equal speed the XCDs advance in step and the j-th blocks of all XCDs should
    // be equally long: that holds
    // if every XCD's range is a whole number of groups.  Where the group count is no multiple of 8
    // the launcher deals each group's blocks into d interleaved sub-groups (block q belongs to
    // sub-group (nqb-1-q) % d), each with the group's length profile, and the list runs over those.
    const int d = a.sub_groups > 1 ? a.sub_groups : 1;
    const int per_sub = nqb / d;
    const long long sg = L / per_sub;
    qblk = nqb - 1 - ((int)(sg % d) + d * (int)(L % per_sub));
    L = (sg / d) * nqb;  // first position of the group, for the group index below
    // Consecutive groups differ little in length for a dense batch but a lot for a ragged one (a
    // whole range of them can be empty): a multiplicative shuffle of the group index (stride
    // coprime to the group count, about an eighth of it) deals each XCD an even sample.
    const long long groups = items / nqb;
    int rest = (int)((L / nqb) * (a.pair_stride > 0 ? a.pair_stride : 1) % groups);
    part = rest % parts_other;
    rest /= parts_other;
    hs = rest % nhs;
    rest /= nhs;
    hidx = n_first + rest % n_other;
    rest /= n_other;
    b = rest % p.B;
    seg = rest / p.B;
  }
  return ItemCoords{seg, qblk, hidx, b, hs, part};
}

// Coordinates -> the item's key spans, query rows and outputs.
template <bool kPacked, bool kPieces>
__device__ inline WorkItem resolve_at(const Problem &p, const PrefillArgs &a, const ItemCoords &ic, int rows_per_wg,
                                      int heads_per_wg) {
  WorkItem w;
  const int seg = ic.seg, qblk = ic.qblk, hidx = ic.hidx, b = ic.b, hs = ic.hs, part = ic.part;
  const int kv = p.order[hidx];
  const int pol = p.policy[kv];
  w.kv = kv;
  w.hsub = hs;
  w.b = b;
  w.t0 = qblk * rows_per_wg;
  const long long kv_stride = (long long)p.Hkv * p.D;
  if (kPacked || a.cache == nullptr) {  // SEQ mode: prefix read from k/v by absolute position
    // dense batch: sequence b occupies rows [b*N, (b+1)*N); packed ragged batch: rows
    // [cu[b], cu[b+1]) and lse is [Hq, total rows]
    long long N = a.n_rows, base = (long long)b * N, lse_base = (long long)b * p.Hq * N, lse_stride = N;
    if (kPacked || a.cu_seqlens) {
      base = a.cu_seqlens[b];
      N = a.cu_seqlens[b + 1] - base;
      lse_base = base;
      lse_stride = a.total_rows;
    }
    const long long s = (long long)seg * p.S;
    const long long m_i = (N - s < p.S) ? (N - s) : p.S;  // <= 0 beyond the end of a short sequence
    long long lo = s;
    if (pol & SEGATTN_PAST) lo = 0;
    else if (pol & SEGATTN_TAIL) lo = (s - p.T > 0) ? s - p.T : 0;
    w.n0 = (int)(s - lo);
    w.n1 = (int)m_i;
    w.k0 = a.k + (base + lo) * kv_stride + (long long)kv * p.D;
    w.v0 = a.v + (base + lo) * kv_stride + (long long)kv * p.D;
    w.k1 = a.k + (base + s) * kv_stride + (long long)kv * p.D;
    w.v1 = a.v + (base + s) * kv_stride + (long long)kv * p.D;
    w.stride0 = w.stride1 = kv_stride;
    if (!kPacked && a.ret_k != nullptr && (pol & SEGATTN_PAST)) {
      // retrieved prefix of (b, segment, head): R dense gathered rows (none for the first segment)
      const long long slot = ((long long)b * a.n_seg + seg) * p.n_past + p.past_before[kv];
      w.n0 = seg > 0 ? a.ret_R : 0;
      w.k0 = a.ret_k + slot * a.ret_R * p.D;
      w.v0 = a.ret_v + slot * a.ret_R * p.D;
      w.stride0 = p.D;
    }
    w.q = a.q + (base + s) * p.Hq * p.D;
    const long long osz = p.out_fp32 ? 4 : 2;
    w.out = (unsigned char *)a.out + (base + s) * p.Hq * p.D * osz;
    w.lse = a.lse + lse_base + s;
    w.lse_head_stride = lse_stride;
  } else {  // CTX mode: prefix (and the committed part of the open segment) from the cache
    const int *meta = (const int *)(a.cache + a.geom.meta_off) + ((long long)b * p.Hkv + kv) * kMetaInts;
    int lo, seg_row0;
    window_of(p, a.geom, kv, meta, lo, seg_row0);
    const int hi = seg_row0 + meta[META_FILL];
    const long long m = a.n_rows;
    w.n0 = hi - lo;
    w.n1 = (int)m;
    w.k0 = (const unsigned short *)(a.cache + attn_k_off(p, a.geom, b, kv)) + (long long)lo * p.D;
    w.v0 = (const unsigned short *)(a.cache + attn_v_off(p, a.geom, b, kv)) + (long long)lo * p.D;
    w.stride0 = p.D;
    w.k1 = a.k + (long long)b * m * kv_stride + (long long)kv * p.D;
    w.v1 = a.v + (long long)b * m * kv_stride + (long long)kv * p.D;
    w.stride1 = kv_stride;
    w.q = a.q + (long long)b * m * p.Hq * p.D;
    const long long osz = p.out_fp32 ? 4 : 2;
    w.out = (unsigned char *)a.out + (long long)b * m * p.Hq * p.D * osz;
    w.lse = a.lse + (long long)b * p.Hq * m;
    w.lse_head_stride = m;
  }
  w.nq = w.n1;
  w.out_heads = p.Hq;
  w.ohead0 = kv * p.g + hs * heads_per_wg;
  w.wide = p.out_fp32 != 0;
  if (kPieces && a.piece_rows.d != 0) {  // (the stateful form only)
    const PrefillArgs::PieceList &pl = a.piece_list[hidx < a.piece_list[1].head0 ? 0 : 1];
    const int pieces = piece_count(w.n0, w.n1, a.piece_rows, pl.most);
    if (part >= pieces) {
      w.nq = 0;  // this head's prefix is shorter: no such piece
    } else if (pieces > 1) {
      const int start = part * (int)a.piece_rows.d;
      w.k0 += (long long)start * p.D;
      w.v0 += (long long)start * p.D;
      w.n0 = (part == pieces - 1) ? w.n0 - start : (int)a.piece_rows.d;
      if (part != pieces - 1) w.n1 = 0;
      const long long slot = (long long)(b * pl.most + part) * a.n_rows * pl.heads;
      w.out = (unsigned char *)(pl.out + slot * p.D);
      w.lse = pl.lse + slot;
      w.lse_head_stride = a.n_rows;
      w.out_heads = pl.heads;
      w.ohead0 = (hidx - pl.head0) * p.g + hs * heads_per_wg;
      w.wide = true;
    }
  }
  w.valid = w.t0 < w.nq;
  return w;
}

// Number u of a packed batch's row blocks (packed_units) -> sequence, segment and block.  Every wave
// works it out by itself: a lane per sequence, then a count of the sequences that start at or before u; more
// than 64 sequences are looked at from afar first, every lane at the first one of a 64th of them.  One
// memory round trip per 64-fold (walking the batch 64 sequences at a time: 4096 sequences of 20 to 300 rows,
// 32/8 heads of 128, forward: 7481 -> 5053 us; 1024 sequences 1369 -> 1244).
__device__ inline void packed_block(const Problem &p, const int *cu_seqlens, long long u, int rows_per_block, int &b,
                                    int &seg, int &qblk) {
  const int lane = threadIdx.x & 63;
  int first = 0, n = p.B;  // the sequence is one of first .. first + n - 1
  for (;;) {
    const int step = (n + 63) >> 6, at = lane * step;
    const int i = at < n ? first + at : first;
    const bool starts = at < n && packed_units(cu_seqlens[i], p.S, rows_per_block) + i <= u;
    const int count = __builtin_popcountll(__builtin_amdgcn_ballot_w64(starts));
    const int skip = count > 0 ? (count - 1) * step : 0;
    first += skip;
    n = n - skip < step ? n - skip : step;
    if (step == 1) break;
  }
  b = first;
  int v = (int)(u - packed_units(cu_seqlens[b], p.S, rows_per_block)) - b;
  if (v < 0) v = 0x3fffffff / p.S;  // cu_seqlens[0] was not 0: a block behind every sequence's end
  const int per_seg = (p.S + rows_per_block - 1) / rows_per_block;
  seg = v / per_seg;
  qblk = v - seg * per_seg;
}

__device__ inline int wave_max_i32(int x) {
  auto step = [&](int y) { x = x > y ? x : y; };
  step(__builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true));
  step(__builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true));
  step(__builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true));
  step(__builtin_amdgcn_mov_dpp(x, 0x140, 0xF, 0xF, true));
  const int a = __builtin_amdgcn_readlane(x, 0), b = __builtin_amdgcn_readlane(x, 16);
  const int c = __builtin_amdgcn_readlane(x, 32), d = __builtin_amdgcn_readlane(x, 48);
  const int ab = a > b ? a : b, cd = c > d ? c : d;
  return ab > cd ? ab : cd;
}
__device__ inline int wave_sum_i32(int x) {  // over the 64 lanes: DPP inside the rows of 16, then four lanes
  x += __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);
  x += __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);
  x += __builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true);
  x += __builtin_amdgcn_mov_dpp(x, 0x140, 0xF, 0xF, true);
  return (__builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16)) +
         (__builtin_amdgcn_readlane(x, 32) + __builtin_amdgcn_readlane(x, 48));
}
// The u-th row block of a packed batch of at most 64 sequences in the order of descending block index
// (longest key range first for heads that see the whole past): false if there are no more than u.
// A lane per sequence; the block index q is found by bisection, with the number of blocks at or
// beyond q as a sum over the lanes: a step per bit of the longest sequence's block count.
__device__ inline bool packed_longest(const Problem &p, const int *cu_seqlens, int u, int rows_per_block, int &b, int &seg,
                                      int &qblk) {
  const int lane = threadIdx.x & 63;
  const int per_seg = (p.S + rows_per_block - 1) / rows_per_block;
  int blocks = 0;
  if (lane < p.B) {
    const int len = cu_seqlens[lane + 1] - cu_seqlens[lane];
    blocks = len > 0 ? len / p.S * per_seg + (len % p.S + rows_per_block - 1) / rows_per_block : 0;
  }
  const int all = wave_sum_i32(blocks);
  if (u >= all) return false;
  int lo = 0, hi = wave_max_i32(blocks), at_hi = 0;  // more than u blocks at or beyond lo, at_hi <= u at or beyond hi
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    const int n = wave_sum_i32(blocks > mid ? blocks - mid : 0);
    if (n > u) {
      lo = mid;
    } else {
      hi = mid;
      at_hi = n;
    }
  }
  // block lo of the (u - at_hi)-th sequence that has one
  const unsigned long long have = __builtin_amdgcn_ballot_w64(blocks > lo);
  const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(have >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)have, 0u));
  b = (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(blocks > lo && rank == u - at_hi));
  seg = lo / per_seg;
  qblk = lo - seg * per_seg;
  return true;
}

// Item index -> coordinates for a packed batch: only the row blocks there are (and at most one per
// sequence that is not), instead of a grid of every sequence padded to the longest -- of eight
// sequences of 65 to 9001 tokens two thirds of that grid's items were empty, and each cost its
// workgroup a turn at the queue.  Items: units x heads x sub-groups, the PAST heads first, longest
// first (up to 64 sequences; beyond that in the order of the batch), then the others: like in
// item_coords an XCD takes a contiguous range of the list ordered by head and row block, from the
// last block on.
__device__ inline ItemCoords packed_coords(const Problem &p, const PrefillArgs &a, int bid, int total_items, int rows_per_wg,
                                           int heads_per_wg) {
  const int nhs = p.g / heads_per_wg, n_first = heads_listed_first(p, a);
  const int units = total_items / (p.Hkv * nhs);
  const int pi = units * n_first * nhs;
  ItemCoords ic;
  ic.part = 0;
  if (bid < pi) {
    const int per = n_first * nhs, u = bid / per, rest = bid - u * per;
    ic.hidx = rest / nhs;
    ic.hs = rest - ic.hidx * nhs;
    if (p.B > 64) {
      packed_block(p, a.cu_seqlens, units - 1 - u, rows_per_wg, ic.b, ic.seg, ic.qblk);
    } else if (!packed_longest(p, a.cu_seqlens, u, rows_per_wg, ic.b, ic.seg, ic.qblk)) {
      ic.b = ic.qblk = 0;
      ic.seg = 0x3fffffff / p.S;  // behind the end of any sequence
    }
  } else {
    const int items = total_items - pi, x = bid & 7;
    int start = 0, first = 0;
#pragma unroll
    for (int xx = 0; xx < 8; ++xx) {
      const int o = (xx - pi) & 7;  // first list position served by XCD xx
      const int cnt = o < items ? (items - o + 7) >> 3 : 0;
      if (xx < x) start += cnt;
      if (xx == x) first = pi + o;
    }
    const int L = start + ((bid - first) >> 3), h = L / units;
    ic.hidx = n_first + h / nhs;
    ic.hs = h % nhs;
    packed_block(p, a.cu_seqlens, units - 1 - (L - h * units), rows_per_wg, ic.b, ic.seg, ic.qblk);
  }
  ic.b = __builtin_amdgcn_readfirstlane(ic.b);  // the same in every lane: keep what follows from them in scalar registers
  ic.seg = __builtin_amdgcn_readfirstlane(ic.seg);
  ic.qblk = __builtin_amdgcn_readfirstlane(ic.qblk);
  return ic;
}

// blockIdx -> work item.  kPacked: the launch has PrefillArgs::packed set; kPieces: it may cut prefixes.  Fixed per
// instantiation, since a kernel that can do everything is slower at each (code and argument words a short
// launch waits for; key-split form, 300 rows, 32/8 heads of 64: 9.7 us with all of it, 8.3 with its own;
// general form, 500 rows: 14.6 and 14.3).
template <bool kPacked, bool kPieces>
__device__ inline WorkItem resolve(const Problem &p, const PrefillArgs &a, int bid, int rows_per_wg,
                                   int heads_per_wg) {
  const int items = a.grid_items > 0 ? a.grid_items : (int)gridDim.x;
  const ItemCoords ic = kPacked ? packed_coords(p, a, bid, items, rows_per_wg, heads_per_wg)
                                : item_coords(p, a, bid, items, heads_per_wg);
  return resolve_at<kPacked, kPieces>(p, a, ic, rows_per_wg, heads_per_wg);
}

__device__ inline int uniform_i32(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline long long uniform_i64(long long x) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(unsigned long long)x);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((unsigned long long)x >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}
template <typename T>
__device__ inline T *uniform_ptr(T *ptr) {
  const unsigned long long u = (unsigned long long)ptr;
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
  return (T *)(((unsigned long long)hi << 32) | lo);
}
// Everything in a work item is the same for the whole workgroup, but some of it comes from memory
// (sequence offsets, cache counters) through vector loads.  Pin the sizes and the K/V pointers to
// scalar registers so that loader pointers and loop bounds derived from them stay out of the
// vector file.
__device__ inline void pin_uniform(WorkItem &w) {
  w.n0 = uniform_i32(w.n0);
  w.n1 = uniform_i32(w.n1);
  w.nq = uniform_i32(w.nq);
  w.t0 = uniform_i32(w.t0);
  w.stride0 = uniform_i32((int)w.stride0);
  w.stride1 = uniform_i32((int)w.stride1);
  w.k0 = uniform_ptr(w.k0);
  w.v0 = uniform_ptr(w.v0);
  w.k1 = uniform_ptr(w.k1);
  w.v1 = uniform_ptr(w.v1);
}

__device__ inline float bf16_bits_to_f32(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

}  // namespace segattn
