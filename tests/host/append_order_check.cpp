// Host check of the append kernel that also counts its rows (CopyArgs::counts): whatever order the waves of
// its workgroups run in, the rows lie where a commit has to leave them and the counters say so.  The kernels
// are those of segattn_cache.hip, run on the CPU; the workgroups of a head share its counters, and the last one
// to arrive rewrites what all the others had to read first.
// Prints "ok <launches>" or the first difference.
#include "../../paper_2605_11744_amd/csrc/segattn_cache.hip"

hipError_t hipGetLastError() { return hipSuccess; }

using namespace segattn;

static int launches = 0;

static void fail(const char *what, int order, int D, int S, int T, int fill, int m, int ret, int b, int h, int row) {
  printf("FAILED: %s, order %d, D=%d S=%d T=%d fill=%d m=%d retrieved=%d, sequence %d head %d row %d\n", what, order, D, S, T, fill,
         m, ret, b, h, row);
  exit(1);
}

static void check(emu::Order order, int D, int S, int T, int fill, int m, int ret_cap) {
  constexpr int B = 2, H = 3;
  const int policy[H] = {SEGATTN_PAST, SEGATTN_TAIL, ret_cap ? SEGATTN_PAST : SEGATTN_TAIL | SEGATTN_PAST};
  const int closed[B] = {2 * S, S};
  Problem p;
  memset(&p, 0, sizeof(p));
  p.B = B, p.Hkv = p.Hq = H, p.g = 1, p.D = D, p.S = S, p.T = T;
  for (int h = 0; h < H; ++h) {
    p.policy[h] = policy[h];
    p.past_before[h] = p.n_past;
    p.n_past += (policy[h] & SEGATTN_PAST) ? 1 : 0;
  }
  CacheGeom g;
  memset(&g, 0, sizeof(g));
  g.pool_cap = 4 * S;
  g.ret_cap = ret_cap;
  g.rows_per_seq = p.n_past * g.pool_cap + (H - p.n_past) * (unsigned long long)(T + S);
  g.kv_off = 1024;
  g.view_off = g.kv_off + B * g.rows_per_seq * 2 * D * 2;
  const size_t bytes = g.view_off + (ret_cap ? (size_t)B * p.n_past * 2 * (ret_cap + S) * D * 2 : 0);
  std::vector<uint4> arena_mem(bytes / 16);
  unsigned char *const arena = (unsigned char *)arena_mem.data();
  memset(arena, 0, bytes);
  int *const meta = (int *)arena;
  for (int b = 0; b < B; ++b)
    for (int h = 0; h < H; ++h) {
      int *x = meta + (b * H + h) * kMetaInts;
      x[META_POOL] = (policy[h] & SEGATTN_PAST) ? closed[b] : 0;
      x[META_TAIL] = T;
      x[META_FILL] = fill;
      x[META_RET] = ret_cap;
    }
  std::vector<uint4> k_mem((size_t)B * m * H * D / 8), v_mem(k_mem.size());
  unsigned short *const k = (unsigned short *)k_mem.data(), *const v = (unsigned short *)v_mem.data();
  for (size_t i = 0; i < k_mem.size() * 8; ++i) {
    k[i] = (unsigned short)(1 + i * 7 % 65521);
    v[i] = (unsigned short)(1 + i * 11 % 65519);
  }
  CopyArgs a;
  memset(&a, 0, sizeof(a));
  a.k = k, a.v = v, a.cache = arena, a.geom = g, a.m = m, a.counts = 1;
  emu::order = order;
  if (launch_cache_append(p, a, nullptr) != hipSuccess) fail("launch", (int)order, D, S, T, fill, m, ret_cap, 0, 0, 0);
  ++launches;

  const bool closes = fill + m == S;
  for (int b = 0; b < B; ++b)
    for (int h = 0; h < H; ++h) {
      const bool past = policy[h] & SEGATTN_PAST;
      auto bad = [&](const char *what, int row) { fail(what, (int)order, D, S, T, fill, m, ret_cap, b, h, row); };
      const int *x = meta + (b * H + h) * kMetaInts;
      if (x[META_FILL] != (closes ? 0 : fill + m)) bad("fill", x[META_FILL]);
      if (x[META_POOL] != (past ? closed[b] + (closes ? S : 0) : 0)) bad("pool", x[META_POOL]);
      if (x[META_TAIL] != T || x[META_RET] != (closes ? 0 : ret_cap) || x[META_ARRIVED] != 0) bad("counters", 0);
      // every row of the head's block: the new ones where they belong, the others untouched
      const int skip = !past && closes ? S - T : 0, first = past ? closed[b] + fill : closes ? 0 : T + fill;
      auto rows = [&](unsigned long long k_off, unsigned long long v_off, int cap, int at) {
        for (int r = 0; r < cap; ++r) {
          const int s = r - at + skip;  // the source row that belongs here
          const bool is_new = r >= at && s < m;
          const unsigned short *want_k = k + (((size_t)b * m + (is_new ? s : 0)) * H + h) * D, *want_v = v + (want_k - k);
          const unsigned short *has_k = (const unsigned short *)(arena + k_off) + (size_t)r * D;
          const unsigned short *has_v = (const unsigned short *)(arena + v_off) + (size_t)r * D;
          for (int d = 0; d < D; ++d)
            if (has_k[d] != (is_new ? want_k[d] : 0) || has_v[d] != (is_new ? want_v[d] : 0)) bad("row", r);
        }
      };
      rows(k_block_off(p, g, b, h), v_block_off(p, g, b, h), (int)head_cap(p, g, h), first);
      if (uses_view(p, g, h)) rows(view_k_off(p, g, b, h), view_v_off(p, g, b, h), ret_cap + S, ret_cap + fill);
    }
}

int main() {
  using emu::Order;
  for (int D : {64, 128})
    for (Order o : {Order::kByGroup, Order::kLeadersFirst, Order::kLeadersLast, Order::kRandom, Order::kRandom, Order::kRandom})
      for (int ret : {0, 32}) {
        check(o, D, 1024, 128, 0, 1, ret);      // one workgroup a head, one row
        check(o, D, 1024, 128, 37, 128, ret);   // one (D = 128) or half of one
        check(o, D, 1024, 128, 611, 173, ret);  // two
        check(o, D, 1024, 1024, 100, 300, ret);
        check(o, D, 1024, 0, 3, 512, ret);      // two or four
        check(o, D, 200, 64, 0, 200, ret);      // a whole segment
        check(o, D, 512, 512, 0, 512, ret);
        check(o, D, 512, 0, 0, 512, ret);
      }
  printf("ok %d\n", launches);
  return 0;
}
