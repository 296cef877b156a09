// Host check of the item numbering of packed batches (packed_units, packed_block, packed_longest, packed_coords
// in segattn_work.h), the device functions run on the CPU by a wave of fibers:
//   * every row block of every sequence appears exactly once per (head, sub-group), the surplus numbers all
//     lie behind the end of a sequence;
//   * the heads listed first own the first items, longest first (up to 64 sequences);
//   * packed_block finds the sequence of a block in batches of one to 300,000 sequences;
//   * the launch rules count the blocks that there are (row_blocks).
// Prints "ok <batches> <items>" or the first failure.
#include "segattn_work.h"

using namespace segattn;

static long long batches = 0, items_checked = 0;

struct Batch {
  std::vector<int> len, cu;
  int S, rows;
  int per_seg() const { return (S + rows - 1) / rows; }
  // block number of a sequence -> is it there?
  bool has(int b, int seg, int blk) const {
    return blk * rows < S && (long long)seg * S + (long long)blk * rows < len[b];
  }
};

static Batch batch(std::vector<int> len, int S, int rows) {
  Batch x;
  x.S = S, x.rows = rows, x.cu = {0};
  for (int l : len) x.cu.push_back(x.cu.back() + l);
  x.len = std::move(len);
  return x;
}

static void fail(const char *what, const Batch &x, long long item) {
  printf("FAILED: %s, %d sequences, %d rows, S=%d, blocks of %d rows, at %lld\n", what, (int)x.len.size(), x.cu.back(), x.S, x.rows,
         item);
  exit(1);
}

static Problem problem(const Batch &x, int Hkv, int n_past, int g) {
  Problem p;
  memset(&p, 0, sizeof(p));
  p.B = (int)x.len.size(), p.Hkv = Hkv, p.g = g, p.Hq = Hkv * g, p.n_past = n_past, p.S = x.S;
  for (int i = 0; i < Hkv; ++i) p.order[i] = i;
  return p;
}

// all items of a launch
static void check(const Batch &x, int Hkv, int n_past, int g, int hw) {
  const Problem p = problem(x, Hkv, n_past, g);
  PrefillArgs a;
  memset(&a, 0, sizeof(a));
  a.cu_seqlens = x.cu.data();
  const int nhs = g / hw, units = (int)(packed_units(x.cu.back(), x.S, x.rows) + p.B), items = units * Hkv * nhs;
  std::vector<ItemCoords> got(items);
  emu::order = emu::Order::kByGroup;
  emu::launch(dim3(1), dim3(64), [&] {
    for (int i = 0; i < items; ++i) {
      const ItemCoords c = packed_coords(p, a, i, items, x.rows, hw);
      if (threadIdx.x == 0) got[i] = c;
    }
  });
  long long blocks = 0;
  int most = 0;  // blocks of the longest sequence
  for (int l : x.len) {
    const int n = l / x.S * x.per_seg() + (l % x.S + x.rows - 1) / x.rows;
    blocks += n;
    most = n > most ? n : most;
  }
  if (units < blocks || units > blocks + 2 * p.B) fail("number of units", x, units);
  std::vector<unsigned char> seen((size_t)p.B * most * Hkv * nhs, 0);
  long long valid = 0, last = 1ll << 40;
  for (int i = 0; i < items; ++i) {
    const ItemCoords c = got[i];
    if (c.b < 0 || c.b >= p.B || c.seg < 0 || c.qblk < 0 || c.hidx < 0 || c.hidx >= Hkv || c.hs < 0 || c.hs >= nhs || c.part != 0)
      fail("coordinate out of range", x, i);
    if ((c.hidx < n_past) != (i < units * n_past * nhs)) fail("heads listed first must own the first items", x, i);
    if (!x.has(c.b, c.seg, c.qblk)) continue;  // surplus
    ++valid;
    const long long n = (long long)c.seg * x.per_seg() + c.qblk;
    if (c.hidx < n_past && p.B <= 64) {
      if (n > last) fail("longest first", x, i);
      last = n;
    }
    unsigned char &s = seen[(((size_t)c.b * most + n) * Hkv + c.hidx) * nhs + c.hs];
    if (s) fail("an item twice", x, i);
    s = 1;
  }
  if (valid != blocks * Hkv * nhs) fail("items missing", x, valid);
  ++batches;
  items_checked += items;
}

// the search alone, at `probes` block numbers and at those around the sequences' starts
static void check_search(const Batch &x, int probes, std::mt19937 &rng) {
  const Problem p = problem(x, 1, 0, 1);
  const long long units = packed_units(x.cu.back(), x.S, x.rows) + p.B;
  std::vector<long long> u = {0, 1, units - 1};
  for (int i = 0; i < probes; ++i) {
    u.push_back(rng() % units);
    const int b = rng() % p.B;
    const long long at = packed_units(x.cu[b], x.S, x.rows) + b;
    for (long long d : {-1, 0, 1})
      if (at + d >= 0 && at + d < units) u.push_back(at + d);
  }
  emu::launch(dim3(1), dim3(64), [&] {
    for (long long i : u) {
      int b, seg, blk;
      packed_block(p, x.cu.data(), i, x.rows, b, seg, blk);
      if (threadIdx.x != 0) continue;
      int lo = 0, hi = p.B - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (packed_units(x.cu[mid], x.S, x.rows) + mid <= i) lo = mid;
        else hi = mid - 1;
      }
      const long long n = i - packed_units(x.cu[lo], x.S, x.rows) - lo;
      if (b != lo || seg != n / x.per_seg() || blk != n % x.per_seg()) fail("packed_block", x, i);
    }
  });
  ++batches;
  items_checked += (long long)u.size();
}

// the row blocks that the launch rules count are those that the launches number
static void check_counts(std::mt19937 &rng) {
  for (int S : {1, 31, 32, 33, 64, 100, 512})
    for (int rows : {8, 32, 128})
      for (int i = 0; i < 200; ++i) {
        std::vector<int> len(1 + rng() % 12, 1 + (int)(rng() % 1200));
        const bool same = i % 2;
        if (!same)
          for (int &l : len) l = (int)(rng() % 1200);
        const Batch x = batch(len, S, rows);
        const int longest = *std::max_element(len.begin(), len.end());
        if (longest == 0) continue;
        double padded = 0;
        for (long long s = 0; s < longest; s += S)
          padded += (double)len.size() * (double)(((longest - s < S ? longest - s : S) + rows - 1) / rows);
        const double units = (double)(packed_units(x.cu.back(), S, rows) + (long long)len.size());
        const Problem p = problem(x, 3, 1, 4);
        if (row_blocks(p, longest, 0, rows) != padded || row_blocks(p, longest, x.cu.back(), rows) != std::min(padded, units))
          fail("counted blocks", x, i);
      }
}

int main() {
  std::mt19937 rng(11);
  check_counts(rng);
  auto lens = [&](int n, int lo, int hi) {
    std::vector<int> l(n);
    for (int &v : l) v = lo + (int)(rng() % (hi - lo + 1));
    return l;
  };
  // S below, at, above and off a multiple of the block; empty sequences at either end and between
  for (int S : {1, 8, 33, 64, 100, 512}) {
    for (int rows : {8, 32, 64}) {
      check(batch({1}, S, rows), 3, 1, 4, 2);
      check(batch({0, 0, 130, 0, 64, 65, 0}, S, rows), 2, 1, 1, 1);
      check(batch(lens(13, 0, 90), S, rows), 1, 1, 1, 1);
    }
  }
  check(batch(lens(64, 0, 40), 32, 32), 2, 1, 1, 1);
  check(batch(lens(65, 0, 40), 32, 32), 2, 1, 2, 1);
  check(batch(lens(200, 0, 20), 100, 8), 2, 2, 1, 1);
  std::vector<int> front = lens(100, 1, 20);
  front[0] = 3000;
  check(batch(front, 256, 64), 2, 1, 1, 1);
  for (int B : {1, 2, 63, 64, 65, 127, 128, 129, 4095, 4096, 4097, 5000, 300000})
    for (int S : {7, 64, 500}) check_search(batch(lens(B, 0, 200), S, 32), 40, rng);
  check_search(batch(std::vector<int>(4200, 0), 64, 32), 40, rng);
  std::vector<int> gap(4200, 0);
  gap[2100] = 100000;
  check_search(batch(gap, 96, 64), 100, rng);
  printf("ok %lld %lld\n", batches, items_checked);
  return 0;
}
