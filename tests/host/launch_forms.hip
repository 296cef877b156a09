// The form a call's launch takes, from the library's own rules (linked from libsegattn.so).  One call per input line,
// one answer per output line:
//   decode D Hq Hkv policy S T capacity resident closed,.. fill,..
//       -> "numbered" | "searched" (every window cut by itself) | "even", slices, numbers by the longest windows
//   chunk D Hq Hkv policy S T capacity rows closed,.. fill,..
//       -> "keysplit" | "piped", waves of a workgroup, pieces of the PAST heads' prefixes at most, of the others'
//   prompt D Hq Hkv policy S T sequences rows
//       -> whole prompts of `rows` rows: "keysplit" | "piped", waves of a workgroup
//   window D Hq Hkv policy S T sequences rows packed
//       -> backward of `sequences` windows of `rows` rows (packed > 0: a batch of as many rows in all): "both" |
//          "split" | "items" (dQ), waves of the split dK/dV form (0: the other one; "both": 4), query heads of a dQ
//          workgroup, "packed" | "padded" (numbering of a packed batch's dQ items) | "dense"
// (policy: a digit per KV head; closed, fill: closed segments and open rows of each sequence).  Needs no GPU: the rules then
// take 256 compute units.
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "segattn_api.hip"  // build_problem, build_geom

struct Call {
  std::vector<uint8_t> policy;
  segattn_config cfg;
  Problem p;
  CacheGeom g;
};

static std::vector<long long> numbers(const std::string &text) {
  std::vector<long long> got;
  std::stringstream s(text);
  for (std::string x; std::getline(s, x, ',');) got.push_back(std::stoll(x));
  return got;
}

static bool read_call(std::istream &in, int batch, long long capacity, Call &c) {
  std::string policy;
  memset(&c.cfg, 0, sizeof(c.cfg));
  in >> c.cfg.head_dim >> c.cfg.n_q_heads >> c.cfg.n_kv_heads >> policy >> c.cfg.seg_len >> c.cfg.tail_len;
  for (char x : policy) c.policy.push_back((uint8_t)(x - '0'));
  c.cfg.batch = batch;
  c.cfg.past_capacity = capacity;
  c.cfg.kv_policy = c.policy.data();
  unsigned long long total;
  return !in.fail() && build_problem(&c.cfg, capacity > 0, c.p) && build_geom(&c.cfg, c.p, c.g, total);
}

// Rows before the new ones that head h of a sequence sees (all closed segments, or the carried tail; its open rows).
static long long before(const Problem &p, int h, long long closed, long long fill) {
  const long long past = closed * p.S;
  if (p.policy[h] & SEGATTN_PAST) return past + fill;
  return ((p.policy[h] & SEGATTN_TAIL) ? std::min<long long>(p.T, past) : 0) + fill;
}

// The fields behind the configuration: two numbers, then the closed segments and open rows of each sequence.
static bool read_sequences(const std::string &line, long long &capacity, long long &number, std::vector<long long> &closed,
                           std::vector<long long> &fill, Call &c) {
  std::istringstream head(line), in(line);
  std::string word, closed_text, fill_text;
  for (int i = 0; i < 7; ++i) head >> word;
  head >> capacity >> number >> closed_text >> fill_text;
  closed = numbers(closed_text);
  fill = numbers(fill_text);
  in >> word;
  return !head.fail() && fill.size() == closed.size() && read_call(in, (int)closed.size(), capacity, c);
}

static bool decode(const std::string &line) {
  long long capacity, resident;
  std::vector<long long> closed, fill;
  Call c;
  if (!read_sequences(line, capacity, resident, closed, fill, c)) return false;
  DecodeArgs a;
  memset(&a, 0, sizeof(a));
  a.geom = c.g;
  for (size_t b = 0; b < closed.size(); ++b)
    for (int h = 0; h < c.p.Hkv; ++h) {
      const long long win = before(c.p, h, closed[b], fill[b]) + 1, slices = (win + c.g.decode_chunk - 1) / c.g.decode_chunk;
      a.total_rows += win;
      a.chunks += slices;
      int &most = (c.p.policy[h] & SEGATTN_PAST) ? a.most_past : a.most_other;
      most = std::max<long long>(most, slices);
    }
  const DecodeSlices s = decode_slices(c.p, a, resident);
  std::cout << (s.numbered ? "numbered " : s.per_window ? "searched " : "even ") << a.chunks << ' '
            << c.p.B * ((long long)c.p.n_past * a.most_past + (long long)(c.p.Hkv - c.p.n_past) * a.most_other) << '\n';
  return true;
}

static bool chunk(const std::string &line) {
  long long capacity, rows;
  std::vector<long long> closed, fill;
  Call c;
  if (!read_sequences(line, capacity, rows, closed, fill, c)) return false;
  static unsigned char arena[1];  // not read by the rules
  PrefillArgs a;
  memset(&a, 0, sizeof(a));
  a.cache = arena;
  a.geom = c.g;
  a.n_rows = (int)rows;
  a.n_seg = 1;
  a.min_first_prefix = a.min_other_prefix = 1ll << 40;
  for (size_t b = 0; b < closed.size(); ++b)
    for (int h = 0; h < c.p.Hkv; ++h) {
      const bool past = c.p.policy[h] & SEGATTN_PAST;
      const long long n = before(c.p, h, closed[b], fill[b]);
      long long &most = past ? a.max_first_prefix : a.max_other_prefix, &least = past ? a.min_first_prefix : a.min_other_prefix;
      most = std::max(most, n);
      least = std::min(least, n);
    }
  const PrefillForm f = choose_prefill(c.p, a);
  const long long grid = c.p.B * c.p.Hkv * (c.p.g / f.hs) * ((rows * f.hs + 31) / 32);  // of the key-split form, nothing cut
  std::cout << (f.keysplit ? "keysplit " : "piped ") << (f.keysplit ? keysplit_waves(c.p, a, grid) : f.nw) << ' ' << (f.cut ? a.parts : 1) << ' '
            << (f.cut ? a.parts_other : 1) << '\n';
  return true;
}

static bool prompt(const std::string &line) {
  std::istringstream head(line), in(line);
  std::string word;
  int batch, rows;
  for (int i = 0; i < 7; ++i) head >> word;
  head >> batch >> rows;
  in >> word;
  Call c;
  if (head.fail() || !read_call(in, batch, 0, c)) return false;
  PrefillArgs a;
  memset(&a, 0, sizeof(a));
  a.n_rows = rows;
  a.n_seg = (rows + c.p.S - 1) / c.p.S;
  const PrefillForm f = choose_prefill(c.p, a);
  const int per_wg = 32 / f.hs, seg = std::min(rows, c.p.S);
  const long long grid = (long long)batch * c.p.Hkv * (c.p.g / f.hs) * a.n_seg * ((seg + per_wg - 1) / per_wg);
  std::cout << (f.keysplit ? "keysplit " : "piped ") << (f.keysplit ? keysplit_waves(c.p, a, grid) : f.nw) << '\n';
  return true;
}

static bool window(const std::string &line) {
  std::istringstream head(line), in(line);
  std::string word;
  int batch, rows;
  long long total;
  for (int i = 0; i < 7; ++i) head >> word;
  head >> batch >> rows >> total;
  in >> word;
  Call c;
  if (head.fail() || !read_call(in, batch, 0, c)) return false;
  static int offsets[1];  // not read by the rules
  BwdArgs a;
  memset(&a, 0, sizeof(a));
  a.n = rows;
  a.total = total;
  if (total > 0) a.cu_seqlens = offsets;
  const int hs = c.p.g % 4 == 0 ? 4 : c.p.g % 2 == 0 ? 2 : 1;
  const bool both = bwd_both_pays(c.p, a), split = !both && bwd_dq_split_pays(c.p, a);
  const int per_wg = split ? 32 / hs : 128 / hs, seg = std::min(rows, c.p.S);
  const bool packed = total > 0 && number_packed(c.p, total, (rows + c.p.S - 1) / c.p.S, (seg + per_wg - 1) / per_wg, per_wg);
  std::cout << (both ? "both 4 " : split ? "split " : "items ");
  if (!both) std::cout << bwd_dkv_split_waves(c.p, a) << ' ';
  std::cout << hs << (packed ? " packed" : total > 0 ? " padded" : " dense") << '\n';
  return true;
}

int main() {
  for (std::string line; std::getline(std::cin, line);) {
    const std::string kind = line.substr(0, line.find(' '));
    if (!(kind == "decode" && decode(line)) && !(kind == "chunk" && chunk(line)) &&
        !(kind == "prompt" && prompt(line)) && !(kind == "window" && window(line))) {
      std::cout << "refused: " << line << '\n';
      return 1;
    }
  }
}
