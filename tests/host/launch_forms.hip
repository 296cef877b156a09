// The form a call's launch takes, from the library's own rules (linked from libsegattn.so).  One call per input line,
// one answer per output line:
//   decode D Hq Hkv policy S T capacity resident closed,.. fill,..
//       -> "numbered" | "searched" (every window cut by itself) | "even", slices, numbers by the longest windows
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

static bool decode(const std::string &line) {
  std::istringstream head(line);
  std::string word, closed_text, fill_text;
  long long capacity, resident;
  for (int i = 0; i < 7; ++i) head >> word;
  head >> capacity >> resident >> closed_text >> fill_text;
  const std::vector<long long> closed = numbers(closed_text), fill = numbers(fill_text);
  std::istringstream in(line);
  in >> word;
  Call c;
  if (head.fail() || fill.size() != closed.size() || !read_call(in, (int)closed.size(), capacity, c)) return false;
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

int main() {
  for (std::string line; std::getline(std::cin, line);) {
    const std::string kind = line.substr(0, line.find(' '));
    if (!(kind == "decode" && decode(line))) {
      std::cout << "refused: " << line << '\n';
      return 1;
    }
  }
}
