// Symbolic replay of the level work item's groups, driven by the device table
// the kernel receives (leaf records, later records): for each p read from
// stdin it prints, per tree layout, the stages and the product formed, as a
// string over x0..x{p-1}.  Slots, ranks and stages are bounds-checked; every
// rank must be read once and no slot before its value's stage.
#include <cstdio>
#include <cstdlib>
#include <iostream>
#include <string>
#include <vector>

#include "plan.hpp"

using namespace dpar;
using S = std::string;

static S ap(const S& a, const S& b) { return "(" + a + "*" + b + ")"; }

static void need(bool ok, const char* what) {
  if (ok) return;
  std::printf("FAILED %s\n", what);
  std::exit(1);
}

static S product(const Tree& t, int p) {
  const GroupPlan g = make_groups(t);
  need(g.ok, "plan");
  const std::vector<uint32_t> tab = group_table(g);
  const size_t later = group_later_at(g.g1);
  need(later % 4 == 0 && tab.size() == later + (size_t)g.g2 * kGroupWords,
       "table size");
  std::vector<int> reads(p, 0);
  auto x = [&](uint32_t r) {
    need(r < (uint32_t)p, "rank");
    ++reads[r];
    return "x" + std::to_string(r);
  };
  std::vector<S> val(g.g1);
  std::vector<int> stage_of(g.g1, 0);  // -1: used up
  for (int i = 0; i < g.g1; ++i) {
    const uint32_t lo = tab[2 * i], shape = tab[2 * i + 1];
    const int n = (int)(shape >> 21);
    need(n >= 1 && n <= kGroupRanks, "leaf group size");
    std::vector<S> v(8);
    for (int h = 1; h < 8; ++h) {
      const uint32_t r = lo + ((shape >> 3 * (h - 1)) & 7u);
      need(r < (uint32_t)p, "leaf rank");  // unused positions are loaded too
      if (h <= n) v[h] = x(r);
    }
    if (n >= 5) v[2] = ap(v[5], v[2]);
    if (n >= 4) v[2] = ap(v[4], v[2]);
    if (n >= 7) v[3] = ap(v[7], v[3]);
    if (n >= 6) v[3] = ap(v[6], v[3]);
    if (n >= 3) v[1] = ap(v[3], v[1]);
    if (n >= 2) v[1] = ap(v[2], v[1]);
    val[i] = v[1];
  }
  int last = 1;
  for (int j = 0; j < g.g2; ++j) {
    const uint32_t* r = tab.data() + later + (size_t)j * kGroupWords;
    const int n = (int)(r[0] & 0xFFu), st = (int)(r[0] >> 8);
    need(n >= 1 && n <= kGroupRanks && st >= last && st < g.nst, "record");
    last = st;
    S w[16];
    for (int h = 1; h < 8; ++h) {
      need(r[h] < (uint32_t)p, "later rank");
      if (h <= n) w[h] = x(r[h]);
    }
    for (int c = n + 1; c <= 2 * n + 1; ++c) {
      const uint32_t s = (r[8 + (c - 2) / 2] >> 16 * (c & 1)) & 0xFFFFu;
      need(s < (uint32_t)g.g1, "slot");
      need(stage_of[s] >= 0 && stage_of[s] < st, "slot's stage");
      stage_of[s] = -1;
      w[c] = val[s];
    }
    for (int h = n; h >= 1; --h) w[h] = ap(w[2 * h], ap(w[2 * h + 1], w[h]));
    need(r[15] < (uint32_t)g.g1 && stage_of[r[15]] == -1, "own slot");
    val[r[15]] = w[1];
    stage_of[r[15]] = st;
  }
  need(stage_of[g.val_a] >= 0 && stage_of[g.val_b] >= 0, "roots");
  const S a = val[g.val_a];
  S b = val[g.val_b];
  if (g.extra >= 0) b = ap(b, x((uint32_t)g.extra));
  for (int i = 0; i < p; ++i) need(reads[i] == 1, "every rank once");
  return p >= 2 ? ap(a, b) : a;
}

int main() {
  int p;
  while (std::cin >> p) {
    std::printf("%d dual %s\n", p, product(build_tree(p), p).c_str());
    std::printf("%d single %s\n", p,
                product(kernel_single_tree(p), p).c_str());
  }
  return 0;
}
