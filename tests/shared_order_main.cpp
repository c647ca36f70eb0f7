// The FP32 additions of shared-sum plans, read from their device tables: each is counted with the
// channels that its result holds (its rounding error grows as that), and a series must carry no
// more of them than channel by channel in blocks of DD_CHAN_BLOCK, the order of the other forms.
#include <algorithm>
#include <cstdio>
#include <map>
#include <random>
#include <vector>

#include "../paper_1401_8258_amd/csrc/dd_internal.h"

struct Sum {
  double lin = 0, sq = 0;
  void add(int n) { lin += n, sq += (double)n * n; }
};

static Sum by_channel(int nchan) {
  Sum s;
  for (int b = 0; b < nchan; b += DD_CHAN_BLOCK) {
    const int e = std::min(nchan, b + DD_CHAN_BLOCK);
    for (int k = 2; k <= e - b; ++k) s.add(k);
    if (b) s.add(e);
  }
  return s;
}

static bool by_table(const dd_plan* p, int g, Sum* s) {
  const std::vector<int32_t>& t = p->dev_table;
  const int nw = p->sh.nw, ints = dd::sh_stage_ints(nw);
  const int64_t at = t[2 * (size_t)g], nst = t[2 * (size_t)g + 1];
  int total = 0, block = 0;
  for (int64_t st = 0; st < nst; ++st) {
    const int32_t* stage = &t[(size_t)(at + st * ints)];
    std::map<int, int> channels;  // of the bundle whose sums start at an LDS offset
    for (int w = 0; w < nw; ++w) {
      const int32_t* rec = stage + w * dd::kShRecInts + dd::kShAddInts;
      for (;;) {
        if (const int m = (rec[7] >> 8) & 7) channels[rec[5]] = m;
        if (!rec[11]) break;
        rec = &t[(size_t)(at + rec[11])];
      }
    }
    const int units = (stage[7] & 255) + 1;
    for (int u = 0; u < units; u += dd::kShG) {  // the first trial's
      auto it = channels.upper_bound(stage[u]);
      if (it == channels.begin()) return false;
      const int m = (--it)->second;
      for (int k = 2; k <= m; ++k) s->add(k);
      if (block) s->add(block + m);
      block += m;
    }
    if (stage[7] >> 8) {
      if (total) s->add(total + block);
      total += block;
      block = 0;
    }
  }
  return total == p->nchan && block == 0;
}

int main() {
  struct C {
    double top, bw, ts, step;
    int nchan, ndm, order;
  };
  const std::vector<C> cs = {{428, 20, 51.2e-6, 0.1, 1024, 2048, 0}, {428, 20, 51.2e-6, 0.1, 64, 128, 0},
                             {428, 20, 51.2e-6, 0.2, 128, 100, 0},   {428, 20, 51.2e-6, 0.1, 130, 33, 0},
                             {428, 20, 51.2e-6, 0.2, 256, 501, 0},   {428, 20, 51.2e-6, 6.0, 160, 9, 0},
                             {428, 20, 51.2e-6, 0.1, 515, 70, 2},    {180, 60, 51.2e-6, 0.1, 300, 64, 0},
                             {428, 20, 51.2e-6, 0.1, 1001, 200, 1},  {428, 20, 51.2e-6, 0.1, 33, 40, 0}};
  int shared = 0, bad = 0;
  for (const C& c : cs)
    for (int dt : {DD_F32, DD_F16}) {
      std::vector<double> f((size_t)c.nchan), dm((size_t)c.ndm);
      for (int i = 0; i < c.nchan; ++i) f[(size_t)i] = c.top - i * (c.bw / c.nchan);
      if (c.order == 1) std::reverse(f.begin(), f.end());
      if (c.order == 2) std::shuffle(f.begin(), f.end(), std::mt19937(7));
      for (int i = 0; i < c.ndm; ++i) dm[(size_t)i] = c.step * i;
      dd_plan* p = nullptr;
      if (dd_plan_create(&p, f.data(), c.nchan, c.ts, dm.data(), c.ndm, dt, nullptr)) continue;
      if (p->sh.on) {
        ++shared;
        const Sum old = by_channel(c.nchan);
        double lin = 0, sq = 0;
        for (int g = 0; g < p->ngroups; ++g) {
          Sum s;
          if (!by_table(p, g, &s)) return std::printf("FAIL: table of group %d\n", g), 1;
          lin = std::max(lin, s.lin / old.lin), sq = std::max(sq, s.sq / old.sq);
        }
        const bool ok = lin <= 1.0 && sq <= 1.0;
        bad += !ok;
        std::printf("%s: nchan %d ndm %d step %g order %d dtype %d: %.3f %.3f of the other forms'\n", ok ? "ok" : "FAIL",
                    c.nchan, c.ndm, c.step, c.order, dt, lin, sq);
      }
      dd_plan_destroy(p);
    }
  std::printf("%s %d\n", bad ? "failed" : "ok", shared);
  return bad || !shared ? 1 : 0;
}
