// The tables of the steps of subband plans (FP32, few channels, workgroups of 8 and 4 wavefronts):
// walked as those of whole beams are.
#define main whole_beams
#include "shared_table_main.cpp"
#undef main

int main() {
  struct C {
    int nchan, first, n, ndm;
    double step;
  };
  // subbands [first, first + n) of nchan channels at nominal DMs, and groups of trials over subbands
  const std::vector<C> cs = {{1024, 0, 32, 60, 1.6},  {1024, 992, 32, 60, 1.6}, {1024, 512, 16, 60, 1.6}, {512, 480, 32, 25, 4.8},
                             {96, 88, 8, 2, 3.2},     {130, 128, 2, 5, 1.6},    {33, 32, 1, 2, 0.4},      {32, 0, 32, 16, 0.1},
                             {64, 0, 64, 33, 0.1},    {1024, 768, 64, 48, 2.0}, {512, 384, 120, 7, 2.0},  {32, 0, 32, 3, 0.1}};
  std::set<int> seen;
  int shared = 0;
  for (const C& c : cs) {
    std::vector<double> f((size_t)c.n), dm((size_t)c.ndm);
    for (int i = 0; i < c.n; ++i) f[(size_t)i] = 428.0 - (c.first + i) * (20.0 / c.nchan);
    for (int i = 0; i < c.ndm; ++i) dm[(size_t)i] = c.step * i;
    dd_plan* p = nullptr;
    if (dd::plan_create(&p, f.data(), c.n, 51.2e-6, dm.data(), c.ndm, DD_F32, nullptr, dd::kLdsBytes, true)) continue;
    if (p->sh.on) {
      ++shared;
      seen.insert(p->sh.nw);
      const int e = check(p);
      if (e) {
        std::printf("FAIL %d: channels %d + %d of %d, %d trials of %g\n", e, c.first, c.n, c.nchan, c.ndm, c.step);
        return 1;
      }
    }
    dd_plan_destroy(p);
  }
  std::printf("ok %d of %zu, workgroups of", shared, cs.size());
  for (int w : seen) std::printf(" %d", w);
  std::printf("\n");
  return seen.count(4) && seen.count(8) ? 0 : 1;
}
