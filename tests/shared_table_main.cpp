// Walks the device table of shared-sum plans on the host: every trial's sample of every channel
// must be the delay table's, and every LDS and input position must lie inside its buffer.
#include <cmath>
#include <cstdio>
#include <random>
#include <set>
#include <vector>

#include "../paper_1401_8258_amd/csrc/dd_internal.h"

static int check(const dd_plan* p) {
  const std::vector<int32_t>& t = p->dev_table;
  const int nw = p->sh.nw, G = dd::kShG, n = G * nw;
  const int ints = dd::sh_stage_ints(nw), vc = dd::sh_row_chunks(p->dtype);
  if (nw < 1 || nw > dd::sh_max_waves(p->dtype)) return 1;
  if (p->sh.lds > dd::kLdsBytes || p->dms_per_group != n || p->ngroups != (p->ndm + n - 1) / n) return 2;
  for (int g = 0; g < p->ngroups; ++g) {
    const int64_t at = t[2 * (size_t)g], nst = t[2 * (size_t)g + 1];
    if (at < 2 * p->ngroups || nst < 1 || at + nst * ints > (int64_t)t.size()) return 3;
    std::set<int> seen;
    int64_t prev_lo = -1, prev_hi = -1;
    int open = 0;  // channels since the last fold
    for (int64_t s = 0; s < nst; ++s) {
      const int32_t* rec = &t[(size_t)(at + s * ints)];
      const int32_t* add = rec + dd::kShFormInts;
      const int nb = add[dd::kShAddInts - 1] >> 1, fold = add[dd::kShAddInts - 1] & 1;
      if (nb < 1 || nb > dd::kShMaxBundles || nb * G >= dd::kShAddInts) return 4;
      int64_t lo = 1 << 30, hi = 0;
      int rows = 0;
      for (int q = 0; q < nb; ++q) {
        auto head = [&](int i) { return rec[4 * (16 * q + i) + 3]; };
        const int m = head(0), slot = head(1), base = head(2);
        int code[dd::kShMaxPat + 1];
        int np = 0;
        for (int k = 0; k <= dd::kShMaxPat; ++k) code[k] = rec[4 * (16 * q + k)];
        while (np < dd::kShMaxPat && code[np] != 64 * dd::kShBlock) ++np;
        if (m < 1 || m > 4 || np < 1 || np > dd::kShMaxPat || slot % 16 || base % 16 || base < dd::kShSpare) return 5;
        if ((int64_t)base + (int64_t)np * slot > p->sh.lds) return 6;
        const int nrow = (slot / 16 + vc - 1) / vc;
        rows += nrow;
        const int ends = rec[4 * dd::kShLaneEnds + 3];
        if (rows > 250 || (q < 3 && ((ends >> (8 * q)) & 255) != rows)) return 7;
        lo = std::min<int64_t>(lo, base), hi = std::max<int64_t>(hi, (int64_t)base + (int64_t)np * slot);
        // raw samples a lane may load past the window start
        const int64_t reach = 4 * ((int64_t)(nrow - 1) * vc + 63) + 8 + (p->dtype == DD_U8 ? dd::kShWords : 0);
        if (reach > rec[4 * dd::kShLaneReach + 3] || reach > dd::ring_mirror(p)) return 8;
        for (int k = 0; k < np; ++k)
          if (code[k] < 0 || code[k] % dd::kShBlock || code[k] / dd::kShBlock > 63) return 9;
        if (code[np] != 64 * dd::kShBlock) return 9;
        for (int j = 0; j < 4; ++j) {
          const int off = rec[4 * (16 * q + j) + 1], ch = rec[4 * (16 * q + j) + 2];
          if (ch < 0 || ch >= p->nchan || off < 0 || off > p->maxdelay) return 10;
          if (j < m && !seen.insert(ch).second) return 11;
        }
        open += m;
        for (int w = 0; w < nw; ++w) {
          if (add[dd::kShAddInts * w + dd::kShAddInts - 1] != (nb << 1 | fold)) return 12;
          for (int k = 0; k < G; ++k) {
            const int d = std::min(g * n + w * G + k, p->ndm - 1);
            const int32_t o = add[dd::kShAddInts * w + G * q + k];
            const int32_t rel = (o & ~15) - base, e = o & 3;
            if ((o & 12) || rel < 0) return 13;
            const int pat = rel / slot, pos = rel % slot;
            if (pat >= np || pos + 16 * (3 * 63 + 63) + 16 > slot) return 14;
            for (int j = 0; j < m; ++j) {
              const int shift = j ? (code[pat] / dd::kShBlock >> (2 * (j - 1))) & 3 : 0;
              const int32_t delay = rec[4 * (16 * q + j) + 1] + shift + pos / 4 + e;
              if (delay != p->delays[(size_t)rec[4 * (16 * q + j) + 2] * p->ndm + d]) return 15;
            }
          }
        }
      }
      if (rows != rec[4 * dd::kShLaneRows + 3]) return 16;
      if (s > 0 && lo < prev_hi && prev_lo < hi) return 17;  // written while the stage before is read
      prev_lo = lo, prev_hi = hi;
      if (open > (p->dtype == DD_U8 ? 256 : dd::kShFold)) return 18;
      if (fold) open = 0;
      else if (s + 1 == nst) return 19;  // the last stage folds
    }
    if ((int)seen.size() != p->nchan) return 20;
  }
  return 0;
}

int main() {
  struct C {
    double top, bw, ts, step, dm0;
    int nchan, ndm;
  };
  std::vector<C> cs = {{428, 20, 51.2e-6, 0.1, 0, 1024, 2048}, {428, 20, 51.2e-6, 0.1, 0, 64, 128},
                       {428, 20, 51.2e-6, 0.1, 0, 1001, 901},  {428, 20, 51.2e-6, 0.2, 0, 256, 501},
                       {180, 60, 81.92e-6, 0.05, 0, 4096, 750}, {180, 60, 81.92e-6, 0.2, 100, 4096, 96},
                       {428, 20, 51.2e-6, 0.1, 0, 1, 1},       {428, 20, 51.2e-6, 5.0, 0, 37, 33},
                       {428, 20, 51.2e-6, 40.0, 0, 7, 12},     {428, 20, 8 * 51.2e-6, 0.1, 85, 512, 400}};
  int shared = 0;
  for (const C& c : cs)
    for (int order = 0; order < 3; ++order)
      for (int dt : {DD_F32, DD_F16, DD_U8}) {
        std::vector<double> f((size_t)c.nchan), dm((size_t)c.ndm);
        for (int i = 0; i < c.nchan; ++i) f[(size_t)i] = c.top - i * (c.bw / c.nchan);
        if (order == 1) std::reverse(f.begin(), f.end());
        if (order == 2) std::shuffle(f.begin(), f.end(), std::mt19937(7));
        for (int i = 0; i < c.ndm; ++i) dm[(size_t)i] = c.dm0 + c.step * i;
        dd_plan* p = nullptr;
        const int rc = dd_plan_create(&p, f.data(), c.nchan, c.ts, dm.data(), c.ndm, dt, nullptr);
        if (rc) continue;  // no form takes this spread
        if (p->sh.on) {
          ++shared;
          const int e = check(p);
          if (e) {
            std::printf("FAIL %d: nchan %d ndm %d step %g order %d dtype %d\n", e, c.nchan, c.ndm, c.step, order, dt);
            return 1;
          }
          if (order == 0)
            std::printf("nchan %d ndm %d step %g dtype %d: wavefronts %d groups %d lds %lld table %zu\n", c.nchan, c.ndm, c.step,
                        dt, p->sh.nw, p->ngroups, (long long)p->sh.lds, p->dev_table.size() * 4);
        }
        dd_plan_destroy(p);
      }
  std::printf("ok %d\n", shared);
  return shared ? 0 : 1;
}
