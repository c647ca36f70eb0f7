// Walks the device table of shared-sum plans on the host: every trial's sample of every channel
// must be the delay table's, and every LDS and input position must lie inside its buffer.
#include <cmath>
#include <cstdio>
#include <map>
#include <random>
#include <set>
#include <vector>

#include "../paper_1401_8258_amd/csrc/dd_internal.h"

struct Form {  // one bundle's patterns of a stage, by LDS offset
  int m, slot, chan[4], off[4], shift[4];
  std::set<int> rows;
};

static int check(const dd_plan* p) {
  const std::vector<int32_t>& t = p->dev_table;
  const int nw = p->sh.nw, G = dd::kShG, n = G * nw;
  const int ints = dd::sh_stage_ints(nw), vc = dd::sh_row_chunks(p->dtype);
  if (nw < 1 || nw > dd::kShWaves) return 1;
  if (p->sh.lds > dd::kLdsBytes || p->dms_per_group != n || p->ngroups != (p->ndm + n - 1) / n) return 2;
  for (int g = 0; g < p->ngroups; ++g) {
    const int64_t at = t[2 * (size_t)g], nst = t[2 * (size_t)g + 1];
    const int64_t end = g + 1 < p->ngroups ? t[2 * (size_t)g + 2] : (int64_t)t.size();
    if (at < 2 * p->ngroups || nst < 1 || at - ints < 2 * p->ngroups || at + (nst + dd::kShPad) * ints > end || end > (int64_t)t.size()) return 3;
    std::set<int> seen;
    int64_t prev_lo = -1, prev_hi = -1;
    int open = 0;  // channels since the last fold
    for (int64_t s = 0; s < nst; ++s) {
      const int32_t* st = &t[(size_t)(at + s * ints)];
      std::map<int, Form> forms;  // by LDS offset
      int64_t lo = 1 << 30, hi = 0;
      for (int w = 0; w < nw; ++w) {
        const int32_t* rec = st + w * dd::kShRecInts + dd::kShAddInts;
        for (int rounds = 0;; ++rounds) {
          if (rounds > 1000) return 4;
          const int m = (rec[7] >> 8) & 7, row = rec[7] & 255, step = rec[7] & 4096 ? -1 : 1;
          const uint8_t* code = reinterpret_cast<const uint8_t*>(rec + 8);
          if (m > 4) return 5;
          if (m == 0 && (code[0] != 64 || rec[11] || rounds)) return 6;
          if (m && code[0] == 64) return 6;
          for (int k = 0; m && code[k] != 64; ++k) {
            if (k >= dd::kShRecPat || code[k] > 63) return 7;
            const int dst = rec[5] + k * rec[6];
            Form f{m, rec[6], {}, {}, {}, {}};
            for (int j = 0; j < m; ++j) {
              f.chan[j] = rec[4] + j * step;
              f.off[j] = rec[0] + (j ? rec[j] / (int)dd::elem_bytes(p->dtype) : 0);
              if (f.off[j] - rec[0] + dd::sh_reach(p->dtype, row) > rec[10]) return 8;
              f.shift[j] = j ? (code[k] >> (2 * (j - 1))) & 3 : 0;
              if (f.chan[j] < 0 || f.chan[j] >= p->nchan || f.off[j] < 0 || f.off[j] > p->maxdelay) return 8;
            }
            if (rec[6] % 16 || rec[5] % 16 || rec[5] < dd::kShSpare || dst + rec[6] > p->sh.lds) return 9;
            auto it = forms.insert({dst, f}).first;
            if (it->second.chan[0] != f.chan[0] || it->second.m != m || it->second.slot != f.slot) return 10;
            if (!it->second.rows.insert(row).second) return 11;
            lo = std::min<int64_t>(lo, dst), hi = std::max<int64_t>(hi, (int64_t)dst + rec[6]);
          }
          // raw samples a lane may load past the window start
          const int64_t reach = 4 * ((int64_t)row * vc + 63) + 8 + (p->dtype == DD_U8 ? dd::kShWords : 0);
          if (m && (reach > dd::sh_reach(p->dtype, row) || rec[10] > dd::ring_mirror(p))) return 12;
          if (!rec[11]) break;
          if (rec[11] < nst * ints || at + rec[11] + dd::kShFormInts > end) return 13;
          rec = &t[(size_t)(at + rec[11])];
        }
      }
      int64_t past = 0;  // the sums of a stage do not overlap and their rows cover their windows
      for (const auto& kv : forms) {
        if (kv.first < past) return 14;
        past = (int64_t)kv.first + kv.second.slot;
        if ((int)kv.second.rows.size() != (kv.second.slot / 16 + vc - 1) / vc) return 15;
        if (*kv.second.rows.rbegin() + 1 != (int)kv.second.rows.size()) return 15;
      }
      const int units = (st[7] & 255) + 1, fold = st[7] >> 8;
      if (units % G || units > G * dd::kShMaxBundles) return 16;
      for (int w = 0; w < nw; ++w) {
        const int32_t* add = st + w * dd::kShRecInts;
        if (add[7] != st[7]) return 17;
        for (int u = 0; u < units; ++u) {
          const int d = std::min(g * n + w * G + u % G, p->ndm - 1);
          auto it = forms.upper_bound(add[u]);
          if (add[u] & 15 || it == forms.begin()) return 18;
          --it;
          const Form& f = it->second;
          const int pos = add[u] - it->first;
          if (pos + 16 * (3 * 63 + 63) + 16 > f.slot) return 19;
          for (int j = 0; j < f.m; ++j) {
            const int32_t delay = f.off[j] + f.shift[j] + pos / 4 + ((add[6] >> (2 * u)) & 3);
            if (delay != p->delays[(size_t)f.chan[j] * p->ndm + d]) return 20;
            // every trial takes every channel of the stage once
            if (w == 0 && u % G == 0 && !seen.insert(f.chan[j]).second) return 21;
          }
          if (w == 0 && u % G == 0) open += f.m;
        }
      }
      if (s > 0 && lo < prev_hi && prev_lo < hi) return 22;  // written while the stage before is read
      prev_lo = lo, prev_hi = hi;
      if (open > (p->dtype == DD_U8 ? 256 : dd::kShFold)) return 23;
      if (fold) open = 0;
      else if (s + 1 == nst) return 24;  // the last stage folds
    }
    if ((int)seen.size() != p->nchan) return 25;
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
