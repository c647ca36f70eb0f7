// Plan creation with little host memory: allocations above a limit fail, as they do under a memory
// cap. A shared-sum table that cannot be had leaves the plan in the form it falls back to; with no
// room for that either the call returns an error. Nothing is thrown across the C entry.
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "../paper_1401_8258_amd/csrc/dd_internal.h"

static size_t g_limit = ~(size_t)0;
void* operator new(size_t n) {
  if (n > g_limit) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main() {
  const int nchan = 4096, ndm = 750;  // delays and direct-read table 12.3 MB each, shared-sum table 30 MB
  std::vector<double> f((size_t)nchan), dm((size_t)ndm);
  for (int i = 0; i < nchan; ++i) f[(size_t)i] = 180.0 - i * (60.0 / nchan);
  for (int i = 0; i < ndm; ++i) dm[(size_t)i] = 0.05 * i;
  dd_plan* p = nullptr;
  if (dd_plan_create(&p, f.data(), nchan, 81.92e-6, dm.data(), ndm, DD_U8, nullptr) || !p->sh.on) return 1;
  if (p->dev_table.size() * 4 <= 16000000) return 2;
  dd_plan_destroy(p);
  g_limit = 16000000;
  p = nullptr;
  if (dd_plan_create(&p, f.data(), nchan, 81.92e-6, dm.data(), ndm, DD_U8, nullptr) || !p) return 3;
  if (p->sh.on || p->dev_table.size() != (size_t)nchan * p->ndm_pad) return 4;
  if (p->ndm_pad != (ndm + 7) / 8 * 8 || p->ngroups * p->dms_per_group != p->ndm_pad) return 5;
  dd_plan_destroy(p);
  g_limit = 1000000;
  p = nullptr;
  if (dd_plan_create(&p, f.data(), nchan, 81.92e-6, dm.data(), ndm, DD_U8, nullptr) >= 0 || p) return 6;
  std::printf("ok\n");
  return 0;
}
