// Host side of the plan: validation, the FP64 delay table (Eq. deltaTEq), tile choice,
// workspace sizing. Built with -ffp-contract=off so each double operation rounds once.
#include <sys/mman.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <limits>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "dd_internal.h"

namespace {

thread_local std::string g_err;
std::atomic<uint64_t> g_next_id{1};

// Approximate dispersion constant of Eq. dispRelationshipEquation (s MHz^2 pc^-1 cm^3).
constexpr double kDm = 4.15e3;

bool valid_tiles(const dd::Tiles& t) {
  auto in = [](int v, std::initializer_list<int> xs) {
    for (int x : xs) if (v == x) return true;
    return false;
  };
  // 8 trials per wavefront: at most 8 wavefronts (512 threads); 4 trials per wavefront (the
  // FP32 producer form only): at most 14 computing wavefronts, 16 with the producers
  const int maxw = t.g == 4 ? 16 : 8;
  return (t.g == 8 || t.g == 4) && t.w >= 0 && t.w <= (t.g == 4 ? 14 : 8) && t.s == 8 && t.cc >= 0 && t.cc <= 8 &&
         in(t.pw, {-1, 0, 1, 2, 3, 4}) && !(t.pw > 0 && t.w + t.pw > maxw);
}

// Largest in-group delay spread over all channels, for groups of gw trials with the last
// trial repeated as padding.
int32_t compute_span(const std::vector<int32_t>& delays, int32_t nchan, int32_t ndm, int gw) {
  const int ngroups = (ndm + gw - 1) / gw;
  int32_t span = 0;
  for (int32_t c = 0; c < nchan; ++c) {
    const int32_t* row = &delays[(size_t)c * ndm];
    for (int gi = 0; gi < ngroups; ++gi) {
      const int d0 = gi * gw, d1 = std::min(d0 + gw, (int)ndm) - 1;
      span = std::max(span, row[d1] - row[d0]);
    }
  }
  return span;
}

}  // namespace

namespace dd {

int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}
void clear_error() { g_err.clear(); }

int64_t elem_bytes(int32_t dtype) { return dtype == DD_F32 ? 4 : dtype == DD_F16 ? 2 : 1; }

WsLayout workspace_layout(const dd_plan* p, int64_t nout, bool linear) {
  WsLayout l{};
  l.table_off = 0;
  l.table_bytes = (int64_t)p->dev_table.size() * 4;
  l.nseg = nout > 0 ? (nout + kStatSeg - 1) / kStatSeg : 1;
  l.ntile = nout > 0 ? (nout + kTile - 1) / kTile : 1;
  int64_t o = align_up(l.table_bytes);
  l.part_off = o;
  o = align_up(o + (int64_t)p->ndm * l.ntile * 16);
  l.thr_off = o;
  o = align_up(o + (int64_t)p->ndm * 24);  // {mean, rms, threshold} per trial
  l.cnt_off = o;
  o = align_up(o + (int64_t)p->ndm * l.nseg * 4);
  l.offs_off = o;
  o = align_up(o + (int64_t)p->ndm * l.nseg * 8 + 8);
  l.tail_off = o;
  l.tail_bytes = p->dtype == DD_U8 && p->launch.form == kFormLds && !p->sh.on ? (int64_t)p->launch.L + 64 : 0;
  o = align_up(o + 2 * l.tail_bytes);
  l.quad_off = o;
  l.quad_bytes = linear && runs_direct(p) ? 4 * (int64_t)p->nchan * direct_quad_row(nout) : 0;
  o = align_up(o + l.quad_bytes);
  l.total = o;
  return l;
}

int64_t ring_table_bytes(const dd_plan* p) { return align_up((int64_t)p->dev_table.size() * 4); }

// 8-bit input keeps its samples as bytes in LDS: four byte-shifted copies of L bytes
// (L a multiple of 256), filled by 1024-byte and 256-byte DMAs, plus 256 bytes of offsets.
Launch choose_launch_u8(int32_t max_span, int nw, int cs_req, int64_t lds_cap) {
  Launch best{};
  const int64_t L = (kTile + (int64_t)max_span + 255) / 256 * 256;
  const int64_t per_chan = 4 * L + 256;
  const int64_t nchunk = 4 * (L / 1024 + (L % 1024) / 256) + 1;
  const int cs_hi = cs_req > 0 ? std::min(cs_req, nw) : nw;
  int64_t best_score = -1;
  for (int cs = cs_hi; cs >= 1; --cs) {
    if (nw % cs) continue;
    const int wpc = nw / cs;
    const int64_t nd = (nchunk + wpc - 1) / wpc;
    if (nd > kMaxDma) continue;
    int nb = (int)std::min<int64_t>(lds_cap / (cs * per_chan), 16);
    while (nb > 2 && (int64_t)(nb - 2) * nd > 63) --nb;
    if (nb < 2) continue;
    if (cs_req > 0 && best_score >= 0) break;
    const int64_t score = (int64_t)std::min(nb * cs, 24) * 64 + cs;  // deep enough, then fewest barriers
    if (score > best_score) {
      best_score = score;
      best.L = (int)L;
      best.cs = cs;
      best.nb = nb;
      best.nd = (int)nd;
      best.x4 = 1;
    }
  }
  if (best_score < 0) return Launch{};
  best.lds = (int64_t)best.nb * best.cs * per_chan;
  best.ndw = best.nd;
  return best;
}

Launch choose_launch(int32_t max_span, int nw, int nchan, int cs_req, int64_t lds_cap, int elem_bytes) {
  if (elem_bytes == 1) return choose_launch_u8(max_span, nw, cs_req, lds_cap);
  Launch best{};
  (void)nchan;
  // words one channel copy covers: tile + group spread (lane reads end at k - m + 511)
  const int64_t L = (kTile + (int64_t)max_span + 63) / 64 * 64;  // whole 64-word DMA chunks
  // a channel's slot: four shifted copies plus the group's 64 trial offsets
  const int64_t per_chan = (4 * L + 64) * 4;
  const int64_t nchunk = 4 * (L / 64) + 1;
  const int cs_hi = cs_req > 0 ? std::min(cs_req, nw) : nw;
  int64_t best_score = -1;
  for (int cs = cs_hi; cs >= 1; --cs) {
    if (nw % cs) continue;  // each stage channel gets nw / cs whole wavefronts
    const int wpc = nw / cs;
    // FP32: 256-word chunks by 16-byte DMAs plus one offsets DMA; otherwise 64-word
    // chunks (the last one the offsets), split over the channel's wavefronts
    const int64_t njx = (L / 64 + wpc - 1) / wpc;
    const int x4 = elem_bytes == 4 && njx <= kMaxX4;
    const int64_t nd = x4 ? njx + 1 : (nchunk + wpc - 1) / wpc;
    if (nd > kMaxDma) continue;
    int nb = (int)std::min<int64_t>(lds_cap / (cs * per_chan), 16);
    // with later stages in flight the wait counts them (vmcnt <= 63); a two-stage ring
    // always waits for everything, so any DMA count is legal there
    while (nb > 2 && (int64_t)(nb - 2) * nd > 63) --nb;
    if (nb < 2) continue;
    if (cs_req > 0 && best_score >= 0) break;  // an explicit request takes the largest fitting divisor
    const int64_t score = (int64_t)nb * cs * 16 + cs;  // most channels in flight, then fewest barriers
    if (score > best_score) {
      best_score = score;
      best.L = (int)L;
      best.cs = cs;
      best.nb = nb;
      best.nd = (int)nd;
      best.x4 = x4;
    }
  }
  if (best_score < 0) return Launch{};
  best.lds = (int64_t)best.nb * best.cs * per_chan;
  best.ndw = best.nd;
  return best;
}

// FP32 input, one producer wavefront: it issues every channel of a stage whole (the four
// copies as L/64 16-byte DMAs, then the offsets), so any stage width works, and the
// computing wavefronts never wait on a DMA issue. A channel's copies must fit the 16
// per-lane descriptors (L <= 1024 words).
Launch choose_launch_prod(int32_t max_span, int nchan, int cs_req, int64_t lds_cap, int nprod) {
  Launch best{};
  const int64_t L = (kTile + (int64_t)max_span + 63) / 64 * 64;
  if (L / 64 > kMaxX4) return best;
  const int64_t per_chan = (4 * L + 64) * 4;
  const int nd = (int)(L / 64) + 1;
  // at least one channel per producer (stage channels past the last repeat it)
  const int cs_hi = cs_req > 0 ? cs_req : std::max(nprod, std::min(8, nchan));
  int64_t best_score = -1;
  for (int cs = cs_hi; cs >= 1; --cs) {
    if (cs % nprod) continue;  // each producer takes cs / nprod whole channels
    const int64_t ndw = (int64_t)(cs / nprod) * nd;
    int nb = (int)std::min<int64_t>(lds_cap / (cs * per_chan), 16);
    // every DMA of the nb - 1 stages ahead is in flight at once: a wavefront issues at
    // most 63 before it stalls (vmcnt), so the producer never waits to issue
    while (nb > 2 && (int64_t)(nb - 1) * ndw > 63) --nb;
    if (nb < 2 || ndw > 63) continue;
    if (cs_req > 0 && best_score >= 0) break;
    // the fewest barriers, then the deepest ring: the producers keep their DMAs ahead of
    // the computing wavefronts, so a double buffer of wide stages measured fastest
    const int64_t score = (int64_t)cs * 64 + nb;
    if (score > best_score) {
      best_score = score;
      best.L = (int)L;
      best.cs = cs;
      best.nb = nb;
      best.nd = nd;
      best.ndw = (int)ndw;
    }
  }
  if (best_score < 0) return Launch{};
  best.x4 = 1;
  best.prod = nprod;
  best.lds = (int64_t)best.nb * best.cs * per_chan;
  return best;
}

// Register-window form: groups of 64 trials (8 wavefronts of 8), one padded copy of each
// channel per LDS slot. Per (group, channel, wavefront) the table holds the window's LDS byte
// offset (a = the wavefront's first relative delay rounded down to 8: 12 words per 8
// samples, so 6a bytes) and the eight trials' register indices (relative delay - a), one
// byte each. Returns false when some window needs more than kRwMaxChunks chunks or the slots
// do not fit in LDS.
bool plan_regwin(dd_plan* p, int64_t lds_cap) {
  const int G = 8, NW = kRwTrials / 8;
  const int32_t nchan = p->nchan, ndm = p->ndm;
  const int ngroups = (ndm + kRwTrials - 1) / kRwTrials;
  std::vector<int32_t> tab;
  const int64_t moff = ((int64_t)ngroups * nchan + 3) / 4 * 4;
  // seven channels of zero records after the last group: a stage reads eight channels' records
  tab.assign((size_t)(moff + ((int64_t)ngroups * nchan + kRwStage - 1) * NW * 4), 0);
  int32_t max_idx = 0, max_a = 0, span = 0;
  for (int gi = 0; gi < ngroups; ++gi) {
    for (int32_t c = 0; c < nchan; ++c) {
      const int32_t* row = &p->delays[(size_t)c * ndm];
      auto dl = [&](int d) { return row[d < ndm ? d : ndm - 1]; };  // padded trials repeat the last DM
      const int32_t first = dl(gi * kRwTrials);
      tab[(size_t)gi * nchan + c] = first;
      span = std::max(span, dl(gi * kRwTrials + kRwTrials - 1) - first);
      for (int w = 0; w < NW; ++w) {
        const int d0 = gi * kRwTrials + G * w;
        const int32_t a = (dl(d0) - first) & ~7;
        uint32_t pk[2] = {0u, 0u};
        int32_t wmax = 0;
        for (int g = 0; g < G; ++g) {
          const int32_t idx = dl(d0 + g) - first - a;
          max_idx = std::max(max_idx, idx);
          wmax = std::max(wmax, idx);
          if (idx > 4 * kRwMaxChunks - 8) return false;
          pk[g / 4] |= (uint32_t)idx << (8 * (g % 4));
        }
        max_a = std::max(max_a, a);
        int32_t* m = &tab[(size_t)(moff + (((int64_t)gi * nchan + c) * NW + w) * 4)];
        m[0] = 6 * a;
        m[1] = (int32_t)pk[0];
        m[2] = (int32_t)pk[1];
        m[3] = (wmax + 8 + 3) / 4;  // chunks this wavefront's window needs in this channel
      }
    }
  }
  int nch = (max_idx + 8 + 3) / 4;
  nch = nch <= 6 ? 6 : nch <= 8 ? 8 : nch <= 10 ? 10 : 12;
  // samples the windows touch (lane 63 reads up to 8 * 63 + a + 4 nch - 1), and the 16-byte
  // DMAs that cover them: three 16-byte positions per 8 samples (two of data, one of padding)
  const int64_t need = 8 * 63 + (int64_t)max_a + 4 * nch;
  const int ndma = (int)((3 * ((need + 7) / 8) + 63) / 64);
  const int xs = 8 * ((64 * ndma - 1) / 3 + 1);
  const int64_t stage = (int64_t)kRwStage * 1024 * ndma;
  int nb = (int)std::min<int64_t>(lds_cap / stage, 8);
  while (nb > 2 && (int64_t)(nb - 2) * ndma > 63) --nb;  // a wait counts at most 63 DMAs
  if (nb < 2) return false;
  Launch l{};
  l.form = kFormRegWin;
  l.L = xs;
  l.cs = kRwStage;
  l.nb = nb;
  l.nd = ndma;
  l.ndw = ndma;
  l.x4 = 1;
  l.nch = nch;
  l.lds = (int64_t)nb * stage;
  p->launch = l;
  p->tiles = Tiles{G, NW, 8, kRwStage, -1};
  p->dms_per_group = kRwTrials;
  p->ngroups = ngroups;
  p->ndm_pad = ngroups * kRwTrials;
  p->max_span = span;
  p->dev_table.swap(tab);
  return true;
}

// Direct-read form: t.g trials per wavefront, t.w wavefronts per workgroup; the table is the
// plain delays per (channel, padded trial). A wavefront's loads span at most two 1024-sample
// sub-tiles, so a ring's mirror of launch.L + 64 samples covers every window that starts
// before the ring's end.
int plan_direct(dd_plan* p, const Tiles& t) {
  if (t.g != 1 && t.g != 2 && t.g != 4)
    return fail(DD_ERR_UNSUPPORTED, "the direct-read form takes dms_per_wave 1, 2 or 4");
  if (t.w < 1 || t.w > 8) return fail(DD_ERR_UNSUPPORTED, "the direct-read form takes waves 1..8");
  if (t.s != 16 && !(t.s == 32 && t.g <= 2))
    return fail(DD_ERR_UNSUPPORTED, "the direct-read form takes samples_per_lane 16, or 32 with dms_per_wave "
                                    "1 or 2");
  const int32_t nchan = p->nchan, ndm = p->ndm;
  p->tiles = Tiles{t.g, t.w, t.s, 0, -1};
  p->dms_per_group = t.g * t.w;
  p->ngroups = (ndm + p->dms_per_group - 1) / p->dms_per_group;
  p->ndm_pad = p->ngroups * p->dms_per_group;
  p->max_span = compute_span(p->delays, nchan, ndm, p->dms_per_group);
  Launch l{};
  l.form = kFormDirect;
  l.L = (int)(2 * kDirectTile);  // the widest wavefront tile (two sub-tiles)
  p->launch = l;
  return DD_OK;
}

// The direct-read form's device table: every channel's delays, the last trial's in the padding.
void table_direct(dd_plan* p) {
  const int32_t nchan = p->nchan, ndm = p->ndm;
  p->dev_table.assign((size_t)nchan * p->ndm_pad, 0);
  for (int32_t c = 0; c < nchan; ++c) {
    const int32_t* row = &p->delays[(size_t)c * ndm];
    int32_t* drow = &p->dev_table[(size_t)c * p->ndm_pad];
    for (int32_t d = 0; d < p->ndm_pad; ++d) drow[d] = row[d < ndm ? d : ndm - 1];
  }
}

// The LDS form's device table: per (channel, trial) the LDS byte offset of the trial's first
// 4-sample chunk inside the channel slot: relative delay k to the group's first trial is read
// from copy m = k & 3 at word k - m; then [ngroups][nchan] the groups' first delays.
void table_lds(dd_plan* p) {
  const int32_t nchan = p->nchan, ndm = p->ndm;
  p->dev_table.resize((size_t)nchan * p->ndm_pad + (size_t)p->ngroups * nchan);
  int32_t* gb = &p->dev_table[(size_t)nchan * p->ndm_pad];
  for (int32_t c = 0; c < nchan; ++c) {
    const int32_t* row = &p->delays[(size_t)c * ndm];
    int32_t* drow = &p->dev_table[(size_t)c * p->ndm_pad];
    for (int32_t gi = 0; gi < p->ngroups; ++gi) {
      const int32_t base = row[gi * p->dms_per_group];
      gb[(size_t)gi * nchan + c] = base;
      for (int32_t j = 0; j < p->dms_per_group; ++j) {
        const int32_t d = gi * p->dms_per_group + j;
        const int32_t k = row[d < ndm ? d : ndm - 1] - base;
        const int32_t m = k & 3;
        // byte offset: 32-bit words for 16/32-bit input, bytes for 8-bit input
        drow[d] = p->dtype == DD_U8 ? m * p->launch.L + (k - m) : 4 * (m * p->launch.L + (k - m));
      }
    }
  }
}

// ------------------------------------------------------------------ shared-sum form

namespace {

constexpr int kShMaxTrials = 2 * 16;  // trials of a group

// One bundle of 1..4 consecutive channels for one group of trials.
struct Bundle {
  Bundle() {}  // many are tried: nothing is cleared
  int c0, m, np, slot, rows;  // lowest channel, channels, patterns, bytes of a pattern's sums, rows
  int records() const { return rows * ((np + kShRecPat - 1) / kShRecPat); }
  int32_t off[4], chan;   // window starts; the first channel
  bool down;              // the channels run down from it
  uint8_t code[kShMaxPat];
  int32_t trial[kShMaxTrials];  // byte offset from the bundle's LDS base | words past 16 bytes
  int64_t bytes() const { return (int64_t)np * slot; }
  double cost;
};

// Clocks of one CU with all its wavefronts at work (measured): a trial's sum of one bundle
// added, a pattern's sums of one row formed, and what a row takes besides.
constexpr double kShAddClk = 26.0;
constexpr double kShPatClk = 21.0;
constexpr double kShRowClk = 60.0;

// Channels c0 .. c0 + m - 1 for trials d0 .. d0 + n - 1 (past the last trial: the last one).
// Delays relative to the first channel must not be negative (channels neither rising nor
// falling in frequency may fail this). False when the patterns are too many or too wide, or the sums take more than cap bytes.
bool make_bundle(const dd_plan* p, int c0, int m, int d0, int n, int64_t cap, Bundle* b) {
  const int32_t ndm = p->ndm;
  const int nd = std::min(n, (int)ndm - d0);  // trials of the group's own
  // the channels in order of their delays, up or down from the smallest
  const int32_t* row[4];
  auto last = [&](int j) { return p->delays[(size_t)(c0 + j) * ndm + d0 + nd - 1]; };
  b->down = m > 1 && last(m - 1) < last(0);
  b->chan = b->down ? c0 + m - 1 : c0;
  for (int j = 0; j < m; ++j) row[j] = &p->delays[(size_t)(b->down ? c0 + m - 1 - j : c0 + j) * ndm + d0];
  const int32_t k0 = row[0][0];
  const int64_t chunks = (int64_t)(row[0][nd - 1] - k0) / 4 + 4 * 63 + 1;
  if (16 * chunks > cap) return false;
  b->c0 = c0;
  b->m = m;
  b->slot = (int)(16 * chunks);
  b->rows = (int)((chunks + sh_row_chunks(p->dtype) - 1) / sh_row_chunks(p->dtype));
  if (b->rows > kShMaxRows) return false;
  // most bundles that fail do so by their first and last trials
  for (int j = 1; j < m; ++j)
    if (std::abs((row[j][nd - 1] - row[0][nd - 1]) - (row[j][0] - row[0][0])) > kShMaxE) return false;
  int32_t code[kShMaxTrials] = {0};
  b->off[0] = k0;
  for (int j = 1; j < m; ++j) {
    int32_t rel[kShMaxTrials], lo, hi;
    const int32_t *rj = row[j], *r0 = row[0];
    lo = hi = rj[0] - r0[0];
    for (int t = 0; t < nd; ++t) {
      const int32_t r = rj[t] - r0[t];
      rel[t] = r;
      lo = r < lo ? r : lo;
      hi = r > hi ? r : hi;
    }
    if (hi - lo > kShMaxE || lo < 0 || lo > kShMaxOff) return false;
    b->off[j] = k0 + lo;
    for (int t = 0; t < nd; ++t) code[t] |= (rel[t] - lo) << (2 * (j - 1));
  }
  // channels the bundle lacks repeat the first one's start (their samples are not loaded)
  for (int j = m; j < 4; ++j) b->off[j] = b->off[0];
  int8_t slot_of[64];
  std::memset(slot_of, -1, sizeof(slot_of));
  b->np = 0;
  for (int t = 0; t < nd; ++t) {
    const int c = code[t];
    if (slot_of[c] < 0) {
      if (b->np == kShMaxPat) return false;
      slot_of[c] = (int8_t)b->np;
      b->code[b->np++] = (uint8_t)c;
    }
    const int32_t k = row[0][t] - k0;
    b->trial[t] = slot_of[c] * b->slot + (k & ~3) * 4 + (k & 3);
  }
  if (b->bytes() > cap) return false;
  for (int t = nd; t < n; ++t) b->trial[t] = b->trial[nd - 1];
  b->cost = n * kShAddClk + b->rows * (b->np * kShPatClk + kShRowClk);
  return true;
}

// Bundles of channels [c0, c1) (at most 4 channels): one of all, or its halves where that is
// cheaper or the whole does not fit. False when even single channels do not fit.
bool bundle_quad(const dd_plan* p, int c0, int c1, int d0, int n, int64_t cap, std::vector<Bundle>* out, double* cost) {
  const int m = c1 - c0;
  const size_t at = out->size();
  out->resize(at + 1);
  const bool whole = m != 3 && make_bundle(p, c0, m, d0, n, cap, &(*out)[at]);
  // a bundle of half the channels adds as much per trial: halves can only pay when the whole
  // forms more than that
  if (whole) {
    const double c = (*out)[at].cost;
    if (m == 1 || c <= 2 * (n * kShAddClk + (*out)[at].rows * (kShPatClk + kShRowClk))) {
      *cost += c;
      return true;
    }
  } else {
    out->pop_back();
    if (m == 1) return false;
  }
  const int mid = c0 + (m >= 3 ? 2 : 1);
  double hc = 0;
  const bool halves = bundle_quad(p, c0, mid, d0, n, cap, out, &hc) && bundle_quad(p, mid, c1, d0, n, cap, out, &hc);
  if (whole && (!halves || (*out)[at].cost <= hc)) {
    out->resize(at + 1);
    *cost += (*out)[at].cost;
    return true;
  }
  if (!halves) {
    out->resize(at);
    return false;
  }
  if (whole) out->erase(out->begin() + (std::ptrdiff_t)at);
  *cost += hc;
  return true;
}

// The FP32 additions of a series, by the channels that their results hold: a result's rounding
// error grows as its size, so the variance of a total's error as the number of channels (noise
// about zero) up to its square (noise on a level) summed over the additions.
struct Adds {
  double lin = 0, sq = 0;
  void add(int n) {
    lin += n;
    sq += (double)n * n;
  }
  bool no_more_than(const Adds& o) const { return lin <= o.lin && sq <= o.sq; }
};

// Channels [c0, c1) in blocks of DD_CHAN_BLOCK, channel by channel, joining a total of the c0
// channels before them.
Adds by_channel(int c0, int c1) {
  Adds a;
  for (int b = c0; b < c1; b += DD_CHAN_BLOCK) {
    const int e = std::min(c1, b + DD_CHAN_BLOCK);
    for (int k = 2; k <= e - b; ++k) a.add(k);
    if (b) a.add(e);
  }
  return a;
}

// The same channels as one block of these bundles.
Adds by_bundle(int c0, const std::vector<Bundle>& v, const std::vector<int>& order) {
  Adds a;
  int n = 0;
  for (int i : order) {
    for (int k = 2; k <= v[(size_t)i].m; ++k) a.add(k);
    if (n) a.add(n + v[(size_t)i].m);
    n += v[(size_t)i].m;
  }
  if (c0) a.add(c0 + n);
  return a;
}

}  // namespace

namespace {

// Asks for large pages for what a table has reserved: the page faults of filling one of tens of
// megabytes take as long as its contents (4096 channels x 2048 trials, 84 MB: 33 -> 25 ms).
void huge_pages(const std::vector<int32_t>& v) {
  const uintptr_t page = (uintptr_t)2 << 20;
  const uintptr_t a = (reinterpret_cast<uintptr_t>(v.data()) + page - 1) / page * page;
  const uintptr_t e = reinterpret_cast<uintptr_t>(v.data() + v.capacity()) / page * page;
  if (a < e) (void)madvise(reinterpret_cast<void*>(a), e - a, MADV_HUGEPAGE);  // a hint only
}

}  // namespace

// Device table: per group {offset, stages}, then the stages' records (dd_internal.h).
bool plan_shared(dd_plan* p, int64_t lds_cap, double max_cost) {
  const int32_t nchan = p->nchan, ndm = p->ndm;
  const int fold = p->dtype == DD_U8 ? 256 : kShFold;
  const int32_t eb = (int32_t)elem_bytes(p->dtype);
  const int maxw = kShWaves, G = kShG;
  // Wavefronts per workgroup: one, two or four workgroups share a CU's wavefront slots and its
  // LDS. More trials per workgroup share each sum, fewer keep windows short where delays
  // grow by many samples per trial. The cheapest in LDS clocks per trial on a sample of the
  // groups and channels wins.
  // An FP32 plan of few channels (a step of a subband plan) has few stages, and a workgroup alone
  // on its CU would leave it idle while it starts and while it stores its series: two or four
  // share it (passes of 32-channel subbands 1 to 9% faster than with one).
  const bool few = p->dtype == DD_F32 && nchan < kShMinChans;
  int best_div = 0;
  double best = 0;
  std::vector<Bundle> v;
  for (int div = few ? 2 : 1; div <= 4; div *= 2) {
    const int n = G * (maxw / div);
    if (div < 4 && ndm <= n / 2) continue;  // half the workgroup or more would be padding
    const int64_t cap = (lds_cap / div - kShSpare) / 2 / 256 * 256;
    const int ng = (ndm + n - 1) / n, nq = (nchan + 3) / 4;
    const int gs = std::max(1, ng / 4), qs = std::max(1, nq / 16);
    double cost = 0;
    int64_t cnt = 0;
    bool ok = true;
    for (int g = ng - 1; g >= 0 && ok; g -= gs)
      for (int q = nq - 1; q >= 0 && ok; q -= qs) {
        v.clear();
        ok = bundle_quad(p, 4 * q, std::min(nchan, 4 * q + 4), g * n, n, cap, &v, &cost);
        ++cnt;
      }
    if (!ok || !cnt) continue;
    const double per = cost / ((double)cnt * n);
    if (!best_div || per < best) best = per, best_div = div;
  }
  if (!best_div || !(best < max_cost)) return false;
  const int nw = maxw / best_div, n = G * nw;
  const int64_t cap = (lds_cap / best_div - kShSpare) / 2 / 256 * 256;
  const int ng = (ndm + n - 1) / n;
  // ndm_pad is still the other form's (kShDirectClk, kShLdsClk)
  const double clk = best * ((double)ng * n) / p->ndm_pad;
  if (p->dtype == DD_U8 && !(clk < kShDirectClk)) return false;
  const bool lds_best = p->dtype == DD_F32 && p->tiles.g == 4 && p->tiles.w == 14 && ndm > kShLdsTrials;
  if (lds_best && !(clk < kShLdsClk)) return false;
  const int ints = sh_stage_ints(nw);
  std::vector<int32_t> tab((size_t)(2 * ng + 63) / 64 * 64 + (size_t)ints, 0);
  int64_t max_reach = 0, stages = 0;
  std::vector<int> order;
  // a group's records of further rounds, after its stages: (the record to link from, their place)
  std::vector<int32_t> over;
  struct Link {
    bool over;
    size_t at, to;
  };
  std::vector<Link> links;
  for (int g = 0; g < ng; ++g) {
    const size_t first = tab.size();
    int nst = 0;
    over.clear();
    links.clear();
    v.clear();
    for (int f0 = 0, f1 = 0; f0 < nchan; f0 = f1) {
      double cost = 0;
      f1 = std::min(nchan, f0 + fold);
      for (int q = v.empty() ? f0 : v.back().c0 + v.back().m; q < f1; q += 4)
        if (!bundle_quad(p, q, std::min(f1, q + 4), g * n, n, cap, &v, &cost)) return false;
      // the block's length: the FP32 additions of a longer one may round worse than channel by
      // channel (those of DD_CHAN_BLOCK channels never do: its partial sums are among the others')
      for (int len = fold;; len /= 2) {
        f1 = std::min(nchan, f0 + len);
        order.clear();
        for (size_t i = 0; i < v.size() && v[i].c0 < f1; ++i) order.push_back((int)i);
        // bundles of like pattern counts share a stage: its slowest row sets its time
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return v[(size_t)a].np < v[(size_t)b].np; });
        if (p->dtype == DD_U8 || len <= DD_CHAN_BLOCK || by_bundle(f0, v, order).no_more_than(by_channel(f0, f1))) break;
      }
      for (size_t i = 0; i < order.size();) {
        // up to kShMaxBundles bundles that fit half the LDS share: as many as leave the fewest
        // wavefronts without a row in the last round of rows
        size_t e = i + 1;
        int64_t bytes = 0;
        int nrec = 0;
        double best_fill = 0;
        for (size_t k = i; k < order.size() && k - i < (size_t)kShMaxBundles; ++k) {
          const Bundle& b = v[(size_t)order[k]];
          bytes += b.bytes();
          nrec += b.records();
          if (bytes > cap) break;
          const double fill = (double)nrec / ((nrec + nw - 1) / nw * nw);
          if (fill >= best_fill) best_fill = fill, e = k + 1;
        }
        const int nb = (int)(e - i);
        const size_t st = tab.size();
        tab.resize(st + (size_t)ints, 0);
        int64_t base[kShMaxBundles];  // the bundles' LDS offsets; odd stages use the second half
        int64_t o = kShSpare + (nst & 1 ? cap : 0);
        for (int q = 0; q < nb; ++q) base[q] = o, o += v[(size_t)order[i + q]].bytes();
        for (int w = 0; w < nw; ++w) {
          int32_t* rec = &tab[st + (size_t)w * kShRecInts];
          for (int q = 0; q < nb; ++q)
            for (int t = 0; t < G; ++t) {
              const int32_t tr = (int32_t)base[q] + v[(size_t)order[i + q]].trial[G * w + t];
              rec[G * q + t] = tr & ~15;
              rec[6] |= (tr & 3) << (2 * (G * q + t));
            }
          rec[7] = (G * nb - 1) | (e == order.size() ? 256 : 0);
        }
        // the rows, those of many patterns in parts and first, round the wavefronts
        int w = 0;
        bool more = false;  // further rounds
        Link last[16];      // each wavefront's last record
        for (int q = nb - 1; q >= 0; --q) {
          const Bundle& b = v[(size_t)order[i + q]];
          const int parts = (b.np + kShRecPat - 1) / kShRecPat;
          int32_t far = 0;
          int32_t like[kShFormInts] = {};  // the part's records, their row aside
          like[0] = b.off[0];
          for (int j = 1; j < 4; ++j) {
            far = std::max(far, b.off[j] - b.off[0]);
            like[j] = (b.off[j] - b.off[0]) * eb;
          }
          like[4] = b.chan;
          like[6] = b.slot;
          like[7] = b.m << 8 | (b.down ? 4096 : 0);
          for (int part = 0; part < parts; ++part) {
            const int p0 = b.np * part / parts, p1 = b.np * (part + 1) / parts;
            like[5] = (int32_t)(base[q] + (int64_t)p0 * b.slot);
            uint8_t code[8];
            for (int c = 0; c < 8; ++c) code[c] = p0 + c < p1 ? b.code[p0 + c] : 64;
            std::memcpy(like + 8, code, 8);
            for (int row = 0; row < b.rows; ++row) {
              size_t at = st + (size_t)w * kShRecInts + kShAddInts;
              if (more) {
                at = over.size();
                over.resize(at + kShFormInts);
                links.push_back({last[w].over, last[w].at, at});
              }
              last[w] = {more, at, 0};
              int32_t* rec = more ? &over[at] : &tab[at];
              std::memcpy(rec, like, sizeof(like));
              rec[7] |= row;
              rec[10] = far + sh_reach(p->dtype, row);
              if (++w == nw) w = 0, more = true;
            }
          }
          max_reach = std::max<int64_t>(max_reach, far + sh_reach(p->dtype, b.rows - 1));
        }
        // wavefronts without a row: no channels and no pattern
        for (; !more && w < nw; ++w) {
          int32_t* rec = &tab[st + (size_t)w * kShRecInts + kShAddInts];
          rec[8] = rec[9] = 0x40404040;
        }
        ++nst;
        i = e;
      }
      v.erase(v.begin(), v.begin() + (std::ptrdiff_t)order.size());
    }
    tab.resize(tab.size() + (size_t)kShPad * ints, 0);
    const int32_t after = (int32_t)(tab.size() - first);
    for (const Link& l : links) (l.over ? over[l.at + 11] : tab[l.at + 11]) = after + (int32_t)l.to;
    tab.insert(tab.end(), over.begin(), over.end());
    tab[2 * (size_t)g] = (int32_t)first;
    tab[2 * (size_t)g + 1] = nst;
    stages += nst;
    if (tab.size() > ((size_t)1 << 29)) return false;
    if (g == 0) {
      tab.reserve(std::min((size_t)1 << 29, tab.size() * (size_t)ng / 4 * 5));
      huge_pages(tab);
    }
  }
  p->sh.on = true;
  p->sh.nw = nw;
  p->sh.lds = kShSpare + 2 * cap;
  p->sh.mirror = (int32_t)max_reach;
  p->sh.stages = (double)stages / ng;
  p->dms_per_group = n;
  p->ngroups = ng;
  p->ndm_pad = ng * n;
  p->dev_table.swap(tab);
  return true;
}

}  // namespace dd

extern "C" {

const char* dd_last_error(void) { return g_err.c_str(); }

const char* dd_version(void) { return "1.5"; }

}  // extern "C"

namespace dd {

namespace {

// plan_shared, or no shared-sum form where its table, which may be several times the others', does
// not fit the host's memory.
bool try_shared(dd_plan* p, int64_t lds_cap, double max_cost) {
  try {
    return plan_shared(p, lds_cap, max_cost);
  } catch (const std::bad_alloc&) {
    return false;
  }
}

int create(dd_plan** out, const double* freq_mhz, int32_t nchan, double tsamp_s, const double* dm,
           int32_t ndm, int32_t in_dtype, const dd_tuning* tuning, int64_t lds_cap, bool shared_any) {
  dd::clear_error();
  if (!out) return dd::fail(DD_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  if (!freq_mhz || !dm) return dd::fail(DD_ERR_INVALID_ARG, "freq_mhz and dm must be non-NULL");
  if (nchan < 1 || ndm < 1) return dd::fail(DD_ERR_INVALID_ARG, "nchan and ndm must be >= 1");
  if (!(tsamp_s > 0.0) || !std::isfinite(tsamp_s))
    return dd::fail(DD_ERR_INVALID_ARG, "tsamp must be finite and > 0");
  if (in_dtype != DD_F32 && in_dtype != DD_F16 && in_dtype != DD_U8)
    return dd::fail(DD_ERR_INVALID_ARG, "unknown input dtype");
  double fmax = 0.0;
  for (int32_t c = 0; c < nchan; ++c) {
    if (!std::isfinite(freq_mhz[c]) || !(freq_mhz[c] > 0.0))
      return dd::fail(DD_ERR_INVALID_ARG, "frequencies must be finite and > 0 (channel " +
                                              std::to_string(c) + ")");
    if (freq_mhz[c] > fmax) fmax = freq_mhz[c];
  }
  for (int32_t d = 0; d < ndm; ++d) {
    if (!std::isfinite(dm[d]) || dm[d] < 0.0)
      return dd::fail(DD_ERR_INVALID_ARG, "DMs must be finite and >= 0 (trial " + std::to_string(d) + ")");
    if (d > 0 && dm[d] < dm[d - 1])
      return dd::fail(DD_ERR_INVALID_ARG, "DM trials must be in non-decreasing order");
  }

  dd::Tiles t{8, 0, 8, 0, 0};
  const int form_req = tuning ? tuning->kernel_form : DD_FORM_AUTO;
  if (form_req != DD_FORM_AUTO && form_req != DD_FORM_LDS && form_req != DD_FORM_REGWIN &&
      form_req != DD_FORM_DIRECT)
    return dd::fail(DD_ERR_UNSUPPORTED, "unknown kernel_form");
  if (form_req == DD_FORM_REGWIN && in_dtype != DD_F32)
    return dd::fail(DD_ERR_UNSUPPORTED, "the register-window form takes FP32 input only");
  if (form_req == DD_FORM_DIRECT && in_dtype != DD_U8)
    return dd::fail(DD_ERR_UNSUPPORTED, "the direct-read form takes 8-bit input only");
  // the register-window form is the FP32 default when no tile field is set
  const bool tiles_set = tuning && (tuning->dms_per_wave || tuning->waves || tuning->samples_per_lane ||
                                    tuning->chan_stage || tuning->producer_waves);
  const bool try_regwin = in_dtype == DD_F32 && (form_req == DD_FORM_REGWIN ||
                                                 (form_req == DD_FORM_AUTO && !tiles_set && dd::kAutoRegWin));
  if (tuning) {
    if (tuning->dms_per_wave) t.g = tuning->dms_per_wave;
    if (tuning->waves) t.w = tuning->waves;
    if (tuning->samples_per_lane) t.s = tuning->samples_per_lane;
    t.cc = tuning->chan_stage;
    t.pw = tuning->producer_waves;
  }
  // a plan without any choice of the caller's runs in the shared-sum form where it pays
  // (plan_shared), except FP32 beams of few channels (kShMinChans)
  const bool auto_form =
      form_req == DD_FORM_AUTO && !tiles_set && (shared_any || !(in_dtype == DD_F32 && nchan < dd::kShMinChans));
  const double sh_cost = in_dtype == DD_F32 && nchan < dd::kShMinChans ? dd::kShFewClk
                                                                       : std::numeric_limits<double>::infinity();
  // 8-bit input takes the direct-read form unless the caller asks for another form or sets
  // an LDS-form tile field
  const bool direct = form_req == DD_FORM_DIRECT || (form_req == DD_FORM_AUTO && in_dtype == DD_U8 && !tiles_set);
  if (direct) {
    t.g = tuning && tuning->dms_per_wave ? tuning->dms_per_wave : 2;
    t.w = tuning && tuning->waves ? tuning->waves : 4;
    t.s = tuning && tuning->samples_per_lane ? tuning->samples_per_lane : 16;
  } else if (!valid_tiles(t)) {
    return dd::fail(DD_ERR_UNSUPPORTED, "unsupported tuning");
  }
  if (t.pw > 0 && in_dtype != DD_F32 && !direct)
    return dd::fail(DD_ERR_UNSUPPORTED, "producer wavefronts are available for FP32 input only");
  if (!direct && t.g == 4 && (in_dtype != DD_F32 || t.pw < 0))
    return dd::fail(DD_ERR_UNSUPPORTED, "4 DM trials per wavefront is the FP32 producer form only");

  std::unique_ptr<dd_plan> owner(new dd_plan());
  dd_plan* p = owner.get();
  p->nchan = nchan;
  p->ndm = ndm;
  p->dtype = in_dtype;
  p->tsamp = tsamp_s;
  p->freq.assign(freq_mhz, freq_mhz + nchan);
  p->dm.assign(dm, dm + ndm);
  p->delays.resize((size_t)nchan * ndm);

  // Eq. deltaTEq: x = ((k * DM) * (1/(f*f) - 1/(fr*fr))) / tsamp, round half away from zero.
  // x is not negative (no frequency exceeds fmax) and grows with the trial, so the last one's
  // bounds a channel's delays, and a conversion to an integer is its floor.
  const double inv_ref = 1.0 / (fmax * fmax);
  int32_t maxd = 0;
  for (int32_t c = 0; c < nchan; ++c) {
    const double diff = 1.0 / (freq_mhz[c] * freq_mhz[c]) - inv_ref;
    if (!(((kDm * dm[ndm - 1]) * diff) / tsamp_s < (double)std::numeric_limits<int32_t>::max() + 0.5))
      return dd::fail(DD_ERR_INVALID_ARG, "delay exceeds 2^31-1 samples");
    int32_t* row = &p->delays[(size_t)c * ndm];
    for (int32_t d = 0; d < ndm; ++d) {
      const double x = ((kDm * dm[d]) * diff) / tsamp_s;
      const int32_t fl = (int32_t)x;
      row[d] = fl + (x - (double)fl >= 0.5 ? 1 : 0);
    }
    maxd = std::max(maxd, row[ndm - 1]);
  }
  p->maxdelay = maxd;

  if (direct) {
    const int rc = dd::plan_direct(p, t);
    if (rc) return rc;
    if (!(auto_form && try_shared(p, lds_cap, sh_cost))) dd::table_direct(p);
    p->id = g_next_id.fetch_add(1);
    *out = owner.release();
    return DD_OK;
  }
  if (try_regwin) {
    if (dd::plan_regwin(p, lds_cap)) {
      p->id = g_next_id.fetch_add(1);
      *out = owner.release();
      return DD_OK;
    }
    if (form_req == DD_FORM_REGWIN)
      return dd::fail(DD_ERR_UNSUPPORTED, "the delay spread of 8 consecutive DM trials does not fit the register "
                                          "window (at most 40 samples with the alignment)");
  }
  // FP32 input: by default two producer wavefronts issue every LDS DMA beside the computing
  // ones, when one DM group's channel windows fit their 16-byte DMAs. Otherwise, and for
  // other input: 8 DM trials per wavefront, as many wavefronts as keep the LDS ring at least
  // 8 channels deep (unless the caller fixed the count).
  // With trials per wavefront and wavefronts left open, FP32 input first tries 4 trials per
  // wavefront (up to 14 computing wavefronts beside 2 producers in 1024 threads: 56 trials
  // share each staged channel, 10% faster than 6 x 8 on the full workload), then 8.
  int32_t span = 0;
  dd::Launch lg{};
  bool placed = false;
  const bool g_open = !(tuning && (tuning->dms_per_wave || tuning->waves));
  const int g_try[2] = {g_open && in_dtype == DD_F32 ? 4 : t.g, t.g};
  for (int gi = 0; gi < 2 && !placed; ++gi) {
    const int g = g_try[gi];
    if (gi == 1 && g == g_try[0]) break;
    const int maxw = g == 4 ? 16 : 8;  // wavefronts a workgroup may hold (1024 or 512 threads)
    const int npw = t.pw > 0 ? t.pw : (t.pw == 0 && in_dtype == DD_F32 && t.w + 2 <= maxw) ? 2 : 0;
    if (!(in_dtype == DD_F32 && npw > 0)) continue;
    const int wp8[5] = {6, 4, 3, 2, 1};
    const int wp4[5] = {14, 12, 8, 4, 1};
    const int* wp_opts = g == 4 ? wp4 : wp8;
    for (int oi = 0; oi < 5 && !placed; ++oi) {
      const int nw = t.w ? t.w : std::min(wp_opts[oi], maxw - npw);
      const int32_t sp = compute_span(p->delays, nchan, ndm, g * nw);
      const dd::Launch l = dd::choose_launch_prod(sp, nchan, t.cc, lds_cap, npw);
      if (l.nb >= 2) t.g = g, t.w = nw, span = sp, lg = l, placed = true;  // the most wavefronts that fit
      if (t.w) break;
    }
  }
  if (in_dtype == DD_F32 && !placed) {
    if (t.pw > 0 || t.g == 4)
      return dd::fail(DD_ERR_UNSUPPORTED, "one DM group's windows do not fit the producer wavefronts' "
                                          "16-byte DMAs; use fewer DMs per workgroup or no producer");
    if (!(tuning && tuning->waves)) t.w = 0;  // automatic: fall back to the other form
  }
  const int w_opts[4] = {8, 4, 2, 1};
  for (int oi = 0; oi < 4 && !placed; ++oi) {
    const int nw = t.w ? t.w : w_opts[oi];
    span = compute_span(p->delays, nchan, ndm, t.g * nw);
    lg = dd::choose_launch(span, nw, nchan, t.cc, lds_cap, (int)dd::elem_bytes(in_dtype));
    if (t.w || (lg.nb >= 2 && (int64_t)lg.nb * lg.cs >= std::min(8, nchan + 1)) || nw == 1) {
      t.w = nw;
      break;
    }
  }
  if (lg.nb < 2)
    return dd::fail(DD_ERR_UNSUPPORTED, "delay spread of one DM group (" + std::to_string(span) +
                                            " samples) does not fit in LDS; use fewer DMs per workgroup");
  p->tiles = t;
  lg.form = dd::kFormLds;
  p->launch = lg;
  p->dms_per_group = t.g * t.w;
  p->ngroups = (ndm + p->dms_per_group - 1) / p->dms_per_group;
  p->ndm_pad = p->ngroups * p->dms_per_group;
  p->max_span = span;
  if (!(auto_form && try_shared(p, lds_cap, sh_cost))) dd::table_lds(p);
  p->id = g_next_id.fetch_add(1);
  *out = owner.release();
  return DD_OK;
}

}  // namespace

// dd_plan_create with the LDS bytes one workgroup may take (the ring and slots are sized
// within it; a smaller budget lets several workgroups share a CU).
int plan_create(dd_plan** out, const double* freq_mhz, int32_t nchan, double tsamp_s, const double* dm,
                int32_t ndm, int32_t in_dtype, const dd_tuning* tuning, int64_t lds_cap, bool shared_any) {
  try {
    return create(out, freq_mhz, nchan, tsamp_s, dm, ndm, in_dtype, tuning, lds_cap, shared_any);
  } catch (const std::bad_alloc&) {
    return fail(DD_ERR_INVALID_ARG, "out of host memory");
  }
}

}  // namespace dd

extern "C" {

int dd_plan_create(dd_plan** out, const double* freq_mhz, int32_t nchan, double tsamp_s,
                   const double* dm, int32_t ndm, int32_t in_dtype, const dd_tuning* tuning) {
  return dd::plan_create(out, freq_mhz, nchan, tsamp_s, dm, ndm, in_dtype, tuning, dd::kLdsBytes, false);
}

void dd_plan_destroy(dd_plan* plan) { delete plan; }

int dd_plan_query(const dd_plan* p, int64_t nsamp, dd_plan_info* info) {
  dd::clear_error();
  if (!p || !info) return dd::fail(DD_ERR_INVALID_ARG, "plan and info must be non-NULL");
  std::memset(info, 0, sizeof(*info));
  info->nchan = p->nchan;
  info->ndm = p->ndm;
  info->in_dtype = p->dtype;
  info->maxdelay = p->maxdelay;
  info->nsamp = nsamp;
  info->dms_per_wave = p->tiles.g;
  info->waves = p->tiles.w;
  info->samples_per_lane = p->tiles.s;
  info->chan_stage = p->tiles.cc;
  info->producer_waves = p->launch.prod;
  info->max_span = p->max_span;
  info->kernel_form = p->launch.form;
  info->window_chunks = p->launch.form == dd::kFormRegWin ? p->launch.nch : 0;
  info->launch_copies = p->launch.form == dd::kFormLds ? 4 : p->launch.form == dd::kFormRegWin ? 1 : 0;
  info->launch_buf = p->launch.L;
  info->launch_stage = p->launch.cs;
  info->launch_ring = p->launch.nb;
  info->launch_lds = p->launch.lds;
  if (nsamp <= 0) return dd::fail(DD_ERR_INVALID_ARG, "nsamp must be > 0");
  const int64_t ring_row = dd::ring_len_for(p, nsamp) + dd::ring_mirror(p);
  info->ring_bytes = dd::ring_table_bytes(p) +
                     dd::align_up(ring_row * p->nchan * dd::ring_copies(p) * dd::elem_bytes(p->dtype));
  const int64_t nout = nsamp - p->maxdelay;
  // sized for nsamp outputs: covers a plain call (nout < nsamp) and a stream push (<= block)
  info->workspace_bytes = dd::workspace_layout(p, nsamp).total;
  info->stream_workspace_bytes = dd::workspace_layout(p, nsamp, false).total;
  if (nout <= 0) {
    info->nout = 0;
    return dd::fail(DD_ERR_TOO_SHORT, "nsamp must exceed maxdelay (" + std::to_string(p->maxdelay) + ")");
  }
  info->nout = nout;
  info->adds = (int64_t)p->ndm * p->nchan * nout;
  return DD_OK;
}

int dd_plan_kernel(const dd_plan* p, dd_kernel_info* info) {
  dd::clear_error();
  if (!p || !info) return dd::fail(DD_ERR_INVALID_ARG, "plan and info must be non-NULL");
  std::memset(info, 0, sizeof(*info));
  info->form = p->sh.on ? DD_RUNS_SHARED : p->launch.form;
  info->dms_per_wave = p->sh.on ? dd::kShG : p->tiles.g;
  info->waves = p->sh.on ? p->sh.nw : p->tiles.w;
  info->producer_waves = p->sh.on ? 0 : p->launch.prod;
  info->dms_per_group = p->dms_per_group;
  info->tile_samples = p->sh.on                            ? (int32_t)dd::stat_tile(p)
                       : p->launch.form == dd::kFormDirect ? 64 * p->tiles.s
                                                           : (int32_t)dd::kTile;
  info->lds_bytes = p->sh.on ? p->sh.lds : p->launch.lds;
  return DD_OK;
}

int dd_plan_delays(const dd_plan* p, int32_t* host_out) {
  dd::clear_error();
  if (!p || !host_out) return dd::fail(DD_ERR_INVALID_ARG, "plan and host_out must be non-NULL");
  std::memcpy(host_out, p->delays.data(), p->delays.size() * sizeof(int32_t));
  return DD_OK;
}

int dd_time_binning(const double* freq_mhz, int32_t nchan, double tsamp_s, const double* dm, int32_t ndm,
                    int32_t max_log2, double* dm_diag_out, int32_t* log2_out) {
  dd::clear_error();
  if (!freq_mhz || !dm || !log2_out) return dd::fail(DD_ERR_INVALID_ARG, "freq_mhz, dm and log2_out must be non-NULL");
  if (nchan < 1 || ndm < 1) return dd::fail(DD_ERR_INVALID_ARG, "nchan and ndm must be >= 1");
  if (!(tsamp_s > 0.0) || !std::isfinite(tsamp_s)) return dd::fail(DD_ERR_INVALID_ARG, "tsamp must be finite and > 0");
  if (max_log2 < 0 || max_log2 > 16) return dd::fail(DD_ERR_INVALID_ARG, "max_log2 must be in 0..16");
  std::vector<double> f(freq_mhz, freq_mhz + nchan);
  for (double v : f)
    if (!std::isfinite(v) || !(v > 0.0)) return dd::fail(DD_ERR_INVALID_ARG, "frequencies must be finite and > 0");
  for (int32_t d = 0; d < ndm; ++d) {
    if (!std::isfinite(dm[d]) || dm[d] < 0.0) return dd::fail(DD_ERR_INVALID_ARG, "DMs must be finite and >= 0");
    if (d > 0 && dm[d] < dm[d - 1]) return dd::fail(DD_ERR_INVALID_ARG, "DM trials must be in non-decreasing order");
  }
  // Diagonal DM: one over the largest per-DM delay difference (in samples) between
  // neighbouring channels in frequency order; each double operation rounds once.
  std::sort(f.begin(), f.end());
  double worst = 0.0;
  for (size_t c = 0; c + 1 < f.size(); ++c) {
    const double a = f[c], b = f[c + 1];
    const double per_dm = (kDm * (1.0 / (a * a) - 1.0 / (b * b))) / tsamp_s;
    worst = std::max(worst, per_dm);
  }
  const double diag = worst > 0.0 ? 1.0 / worst : std::numeric_limits<double>::infinity();
  if (dm_diag_out) *dm_diag_out = diag;
  for (int32_t d = 0; d < ndm; ++d) {
    int32_t k = 0;
    while (k < max_log2 && dm[d] > diag * (double)(1 << k)) ++k;
    log2_out[d] = k;
  }
  return DD_OK;
}

}  // extern "C"
