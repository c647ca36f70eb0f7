// Internal declarations shared by the host plan code and the HIP launch code.
#pragma once

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/dedisp.h"

namespace dd {

// Byte alignment of every region inside a workspace or ring.
constexpr int64_t kAlign = 256;
// Output samples per time tile of the dedispersion kernel; also the segment of
// the per-series statistics partials (fixed, so the reduction tree does not
// depend on the launch shape or on batching).
constexpr int64_t kTile = 512;
// Output samples per tile of the direct-read form (16 per lane): two statistics segments.
constexpr int64_t kDirectTile = 1024;
// Output samples per candidate-compaction segment.
constexpr int64_t kStatSeg = 8192;
// LDS of one gfx950 workgroup.
constexpr int64_t kLdsBytes = 160 * 1024;
// Most DMA instructions one wavefront issues per stage (its descriptor table spans four
// 64-lane registers).
constexpr int kMaxDma = 256;
// Most 16-byte DMAs one wavefront issues per stage for FP32 input (one descriptor
// register each); beyond that the 4-byte form is used.
constexpr int kMaxX4 = 16;
// Register-window form (FP32): DM trials per workgroup (8 wavefronts of 8) and channels
// per LDS stage; a wavefront's window holds at most kRwMaxChunks 4-sample chunks.
constexpr int kRwTrials = 64;
constexpr int kRwStage = 8;
constexpr int kRwMaxChunks = 12;
// Kernel forms (dd_tuning.kernel_form / dd_plan_info.kernel_form).
constexpr int kFormLds = 1;     // four shifted copies per channel in LDS, one LDS word per add
constexpr int kFormRegWin = 2;  // one copy per channel, register windows added in VGPR index mode
constexpr int kFormDirect = 3;  // 8-bit input read per trial through the caches, no LDS
// DD_FORM_AUTO picks the register-window form for FP32 plans it fits.
constexpr bool kAutoRegWin = false;

// Launch geometry of the dedispersion kernel.
struct Launch {
  int L;        // samples per (channel, copy) buffer (four copies shifted by 0..3 samples);
                // 32-bit words for 16/32-bit input, bytes for 8-bit input
  int cs;       // channels per stage (a divisor of the wavefront count unless prod > 0)
  int nb;       // stages in the LDS ring
  int nd;       // DMA instructions per stage channel share: per wavefront per stage, or
                // with a producer per channel
  int x4;       // FP32 data arrives by 16-byte DMAs
  int64_t lds;  // bytes
  int prod;     // wavefronts that only issue DMAs (0: every wavefront issues its share)
  int ndw;      // DMA instructions per issuing wavefront per stage (the vmcnt unit)
  int form;     // kFormLds, kFormRegWin or kFormDirect; for kFormRegWin, L is the samples a
                // slot's DMAs cover, nd the 16-byte DMAs per slot, cs = kRwStage; for
                // kFormDirect, L is the samples one wavefront load spans (the tile)
  int nch;      // kFormRegWin: 4-sample chunks per window (6, 8, 10 or 12)
};
Launch choose_launch(int32_t max_span, int nw, int nchan, int cs_req, int64_t lds_cap, int elem_bytes);
// FP32 input with nprod producer wavefronts issuing whole channels; nb = 0 if nothing fits.
Launch choose_launch_prod(int32_t max_span, int nchan, int cs_req, int64_t lds_cap, int nprod);

inline int64_t align_up(int64_t x, int64_t a = kAlign) { return (x + a - 1) / a * a; }

// Shared-sum form (csrc/shared.hip): words of a time tile (4 rows x 63 lanes x 4).
constexpr int kShWords = 1008;
// Trials per wavefront and wavefronts of a CU: the sums of two trials (8-bit input: two totals
// per word) fit 128 registers beside a window, so 16 wavefronts.
constexpr int kShG = 2;
constexpr int kShWaves = 16;
// 16-byte window chunks a wavefront forms per row: lanes past it lack a neighbour's words.
constexpr int sh_row_chunks(int dtype) { return dtype == DD_U8 ? 62 : 63; }
constexpr int kShMaxPat = 15;     // patterns of a bundle
constexpr int kShRecPat = 7;      // patterns of a row's record
constexpr int kShMaxE = 3;        // largest shift of a channel in a pattern
// Channels summed in one running FP32 sum before it joins the series' total, at most: plan_shared
// takes 64 or 32 where the additions of a longer block would round worse than channel by channel
// in blocks of DD_CHAN_BLOCK (bundles of one or two channels, and the first blocks of a series).
// Against that order the error of a total is, emulated at 128 / 160 / 1024 channels, 0.80 / 1.00 /
// 0.82 of it for noise about zero and 0.87 / 1.00 / 0.69 for noise on a level of its own size
// (bundles of mostly two, one and four channels; always 128 channels: 1.33 / 1.66 / 0.84 and 1.98 /
// 2.34 / 0.68).
constexpr int kShFold = 128;
// FP32 plans of fewer channels keep the LDS form, so that their series stay those of every explicit
// tiling, bit for bit: that is what this line is for. Their few, wide channels share less (8 to 14
// patterns per 16 to 32 trials at 64 channels, 4 at 1024), but enough to gain (kShFewClk).
constexpr int kShMinChans = 128;
// The steps of a subband plan (few channels: neighbouring pairs share sums, hardly fours) take the
// shared-sum form where its clocks per trial and 4 channels, estimated, are below this. Up to
// there (92 to 158 over subbands of 8 to 64 channels with 16 and 48 trials per nominal DM) it
// measured 1.1 to 1.8 times as fast as the LDS form, whose 56-trial workgroups are mostly padding
// for a handful of nominal DMs; beyond, windows are many times the tile.
constexpr double kShFewClk = 160.0;
// An 8-bit plan takes the shared-sum form where its estimated clocks per trial (with both forms'
// padding) and 4 channels are below this, else the direct-read form. Wide channels and coarse
// trials at low frequencies leave one channel a bundle and long windows: at 207 to 340 clocks
// (512 to 4096 channels of 120-180 MHz, steps of 0.1 to 0.2) the shared-sum form took 1.16 to 2.1
// times the direct-read form's time, at 193 1.26, at 91 (4096 channels, steps of 0.05) 0.46 to 0.51
// and at 49 (408-428 MHz) 0.26. In between the clocks do not tell the two apart, as the direct-read
// form's time varies too: at 131 to 135 0.71 (130 channels x 200 trials of 0.5), 0.95 and 1.01, at
// 149 to 180 0.76 (1024 channels in no order), 0.91 (4096 x 1150 trials of 0.1), 0.93 and 1.07. The
// line keeps the direct-read form for most of these.
constexpr double kShDirectClk = 140.0;
// An FP32 plan of more than kShLdsTrials trials whose LDS form keeps its best tiling (14 wavefronts
// of 4 trials: windows of up to 1024 words) takes that form where the shared-sum form's estimated
// clocks per trial (with both forms' padding) and 4 channels are kShLdsClk or more: the LDS form
// does not care which channels neighbour each other. 256 and 1024 channels of 408-428 MHz, 500 and
// 1000 trials, 65,536 to 262,144 samples: the shared-sum form takes 1.07 to 1.5 times the LDS form's
// time at 147 to 155 clocks (channels in no order), 0.96 to 1.28 times at 121 to 126 (three in four
// shuffled), 0.81 to 1.12 at 105 (threes), 0.76 to 1.01 at 95 (half shuffled), 0.69 to 0.94 at 84
// (pairs). With fewer trials the LDS form leaves the chip idle on all but long inputs: at 350 trials
// in no order the shared-sum form takes 0.96 to 1.03 times its time on 65,536 samples (1.35 on
// 262,144), at 100 and 200 trials 0.33 to 0.72 on 16,384 and 65,536 (1.0 to 1.2 on 262,144). Where
// longer delays leave it fewer wavefronts it loses at any cost (steps of 0.3 and 0.5 in no order:
// 1.16 to 1.8 times slower; coarser ordered beams 4 to 70 times), and for FP16 input, which it
// takes without producers, everywhere (1.1 times slower at least).
constexpr double kShLdsClk = 112.0;
constexpr int kShLdsTrials = 384;
constexpr int kShMaxBundles = 3;  // bundles of a stage
constexpr int kShBlock = 136;     // bytes of code per pattern block
constexpr int kShSpare = 1024;    // LDS bytes before the stages: where lanes without a chunk write
// A stage's records: per wavefront one to add from and one to form from.
// Adding, kShAddInts ints: the LDS offsets of its trials' windows (their 16-byte boundaries) in
// the stage's bundles, bundle-major; the words their starts lie past those, 2 bits each; the last
// unit | fold << 8.
// Forming a row, kShFormInts ints: the window start of the bundle's first channel and the bytes
// from there to the other three's; the first channel; the LDS offset and the bytes of the first
// of the record's patterns' sums; row | channels << 8 | 4096 if they run down from the first; 8
// bytes of pattern numbers, 64 past the last; the samples past the first channel's window start
// that the row may load; the ints from the group's first record to the wavefront's next row of
// the stage, or 0. No channels: no row. A group's stages are followed by kShPad of no use, and
// the first group's preceded by one, so that records can be loaded ahead unchecked.
constexpr int kShPad = 3;
constexpr int kShMaxOff = 8192;  // samples between the window starts of a bundle's channels
constexpr int kShAddInts = 8;
constexpr int kShFormInts = 12;
constexpr int kShRecInts = kShAddInts + kShFormInts;
constexpr int kShMaxRows = 200;  // rows of a bundle
// Samples past a window's start that row `row` may load.
constexpr int sh_reach(int dtype, int row) {
  return 4 * ((row + 1) * sh_row_chunks(dtype) + 64) + 8 + (dtype == DD_U8 ? kShWords : 0);
}
constexpr int sh_stage_ints(int nw) { return kShRecInts * nw; }
static_assert(kShG * kShMaxBundles <= 6, "a wavefront's units fit its record");
struct Shared {
  bool on = false;
  int32_t nw = 0;      // wavefronts per workgroup
  int32_t mirror = 0;  // samples past a window's start that a unit may read
  int64_t lds = 0;     // bytes (the spare slot and two stages)
  double stages = 0;   // per group, on average
};

struct Tiles {
  int32_t g;   // DM trials per wavefront
  int32_t w;   // wavefronts per workgroup (each on its own G trials)
  int32_t s;   // output samples per lane (fixed: 8, two chunks of 4)
  int32_t cc;  // channels staged into LDS per barrier pair (0 = automatic)
  int32_t pw;  // producer wavefronts requested: -1 none, 0 automatic, 1 one
};

}  // namespace dd

struct dd_plan {
  int32_t nchan = 0, ndm = 0, dtype = DD_F32;
  double tsamp = 0.0;
  std::vector<double> freq, dm;
  std::vector<int32_t> delays;      // [nchan][ndm], Eq. deltaTEq
  int32_t maxdelay = 0;
  dd::Tiles tiles{};
  int32_t dms_per_group = 0;        // g * w
  int32_t ngroups = 0;
  int32_t ndm_pad = 0;              // ngroups * dms_per_group
  // device table: [nchan][ndm_pad] LDS byte offset of each trial's first chunk inside its
  // channel slot (padded trials repeat the last DM), then [ngroups][nchan] group first delays
  std::vector<int32_t> dev_table;
  int32_t max_span = 0;             // max over channels and groups of the in-group delay spread
  dd::Launch launch{};               // kernel geometry (fixed at plan time: the offsets depend on it)
  uint64_t id = 0;
  // Plans without a tuning run in the shared-sum form where it pays (sh.on); tiles and launch
  // then describe the form the plan would otherwise take, and dms_per_group, ngroups and
  // dev_table belong to the shared-sum form.
  dd::Shared sh;
};

struct dd_stream {
  const dd_plan* plan = nullptr;
  int64_t block = 0;        // largest block accepted
  int64_t ring_len = 0;     // R: samples per channel in the ring
  int64_t ring_row = 0;     // R + mirror: a channel row; [R, ring_row) repeats [0, ring_row - R)
  void* ring = nullptr;     // device: [table | ring data]
  int64_t received = 0;     // total samples appended
  int64_t next_seq = 0;
  int64_t emitted = 0;      // global output times already produced ([0, emitted))
  int64_t pending_t0 = 0, pending_n = 0;  // window appended but not yet dedispersed
  bool gap_fill = false;    // missing blocks become zeros instead of DD_ERR_SEQUENCE
};

namespace dd {

// Thread-local error message helpers (implemented in plan.cpp).
int fail(int code, const std::string& msg);
void clear_error();
// dd_plan_create with the LDS bytes one workgroup may take (csrc/plan.cpp), and whether FP32 plans
// below kShMinChans channels may take the shared-sum form (where it is cheaper: kShFewClk);
// dd_plan_create passes kLdsBytes and false.
int plan_create(dd_plan** out, const double* freq_mhz, int32_t nchan, double tsamp_s, const double* dm,
                int32_t ndm, int32_t in_dtype, const dd_tuning* tuning, int64_t lds_cap, bool shared_any);

// Workspace layout for one dd_dedisperse call.
struct WsLayout {
  int64_t table_off, table_bytes;
  int64_t part_off;    // double [ndm][ntile][2]: sum x, sum x^2 per 512-sample tile
  int64_t thr_off;     // double [ndm][3]: mean, rms, threshold
  int64_t cnt_off;     // int32 [ndm][nseg]
  int64_t offs_off;    // int64 [ndm][nseg]
  int64_t tail_off;    // 8-bit input: copy of the last tail_bytes of the input, then as many
  int64_t tail_bytes;  // bytes of padding (a window starting in the copy reads at most that far)
  int64_t quad_off;    // direct-read form, linear input: the four shifted copies of the input
  int64_t quad_bytes;
  int64_t nseg;        // candidate segments
  int64_t ntile;       // statistics segments
  int64_t total;
};
// Workspace of a call on n samples: linear input (dd_dedisperse) or a stream push of at
// most n samples (no region for the direct-read form's copies, which the ring holds).
WsLayout workspace_layout(const dd_plan* p, int64_t n, bool linear = true);
int64_t ring_table_bytes(const dd_plan* p);
// Samples after a ring row's R that mirror its start, so no channel window the kernel
// reads (at most launch.L + 3 samples from any start in [0, R), or the shared-sum form's
// sh.mirror) wraps. A mirror longer than R is filled for R samples only: what lies past them no
// stored output of a window looks at.
inline int64_t ring_mirror(const dd_plan* p) {
  return std::max<int64_t>((int64_t)p->launch.L + 64, p->sh.on ? p->sh.mirror : 0);
}
inline int64_t ring_len_for(const dd_plan* p, int64_t block) { return align_up(block + (int64_t)p->maxdelay, 64); }
// Rows a stream's ring keeps per channel: the direct-read form keeps its four shifted copies.
inline bool runs_direct(const dd_plan* p) { return p->launch.form == kFormDirect && !p->sh.on; }
inline int64_t ring_copies(const dd_plan* p) { return runs_direct(p) ? 4 : 1; }
// Statistics partials per series: one per time tile of the kernel that runs.
inline int64_t stat_tile(const dd_plan* p) { return !p->sh.on ? kTile : p->dtype == DD_U8 ? 2 * kShWords : kShWords; }
inline int64_t stat_tiles(const dd_plan* p, int64_t nout) { return (nout + stat_tile(p) - 1) / stat_tile(p); }
int64_t elem_bytes(int32_t dtype);
// kFormRegWin device table: [ngroups][nchan] group first delays, then from this int32
// offset [ngroups][nchan][8 wavefronts] int4 {window byte offset, trial indices 0-3, 4-7, 0},
// followed by kRwStage - 1 channels of zero records.
bool plan_regwin(dd_plan* p, int64_t lds_cap);
inline int64_t rw_meta_offset(const dd_plan* p) { return ((int64_t)p->ngroups * p->nchan + 3) / 4 * 4; }
// Input view: linear rows, or a per-channel ring of ring_len samples in which
// window position p lives at (win0 + p) mod ring_len. A ring row continues past
// ring_len with a mirror of its start, so a window read from any start in
// [0, ring_len) is contiguous.
struct InView {
  const void* ptr;
  int64_t row_stride;  // elements between channel rows (ring: ring_len + mirror)
  int64_t nvalid;      // window positions [0, nvalid) hold data
  int64_t ring_len;    // 0 for linear input
  int64_t win0;        // ring only: global sample of window position 0
};
// Launch of the register-window kernel for nout outputs (statistics partials into part
// when non-null); defined with the kernel.
int launch_regwin(const dd_plan* p, const InView& in, const int32_t* d_table, int64_t nout, float* out,
                  int64_t out_stride, double* part, void* stream);
// Shared-sum form: fills sh, the groups and the device table and returns true, or leaves the
// plan as it is and returns false where that form does not fit or is estimated to take max_cost
// clocks or more per trial and 4 channels of a tile.
bool plan_shared(dd_plan* p, int64_t lds_cap, double max_cost);
int launch_shared(const dd_plan* p, const InView& in, const int32_t* d_table, int64_t nout, float* out,
                  int64_t out_stride, double* part, void* stream);
// One shared-sum item of a batched call; the items of one input type and workgroup size run in
// one launch over all their units.
struct SharedItem {
  const dd_plan* plan;
  InView in;
  const int32_t* table;
  int64_t nout;
  float* out;
  int64_t out_stride;
  double* part;
};
// Bytes of device descriptors a batched shared-sum launch of n items uploads.
int64_t shared_batch_desc_bytes(int32_t n);
int launch_shared_batch(const std::vector<SharedItem>& items, void* d_desc, int64_t desc_bytes, void* stream);
// Direct-read form (8-bit input): device table [nchan][ndm_pad] of plain delays (padded trials
// repeat the last DM). Fills the plan's tiles, groups, launch and table.
int plan_direct(dd_plan* p, const Tiles& t);
// Bytes per copy row of the direct-read form's copies of an nsamp-sample linear input: the
// last tile's windows (two sub-tiles at most) read at most 2 kDirectTile bytes past the
// last sample's position.
inline int64_t direct_quad_row(int64_t nsamp) { return align_up(nsamp + 2 * kDirectTile + 64, 64); }
// Linear input: writes the copies into quad_ws first. Ring input: in.ptr is the ring's
// copies, in.row_stride their row length.
int launch_direct(const dd_plan* p, const InView& in, const int32_t* d_table, int64_t nout, float* out,
                  int64_t out_stride, double* part, void* quad_ws, void* stream);
// One item of a batched direct-read launch (what launch_direct takes).
struct DirectItem {
  const dd_plan* plan;
  InView in;
  const int32_t* table;
  int64_t nout;
  float* out;
  int64_t out_stride;
  double* part;
  void* quad_ws;
};
// Bytes of device descriptors a batched direct-read launch of n items uploads.
int64_t direct_batch_desc_bytes(int32_t n);
int launch_direct_batch(const std::vector<DirectItem>& items, void* d_desc, int64_t desc_bytes, void* stream);
// n samples of a block (zeros when blk is null) into a direct-read stream ring of copy rows
// of lq bytes, starting at ring position pos0.
int append_direct(const dd_plan* p, const void* blk, int64_t in_stride, int64_t n, void* ring, int64_t lq,
                  int64_t ring_len, int64_t pos0, void* stream);
// Exclusive scan of n int32 counts into offs[n] (int64) and their total into *total, by
// many blocks in three launches that use no memory beyond offs (csrc/dedisp.hip).
int launch_count_scan(const int32_t* cnt, int64_t n, int64_t* offs, int64_t* total, void* stream);

}  // namespace dd
