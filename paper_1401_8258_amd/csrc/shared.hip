// Shared-sum form (gfx950, wave64): Eq. bruteEquation with the sums that several DM trials
// have in common formed once.
//
// Within a few neighbouring channels the delays of the trials of one DM group differ by a
// handful of patterns only: for channels c..c+3 the relative delays delta[c+j][d] -
// delta[c][d] of 36 consecutive trials take about 4 distinct values on the 408-428 MHz band.
// For every such bundle of up to 4 channels the workgroup forms each pattern's sum
//   S_p[x] = sum_j A[c_j][base_j + e_pj + x]      (window positions x, e_pj in 0..3)
// once in LDS, and every trial adds one S_p at its own offset instead of 4 channels. The
// sums are the same channels' samples; FP32 sums them inside the bundle in order, bundles in
// order inside blocks of DD_CHAN_BLOCK channels, blocks in order, so no sum has more or
// larger partial sums than channel by channel. 8-bit codes are exact integers either way.
//
// Work unit: one time tile x one group of trials. A tile is 1008 words: 4 rows of 63 lanes of
// 4 words. For FP32 and FP16 a word is one FP32 sample; for 8-bit input a word holds two
// 16-bit sums, of samples t and t + 1008 (so a shift of the window is a shift of words for
// both, and one 32-bit add serves two outputs), and the tile is 2016 samples. Lane 63 of a
// row holds the first words of the next row: a trial whose window starts s = 1..3 words past
// a 16-byte boundary takes its last words from the next lane by DPP, so one copy of each sum
// serves every alignment with four conflict-free ds_read_b128 per 16 words.
//
// A stage is up to four bundles, double-buffered in LDS, with one barrier a stage. Every
// wavefront adds the stage's sums to its trials and forms its share of the next stage's, in
// rows of 62-63 lanes x 4 window words of one bundle, from raw samples loaded into registers
// a stage earlier. Both parts are bound by instruction issue (a wavefront alone issues one
// instruction in about 6 clocks), so the forming is spread over all of them.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <cstdint>
#include <string>

#include "dd_device.h"
#include "dd_internal.h"

namespace {

using dd::block_barrier;
using dd::ci32_t;

// input and table reads are global (not flat) loads: a flat load would be waited on with LDS
#define DD_GLOBAL __attribute__((address_space(1)))
typedef const DD_GLOBAL char* gptr_t;
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u2u_t __attribute__((ext_vector_type(2), aligned(4)));
typedef int32_t i4_t __attribute__((ext_vector_type(4)));

constexpr int kRow = 63;          // lanes of a row with outputs of their own
constexpr int kRowB = kRow * 16;  // bytes from one row's lane to the next row's
static_assert(kRowB == 1008, "the row offsets of the window reads are written out");

struct ShParams {
  const void* in;
  int64_t row_stride, nvalid, win0;
  uint32_t ring, limit;  // ring length (0: linear); samples of a row that may be loaded
  const int32_t* tab;
  float* out;
  double* part;
  int64_t out_stride, nout, nitems, ntile;
  int32_t ngroups, ndm, per_group, nw;
};

// Lane l gets lane l + 1's value.
__device__ __forceinline__ uint32_t next_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xF, 0xF, true);
}

template <int DT>
struct Word {
  using T = float;
};
template <>
struct Word<DD_U8> {
  using T = uint32_t;
};

// ------------------------------------------------------------------ forming the sums

template <int DT>
constexpr int kEB = DT == DD_F32 ? 4 : DT == DD_F16 ? 2 : 1;
template <int DT>
constexpr int kDw = DT == DD_F32 ? 4 : DT == DD_F16 ? 2 : 1;  // dwords of 4 samples
template <int DT>
constexpr int kRawN = DT == DD_F32 ? 4 : 2;  // raw dwords a lane holds per channel

// A row of one bundle, wave-uniform, and the raw samples it is formed from.
template <int DT>
struct Row {
  int live, slot, dst, row, first;      // bytes per pattern, LDS offset, row, its codes' first lane
  uint32_t sh;                          // per channel 2 bits: bytes its first sample lies past the dword
  uint32_t v[4][kRawN<DT>];
};

// A stage's record (lane l: four ints, dd_internal.h) and its window starts: lane 16 b + j
// holds channel j's of bundle b.
struct Stage {
  i4_t meta;
  uint64_t start;
  uint64_t safe;  // lanes whose whole window lies inside the input
};

__device__ __forceinline__ int lane_w(const Stage& f, int l) { return __builtin_amdgcn_readlane(f.meta.w, l); }
__device__ __forceinline__ int stage_rows(const Stage& f) { return lane_w(f, dd::kShLaneRows); }

// Window starts: sample wbase + offset of its channel, less ring_len past the ring's end (the
// difference wraps to a large number before it; ring_len is 0 for linear input).
template <int DT>
__device__ __forceinline__ void open_stage(const ShParams& P, uint32_t wbase, Stage& f) {
  constexpr int EB = kEB<DT>;
  const uint32_t s0 = wbase + (uint32_t)f.meta.y, s1 = s0 - P.ring;
  const uint32_t s = s1 < s0 ? s1 : s0;
  const uint64_t stride = (uint64_t)P.row_stride * EB;
  const uint64_t at = (uint64_t)(uint32_t)f.meta.z * (uint32_t)stride + (uint64_t)P.in;
  f.start = at + ((uint64_t)((uint32_t)f.meta.z * (uint32_t)(stride >> 32)) << 32) + (uint64_t)s * EB;
  const int reach = lane_w(f, dd::kShLaneReach);  // samples past its start a window may load
  f.safe = __ballot(s + (uint32_t)reach <= P.limit);
}

// This lane's dwords of one channel, from the scalar window start p and the lane's offset vo.
template <int DT>
__device__ __forceinline__ void load_words(gptr_t p, uint32_t vo, uint32_t (&v)[kRawN<DT>]) {
  if constexpr (DT == DD_F32) {
    const u4u_t q = *(const DD_GLOBAL u4u_t*)(p + vo);
    v[0] = q.x, v[1] = q.y, v[2] = q.z, v[3] = q.w;
  } else if constexpr (DT == DD_F16) {
    const u2u_t q = *(const DD_GLOBAL u2u_t*)(p + vo);
    v[0] = q.x, v[1] = q.y;
  } else {
    v[0] = *(const DD_GLOBAL uint32_t*)(p + vo);
    v[1] = *(const DD_GLOBAL uint32_t*)(p + dd::kShWords + vo);
  }
}

// Row t of the stage: its header, and its raw samples' loads: lane l of row r of a bundle loads
// the 4 window positions 4 (r VC + l) .. + 3 of every channel (8-bit input: also those 1008
// samples later), in whole dwords; channels the bundle lacks are zeros. Where a window would
// pass the last sample, each dword is clamped to that of the last sample: positions past it
// are used by no stored output. The usual case is one block of loads with scalar starts: a
// choice per channel, or starts in vector registers, made the compiler wait for earlier loads
// between them (54.2 -> XX ms on the full FP32 workload).
template <int DT>
__device__ __forceinline__ void load_row(const ShParams& P, const Stage& f, int t, int lane, Row<DT>& r) {
  constexpr int VC = dd::sh_row_chunks(DT);
  constexpr int EB = kEB<DT>;
  r.live = t < stage_rows(f);
  if (!r.live) return;
  // the row's bundle, by the rows up to each (bytes; 255 past the last bundle)
  const int ends = lane_w(f, dd::kShLaneEnds);
  const int b = (t >= (ends & 255)) + (t >= ((ends >> 8) & 255));
  static_assert(dd::kShMaxBundles == 3, "two ends tell three bundles apart");
  const int first = 16 * b;
  r.row = b ? t - ((ends >> (8 * b - 8)) & 255) : t;
  r.slot = lane_w(f, first + 1);
  r.dst = lane_w(f, first + 2);
  r.first = first;
  const int m = lane_w(f, first);
  uint64_t start[4];
  r.sh = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)f.start, first + j);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(f.start >> 32), first + j);
    start[j] = (lo & ~3u) | (uint64_t)hi << 32;
    if (DT != DD_F32) r.sh |= (lo & 3u) << (2 * j);
  }
  uint32_t vo = (uint32_t)(r.row * VC + lane) * (4 * kDw<DT>);
  const bool whole = ((f.safe >> first) & 15) == 15;
  if (whole && m == 4) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      asm volatile("" : "+v"(vo));  // a 32-bit offset here, so that the load takes the scalar start
      load_words<DT>((gptr_t)start[j], vo, r.v[j]);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j >= m) {
#pragma unroll
        for (int i = 0; i < kRawN<DT>; ++i) r.v[j][i] = 0;
      } else if (whole) {
        asm volatile("" : "+v"(vo));
        load_words<DT>((gptr_t)start[j], vo, r.v[j]);
      } else {
        // a window starts before the last sample of its channel, so lim is not negative
        const uint64_t row = (uint64_t)P.in +
                             (uint64_t)((int64_t)__builtin_amdgcn_readlane(f.meta.z, first + j) * P.row_stride * EB);
        const uint32_t lim = (uint32_t)(((row + (uint64_t)(P.nvalid * EB - 1)) & ~(uint64_t)3) - start[j]);
#pragma unroll
        for (int i = 0; i < kRawN<DT>; ++i) {
          const uint32_t o = vo + (DT == DD_U8 ? i * dd::kShWords : 4 * i);
          r.v[j][i] = *(const DD_GLOBAL uint32_t*)((gptr_t)start[j] + (o < lim ? o : lim));
        }
      }
    }
  }
}

// Channel j's words at this lane's 4 window positions.
template <int DT>
__device__ __forceinline__ void words(const Row<DT>& r, int j, typename Word<DT>::T (&w)[4]) {
  const uint32_t sh = (r.sh >> (2 * j)) & 3u;
  if constexpr (DT == DD_F32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = __uint_as_float(r.v[j][i]);
  } else if constexpr (DT == DD_F16) {
    const uint32_t d0 = r.v[j][0], d1 = r.v[j][1], d2 = next_lane(d0);
    const uint32_t a[2] = {__builtin_amdgcn_alignbyte(d1, d0, sh), __builtin_amdgcn_alignbyte(d2, d1, sh)};
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = __half2float(__ushort_as_half((unsigned short)(i & 1 ? a[i / 2] >> 16 : a[i / 2] & 0xFFFFu)));
  } else {
    const uint32_t lo = __builtin_amdgcn_alignbyte(next_lane(r.v[j][0]), r.v[j][0], sh);
    const uint32_t hi = __builtin_amdgcn_alignbyte(next_lane(r.v[j][1]), r.v[j][1], sh);
    // v_perm bytes 0-3: second operand (sample t), 4-7: first operand (sample t + 1008)
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_perm(hi, lo, i | 0x0C00u | ((4u + i) << 16) | 0x0C000000u);
  }
}

// The pattern sums of one row into LDS. Sum i is w[0] + the words w[1], w[2], w[3] shifted by
// e1, e2, e3: word k of a lane's 4, shifted by e, is its own word k + e, or word k + e - 4 of
// the next lane (by DPP; the last lane has none, and its sums go to the spare slot). Each of
// the 64 (e1, e2, e3) is a block of its own, kShBlock bytes of 12 adds (8 bytes each), the LDS
// write and a jump to the next pattern's block, whose offset lane `first + i` of codes holds;
// after the last one comes the offset past the table. A jump leaves more than the two
// instructions a DPP operand has to be older than.
#define DD_DPP1 " wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
#define DD_FORM_ADD(n, E, U0, U1, U2, U3, W0, W1, W2, W3)                                          \
  ".if " E " == 0\n\t"                                                                            \
  n "_e64 v112, " U0 ", " W0 "\n\t" n "_e64 v113, " U1 ", " W1 "\n\t"                                 \
  n "_e64 v114, " U2 ", " W2 "\n\t" n "_e64 v115, " U3 ", " W3 "\n\t"                                 \
  ".elseif " E " == 1\n\t"                                                                        \
  n "_e64 v112, " U0 ", " W1 "\n\t" n "_e64 v113, " U1 ", " W2 "\n\t"                                 \
  n "_e64 v114, " U2 ", " W3 "\n\t" n "_dpp v115, " W0 ", " U3 DD_DPP1                                 \
  ".elseif " E " == 2\n\t"                                                                        \
  n "_e64 v112, " U0 ", " W2 "\n\t" n "_e64 v113, " U1 ", " W3 "\n\t"                                 \
  n "_dpp v114, " W0 ", " U2 DD_DPP1 n "_dpp v115, " W1 ", " U3 DD_DPP1                                \
  ".else\n\t"                                                                                     \
  n "_e64 v112, " U0 ", " W3 "\n\t" n "_dpp v113, " W0 ", " U1 DD_DPP1                                 \
  n "_dpp v114, " W1 ", " U2 DD_DPP1 n "_dpp v115, " W2 ", " U3 DD_DPP1                                \
  ".endif\n\t"
#define DD_FORM_GO                               \
  "v_readlane_b32 %[t], %[codes], %[i]\n\t"      \
  "s_add_u32 %[i], %[i], 1\n\t"                  \
  "s_add_u32 vcc_lo, %[tlo], %[t]\n\t"           \
  "s_addc_u32 vcc_hi, %[thi], 0\n\t"             \
  "s_setpc_b64 vcc\n\t"
#define DD_FORM(n)                                                                                 \
  asm volatile(                                                                                    \
      "s_getpc_b64 vcc\n"                                                                          \
      "Ldd_pc_%=:\n\t"                                                                             \
      "s_add_u32 %[tlo], vcc_lo, Ldd_tab_%=-Ldd_pc_%=\n\t"                                         \
      "s_addc_u32 %[thi], vcc_hi, 0\n\t"                                                           \
      DD_FORM_GO                                                                                   \
      "Ldd_tab_%=:\n\t"                                                                            \
      ".irp e3, 0, 1, 2, 3\n\t"                                                                    \
      ".irp e2, 0, 1, 2, 3\n\t"                                                                    \
      ".irp e1, 0, 1, 2, 3\n\t"                                                                    \
      DD_FORM_ADD(n, "\\e1", "%5", "%6", "%7", "%8", "%9", "%10", "%11", "%12")                    \
      DD_FORM_ADD(n, "\\e2", "v112", "v113", "v114", "v115", "%13", "%14", "%15", "%16")           \
      DD_FORM_ADD(n, "\\e3", "v112", "v113", "v114", "v115", "%17", "%18", "%19", "%20")           \
      "ds_write_b128 %[dst], v[112:115]\n\t"                                                       \
      "v_add_u32_e32 %[dst], %[step], %[dst]\n\t"                                                  \
      DD_FORM_GO                                                                                   \
      ".endr\n\t"                                                                                  \
      ".endr\n\t"                                                                                  \
      ".endr\n"                                                                                    \
      "Ldd_end_%=:\n\t"                                                                            \
      ".if Ldd_end_%=-Ldd_tab_%= != 64*%c[block]\n\t.error \"block size\"\n\t.endif"               \
      : [dst] "+v"(dst), [i] "+s"(i), [t] "=&s"(t), [tlo] "=&s"(tlo), [thi] "=&s"(thi)             \
      : "v"(w[0][0]), "v"(w[0][1]), "v"(w[0][2]), "v"(w[0][3]), "v"(w[1][0]), "v"(w[1][1]),        \
        "v"(w[1][2]), "v"(w[1][3]), "v"(w[2][0]), "v"(w[2][1]), "v"(w[2][2]), "v"(w[2][3]),        \
        "v"(w[3][0]), "v"(w[3][1]), "v"(w[3][2]), "v"(w[3][3]), [codes] "v"(codes),                \
        [step] "v"(step), [block] "i"(dd::kShBlock)                                                \
      : "scc", "vcc", "memory", "v112", "v113", "v114", "v115")
__device__ __forceinline__ void form(const float (&w)[4][4], int codes, int i, uint32_t dst, uint32_t step) {
  uint32_t t, tlo, thi;
  DD_FORM("v_add_f32");
}
__device__ __forceinline__ void form(const uint32_t (&w)[4][4], int codes, int i, uint32_t dst, uint32_t step) {
  uint32_t t, tlo, thi;
  DD_FORM("v_add_u32");
}

// Forms row r: the words of its channels, then the sums.
// Lanes without a window chunk of their own write to the spare slot.
template <int DT>
__device__ __forceinline__ void form_row(const Row<DT>& r, int codes, int lane, uint32_t lds, uint32_t spare) {
  using T = typename Word<DT>::T;
  constexpr int VC = dd::sh_row_chunks(DT);
  T w[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) words<DT>(r, j, w[j]);
  const int idx = r.row * VC + lane;
  const bool mine = lane < VC && idx * 16 < r.slot;
  form(w, codes, __builtin_amdgcn_readfirstlane(r.first), mine ? lds + r.dst + 16 * idx : spare + 16 * lane, mine ? r.slot : 0);
}

__device__ __forceinline__ void stage_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wavefront's LDS reads and writes are done
  block_barrier();
}

// ------------------------------------------------------------------ adding them

// The adds of one row of a trial's window, registers v[W0:W3], for the four shifts of the
// window start past its 16-byte boundary (as in DD_FORM_ADD, in place).
#define DD_OWN(n, A, W) n "_e32 %" #A ", v" #W ", %" #A "\n\t"
#define DD_NEXT(n, A, W) n "_dpp %" #A ", v" #W ", %" #A " wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"
#define DD_SH0(n, A0, A1, A2, A3, W0, W1, W2, W3) DD_OWN(n, A0, W0) DD_OWN(n, A1, W1) DD_OWN(n, A2, W2) DD_OWN(n, A3, W3)
#define DD_SH1(n, A0, A1, A2, A3, W0, W1, W2, W3) DD_OWN(n, A0, W1) DD_OWN(n, A1, W2) DD_OWN(n, A2, W3) DD_NEXT(n, A3, W0)
#define DD_SH2(n, A0, A1, A2, A3, W0, W1, W2, W3) DD_OWN(n, A0, W2) DD_OWN(n, A1, W3) DD_NEXT(n, A2, W0) DD_NEXT(n, A3, W1)
#define DD_SH3(n, A0, A1, A2, A3, W0, W1, W2, W3) DD_OWN(n, A0, W3) DD_NEXT(n, A1, W0) DD_NEXT(n, A2, W1) DD_NEXT(n, A3, W2)
// Row by row: wait for the row, add it, start the same row of the next unit's window.
#define DD_WAIT "s_waitcnt lgkmcnt(3)\n\t"
#define DD_ROWS(SH, n, ...) DD_ROWS_(SH, n, __VA_ARGS__)
#define DD_ROWS_(SH, n, A0, A1, A2, A3, A4, A5, A6, A7, A8, A9, A10, A11, A12, A13, A14, A15)             \
  DD_WAIT SH(n, A0, A1, A2, A3, 112, 113, 114, 115) "ds_read_b128 v[112:115], %[va]\n\t"                 \
  DD_WAIT SH(n, A4, A5, A6, A7, 116, 117, 118, 119) "ds_read_b128 v[116:119], %[va] offset:1008\n\t"     \
  DD_WAIT SH(n, A8, A9, A10, A11, 120, 121, 122, 123) "ds_read_b128 v[120:123], %[va] offset:2016\n\t"   \
  DD_WAIT SH(n, A12, A13, A14, A15, 124, 125, 126, 127) "ds_read_b128 v[124:127], %[va] offset:3024\n\t"
// One unit (a trial's window of one bundle): s0 = its shift, then the next unit's offset in s1.
// A register that a read in flight will fill is read only after the wait for it.
#define DD_UNIT(n, K, ...)                      \
  "s_add_u32 %[i], %[i], 1\n\t"                 \
  "v_readlane_b32 %[s1], %[meta], %[i]\n\t"     \
  "s_and_b32 %[s2], %[s1], -16\n\t"             \
  "v_add_u32 %[va], %[s2], %[base]\n\t"         \
  "s_cmp_lt_u32 %[s0], 2\n\t"                   \
  "s_cbranch_scc0 Ldd_c" #K "_%=\n\t"           \
  "s_cmp_eq_u32 %[s0], 0\n\t"                   \
  "s_cbranch_scc0 Ldd_b" #K "_%=\n\t"           \
  DD_ROWS(DD_SH0, n, __VA_ARGS__)               \
  "s_branch Ldd_e" #K "_%=\n"                   \
  "Ldd_b" #K "_%=:\n\t"                         \
  DD_ROWS(DD_SH1, n, __VA_ARGS__)               \
  "s_branch Ldd_e" #K "_%=\n"                   \
  "Ldd_c" #K "_%=:\n\t"                         \
  "s_cmp_eq_u32 %[s0], 2\n\t"                   \
  "s_cbranch_scc0 Ldd_d" #K "_%=\n\t"           \
  DD_ROWS(DD_SH2, n, __VA_ARGS__)               \
  "s_branch Ldd_e" #K "_%=\n"                   \
  "Ldd_d" #K "_%=:\n\t"                         \
  DD_ROWS(DD_SH3, n, __VA_ARGS__)               \
  "Ldd_e" #K "_%=:\n\t"                         \
  "s_and_b32 %[s0], %[s1], 3\n\t"
// The last unit: nothing left to read.
#define DD_LAST_ROWS(SH, n, ...) DD_LAST_ROWS_(SH, n, __VA_ARGS__)
#define DD_LAST_ROWS_(SH, n, A0, A1, A2, A3, A4, A5, A6, A7, A8, A9, A10, A11, A12, A13, A14, A15)      \
  "s_waitcnt lgkmcnt(3)\n\t" SH(n, A0, A1, A2, A3, 112, 113, 114, 115)                                 \
  "s_waitcnt lgkmcnt(2)\n\t" SH(n, A4, A5, A6, A7, 116, 117, 118, 119)                                 \
  "s_waitcnt lgkmcnt(1)\n\t" SH(n, A8, A9, A10, A11, 120, 121, 122, 123)                               \
  "s_waitcnt lgkmcnt(0)\n\t" SH(n, A12, A13, A14, A15, 124, 125, 126, 127)
#define DD_LAST(n, ...)                         \
  "Ldd_last_%=:\n\t"                            \
  "s_cmp_lt_u32 %[s0], 2\n\t"                   \
  "s_cbranch_scc0 Ldd_lc_%=\n\t"                \
  "s_cmp_eq_u32 %[s0], 0\n\t"                   \
  "s_cbranch_scc0 Ldd_lb_%=\n\t"                \
  DD_LAST_ROWS(DD_SH0, n, __VA_ARGS__)          \
  "s_branch Ldd_le_%=\n"                        \
  "Ldd_lb_%=:\n\t"                              \
  DD_LAST_ROWS(DD_SH1, n, __VA_ARGS__)          \
  "s_branch Ldd_le_%=\n"                        \
  "Ldd_lc_%=:\n\t"                              \
  "s_cmp_eq_u32 %[s0], 2\n\t"                   \
  "s_cbranch_scc0 Ldd_ld_%=\n\t"                \
  DD_LAST_ROWS(DD_SH2, n, __VA_ARGS__)          \
  "s_branch Ldd_le_%=\n"                        \
  "Ldd_ld_%=:\n\t"                              \
  DD_LAST_ROWS(DD_SH3, n, __VA_ARGS__)          \
  "Ldd_le_%=:"
// A stage's bundles: units (bundle, trial) in order, meta lane `unit` holding the window's
// LDS byte offset and shift; n is the last unit. All of the window registers' reads end in
// here: one asm block, so that nothing else touches them while a read is in flight.
#define DD_STAGE(n)                                 \
  "s_mov_b32 %[i], 0\n\t"                           \
  "v_readlane_b32 %[s1], %[meta], 0\n\t"            \
  "s_and_b32 %[s2], %[s1], -16\n\t"                 \
  "s_and_b32 %[s0], %[s1], 3\n\t"                   \
  "v_add_u32 %[va], %[s2], %[base]\n\t"             \
  "ds_read_b128 v[112:115], %[va]\n\t"              \
  "ds_read_b128 v[116:119], %[va] offset:1008\n\t"  \
  "ds_read_b128 v[120:123], %[va] offset:2016\n\t"  \
  "ds_read_b128 v[124:127], %[va] offset:3024\n"    \
  "Ldd_l_%=:\n\t"                                   \
  DD_UNIT(n, 0, DD_U0)                              \
  "s_cmp_ge_u32 %[i], %[n]\n\t"                     \
  "s_cbranch_scc1 Ldd_last_%=\n\t"                  \
  DD_UNIT(n, 1, DD_U1)                              \
  "s_branch Ldd_l_%=\n"                             \
  DD_LAST(n, DD_U1)
#define DD_ACC(g)                                                                                          \
  "+v"(acc[g][0]), "+v"(acc[g][1]), "+v"(acc[g][2]), "+v"(acc[g][3]), "+v"(acc[g][4]), "+v"(acc[g][5]),    \
      "+v"(acc[g][6]), "+v"(acc[g][7]), "+v"(acc[g][8]), "+v"(acc[g][9]), "+v"(acc[g][10]),                \
      "+v"(acc[g][11]), "+v"(acc[g][12]), "+v"(acc[g][13]), "+v"(acc[g][14]), "+v"(acc[g][15])
#define DD_STAGE_TMP [va] "=&v"(va), [i] "=&s"(i), [s0] "=&s"(s0), [s1] "=&s"(s1), [s2] "=&s"(s2)
#define DD_STAGE_USE [meta] "v"(meta), [base] "v"(base), [n] "s"(n)
#define DD_STAGE_CLOBBER                                                                                  \
  "scc", "memory", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121", "v122", \
      "v123", "v124", "v125", "v126", "v127"

#define DD_U0 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15
#define DD_U1 16, 17, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31
static_assert(dd::kShG == 2, "the stage's code walks two trials");
__device__ __forceinline__ void add_stage(float (&acc)[2][16], int meta, uint32_t base, int n) {
  uint32_t va, i, s0, s1, s2;
  asm volatile(DD_STAGE("v_add_f32")
               : DD_ACC(0), DD_ACC(1), DD_STAGE_TMP
               : DD_STAGE_USE
               : DD_STAGE_CLOBBER);
}
__device__ __forceinline__ void add_stage(uint32_t (&acc)[2][16], int meta, uint32_t base, int n) {
  uint32_t va, i, s0, s1, s2;
  asm volatile(DD_STAGE("v_add_u32")
               : DD_ACC(0), DD_ACC(1), DD_STAGE_TMP
               : DD_STAGE_USE
               : DD_STAGE_CLOBBER);
}

// Blocks of kShFold channels (FP32) or 256 channels (8-bit codes: 255 x 256 < 2^16) close into
// the running totals.
__device__ __forceinline__ void fold(float (&tot)[16], float (&acc)[16]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    tot[i] += acc[i];
    acc[i] = 0.f;
  }
}
__device__ __forceinline__ void fold(uint32_t (&tot)[32], uint32_t (&acc)[16]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    tot[i] += acc[i] & 0xFFFFu;
    tot[16 + i] += acc[i] >> 16;
    acc[i] = 0u;
  }
}

__device__ __forceinline__ float as_out(float v) { return v; }
__device__ __forceinline__ float as_out(uint32_t v) { return (float)v; }

template <int DT>
__device__ __forceinline__ void unit(const ShParams& P, int64_t tile, int grp, char* smem) {
  using T = typename Word<DT>::T;
  constexpr int G = dd::kShG;
  constexpr int H = DT == DD_U8 ? 2 : 1;  // outputs per word
  const int64_t t0 = tile * (H * dd::kShWords);
  T acc[G][16], tot[G][16 * H];
#pragma unroll
  for (int g = 0; g < G; ++g) {
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[g][i] = T(0);
#pragma unroll
    for (int i = 0; i < 16 * H; ++i) tot[g][i] = T(0);
  }
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  ci32_t tab = (ci32_t)P.tab;
  const int nst = tab[2 * grp + 1];
  const uint32_t wbase = (uint32_t)(P.ring ? (P.win0 + t0) % P.ring : t0);
  const uint32_t lds = dd::lds_addr(smem);
  const uint32_t spare = lds;
  const uint32_t base = lds + 16 * lane;
  const int at_form = 4 * (lane < dd::kShFormInts / 4 ? lane : 0);
  // records, loaded ahead of their use: this lane's four ints of the stage's, and this
  // wavefront's offsets (past the last stage the last record is loaded again, and not used)
  const int ints = dd::sh_stage_ints(P.nw);
  const DD_GLOBAL int32_t* rec = (const DD_GLOBAL int32_t*)P.tab + tab[2 * grp];
  const int at_add = dd::kShFormInts + dd::kShAddInts * wv + (lane & (dd::kShAddInts - 1));

  // Every wavefront alternates adding a stage with forming the next one. Between two barriers
  // the two are independent; half of a SIMD's wavefronts form first (their barrier comes
  // between the adds and the forming, one stage further on), so that the LDS reads of some run
  // beside the LDS writes of others. The first row of a stage's raw samples is loaded when the
  // stage before has been formed.
  const bool form_first = (wv >> 2) & 1;
  // Loads return in order, so what an iteration needs beside the raw samples (the next record
  // to form from, the next offsets) is loaded at its start and waited on before the next raw
  // loads go out.
  const DD_GLOBAL int32_t* arec = rec + at_add;
  int offs = *arec;
  Stage cur;  // the stage to form
  cur.meta = *(const DD_GLOBAL i4_t*)(rec + at_form);
  asm volatile("" : "+v"(offs), "+v"(cur.meta));
  open_stage<DT>(P, wbase, cur);
  Row<DT> r;
  load_row<DT>(P, cur, wv, lane, r);
  int formed = 0;
  int s = form_first ? -2 : -1;
  asm volatile("" : "+s"(s));  // one copy of the loop body: no peeled first iteration
#pragma nounroll
  for (; s < nst; ++s) {
    const int now = offs;
    if (s >= 0 && s + 1 < nst) arec += ints;
    offs = *arec;
    if (formed + 1 < nst) rec += ints;
    const i4_t next = *(const DD_GLOBAL i4_t*)(rec + at_form);  // the stage after cur
    if (s >= 0) {
      const int flags = __builtin_amdgcn_readlane(now, dd::kShAddInts - 1);  // bundles << 1 | fold
      add_stage(acc, now, base, __builtin_amdgcn_readfirstlane(G * (flags >> 1) - 1));
      if (flags & 1) {
#pragma unroll
        for (int g = 0; g < G; ++g) fold(tot[g], acc[g]);
      }
    }
    if (form_first && s >= -1) stage_barrier();
    if (formed < nst) {
      const int rows = stage_rows(cur);
      if (r.live) form_row<DT>(r, cur.meta.x, lane, lds, spare);
      for (int t = wv + P.nw; t < rows; t += P.nw) {
        load_row<DT>(P, cur, t, lane, r);
        form_row<DT>(r, cur.meta.x, lane, lds, spare);
      }
      ++formed;
    }
    cur.meta = next;
    asm volatile("" : "+v"(offs), "+v"(cur.meta));
    if (formed < nst) {
      open_stage<DT>(P, wbase, cur);
      load_row<DT>(P, cur, wv, lane, r);
    }
    if (!form_first) stage_barrier();
  }

  // outputs, and FP64 sums of the tile's outputs per trial (a fixed tree)
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int d = grp * P.per_group + wv * G + g;
    if (d >= P.ndm) break;
    float* row = P.out + (int64_t)d * P.out_stride;
    const bool vec = ((uint64_t)row & 15) == 0;
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t t = t0 + h * dd::kShWords + 4 * (kRow * i + lane);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = as_out(tot[g][16 * h + 4 * i + e]);
        if (lane < kRow) {
          if (t + 4 <= P.nout && vec) {
            *reinterpret_cast<float4*>(row + t) = make_float4(v[0], v[1], v[2], v[3]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (t + e < P.nout) row[t + e] = v[e];
          }
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (t + e < P.nout) {
              const double x = (double)v[e];
              s1 += x;
              s2 += x * x;
            }
        }
      }
    if (P.part) {
      s1 = dd::wave_sum_lane0(s1);
      s2 = dd::wave_sum_lane0(s2);
      if (lane == 0) {
        double* q = P.part + ((int64_t)d * P.ntile + tile) * 2;
        q[0] = s1;
        q[1] = s2;
      }
    }
  }
}

// One unit per workgroup; XCD x (workgroups x, x + 8, ...) takes a contiguous run of units,
// tile-major, so the DM groups of a tile share that XCD's L2.
template <int DT>
__global__ __launch_bounds__(64 * dd::sh_max_waves(DT)) void dedisp_shared(ShParams P) {
  extern __shared__ __align__(16) char smem[];
  const int64_t lin = blockIdx.x;
  const int64_t per = (P.nitems + 7) / 8;
  const int64_t item = (lin & 7) * per + (lin >> 3);
  if ((lin >> 3) >= per || item >= P.nitems) return;  // uniform for the workgroup, before any barrier
  const int64_t tile = item / P.ngroups;
  unit<DT>(P, tile, (int)(item - tile * P.ngroups), smem);
}

}  // namespace

namespace dd {

int launch_shared(const dd_plan* p, const InView& in, const int32_t* d_table, int64_t nout, float* out,
                  int64_t out_stride, double* part, void* stream) {
  if (in.nvalid >= (int64_t)1 << 30 || in.ring_len >= (int64_t)1 << 30)
    return fail(DD_ERR_UNSUPPORTED, "windows of 2^30 samples or more per channel are not supported");
  ShParams P{};
  P.in = in.ptr;
  P.row_stride = in.row_stride;
  P.nvalid = in.nvalid;
  P.win0 = in.win0;
  P.ring = (uint32_t)in.ring_len;
  // a ring row goes on past its length far enough for every window
  P.limit = in.ring_len > 0 ? 0x7fffffffu : (uint32_t)in.nvalid;
  P.tab = d_table;
  P.out = out;
  P.part = part;
  P.out_stride = out_stride;
  P.nout = nout;
  P.ntile = stat_tiles(p, nout);
  P.nitems = P.ntile * p->ngroups;
  P.ngroups = p->ngroups;
  P.ndm = p->ndm;
  P.per_group = p->dms_per_group;
  P.nw = p->sh.nw;
  const int64_t nblocks = (P.nitems + 7) / 8 * 8;
  if (nblocks > 0x7fffffff) return fail(DD_ERR_UNSUPPORTED, "too many work items");
  void (*k)(ShParams) = p->dtype == DD_F32   ? dedisp_shared<DD_F32>
                        : p->dtype == DD_F16 ? dedisp_shared<DD_F16>
                                             : dedisp_shared<DD_U8>;
  if (p->sh.lds > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p->sh.lds);
    if (e != hipSuccess) return fail(DD_ERR_HIP, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
  }
  hipLaunchKernelGGL(k, dim3((unsigned)nblocks), dim3(64 * P.nw), (size_t)p->sh.lds,
                     static_cast<hipStream_t>(stream), P);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(DD_ERR_HIP, std::string("dedisp_shared launch: ") + hipGetErrorString(e));
  return DD_OK;
}

}  // namespace dd
