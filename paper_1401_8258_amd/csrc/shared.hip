// Shared-sum form (gfx950, wave64): Eq. bruteEquation with the sums that several DM trials
// have in common formed once.
//
// Within a few neighbouring channels the delays of the trials of one DM group differ by a
// handful of patterns only: for channels c..c+3 the relative delays delta[c+j][d] -
// delta[c][d] of 32 consecutive trials take about 4 distinct values on the 408-428 MHz band.
// For every such bundle of up to 4 channels the workgroup forms each pattern's sum
//   S_p[x] = sum_j A[c_j][base_j + e_pj + x]      (window positions x, e_pj in 0..3)
// once in LDS, and every trial adds one S_p at its own offset instead of 4 channels. FP32 sums
// the channels of a bundle in order, the bundles of a block of up to kShFold consecutive channels
// in one running sum in the plan's order, and those sums in channel order; the plan chooses the
// blocks so that a total rounds no worse than channel by channel (dd_internal.h). 8-bit codes are
// exact integers either way.
//
// Work unit: one time tile x one group of trials. A tile is 1008 words: 4 rows of 63 lanes of
// 4 words. For FP32 and FP16 a word is one FP32 sample; for 8-bit input a word holds two
// 16-bit sums, of samples t and t + 1008 (so a shift of the window is a shift of words for
// both, and one 32-bit add serves two outputs), and the tile is 2016 samples. Lane 63 of a
// row holds the first words of the next row: a trial whose window starts s = 1..3 words past
// a 16-byte boundary takes its last words from the next lane by DPP, so one copy of each sum
// serves every alignment with four conflict-free ds_read_b128 per 16 words.
//
// A stage is up to three bundles, double-buffered in LDS, with one barrier a stage. Every
// wavefront adds the stage's sums to its trials and forms its share of the next stage's, in
// rows of 62-63 lanes x 4 window words of one bundle, from raw samples loaded into registers
// a stage earlier. Every other four wavefronts form before they add, so that one half's LDS
// writes run beside the other's reads.
//
// What bounds it: instruction issue and LDS together. FP32, 1024 channels x 2048 trials, per 4
// channels of 32 trials x 1008 samples: 1376 clocks of a CU, of which LDS is busy about 840
// (16 bytes a lane read in 4.2 clocks, written in 13.9) and each SIMD issues vector
// instructions for 935. HBM carries 66 GB a launch (the input is 4.3 GB), 1.8 TB/s, a third of a
// copy's rate. Measured and not kept:
// - wavefronts that only form beside ones that only add (12 + 4): bound by the forming ones,
//   101 ms against 59 at the time; all 16 doing both fills the waits of either part;
// - 12 wavefronts of 3 trials with 168 registers: 44.5 ms against 37.3 with 16 of 2;
// - several smaller workgroups per CU: fewer trials share each sum; slower but where the delays
//   grow by many samples a trial, which is what plan_shared weighs;
// - asking for the records' cache lines ahead of their loads: no difference.
// Times before (the LDS form for FP32 and FP16, the direct-read form for 8-bit) and now:
//   FP32, 408-428 MHz, 1024 channels x 1,048,576 samples x 2048 trials   97.2 -> 37.1 ms
//   8-bit, the same band, 1024 x 262,144 x 2000                          22.6 -> 5.9 ms
//   8-bit, 120-180 MHz, 4096 x 200,003 x 750                             22.0 -> 10.9 ms
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

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

static_assert(sizeof(ShParams) % 8 == 0, "copied in 64-bit words");
typedef const __attribute__((address_space(4))) ShParams* cparams_t;

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

// A form record (dd_internal.h) in scalar registers.
struct Rec {
  int off, d[3], chan, dst, slot, row, reach, more;
  uint32_t c0, c1;
};

__device__ __forceinline__ Rec load_rec(ci32_t p) {
  Rec k;
  k.off = p[0];
#pragma unroll
  for (int j = 0; j < 3; ++j) k.d[j] = p[1 + j];
  k.chan = p[4];
  k.dst = p[5];
  k.slot = p[6];
  k.row = p[7];
  k.c0 = (uint32_t)p[8];
  k.c1 = (uint32_t)p[9];
  k.reach = p[10];
  k.more = p[11];
  return k;
}

// What forming a row takes from its record, and the raw samples it is formed from.
template <int DT>
struct Row {
  int dst, slot, row;    // LDS offset, bytes per pattern, row
  uint32_t c0, c1;       // its patterns, a byte each
  uint32_t sh;           // per channel 2 bits: bytes its first sample lies past the dword
  uint32_t v[4][kRawN<DT>];
};

// This lane's dwords of one channel, from the scalar channel start p and the lane's offset vo.
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

// The raw samples' loads of a row: lane l of row r of a bundle loads the 4 window positions
// 4 (r VC + l) .. + 3 of every channel (8-bit input: also those 1008 samples later), in whole
// dwords; channels the bundle lacks are zeros. The first channel's window starts at sample
// wbase + its offset, less the ring's length past its end (the difference wraps to a large
// number before it; the length is 0 for linear input), the others' d bytes further on. Where a
// window would pass the last sample, each dword is clamped to that of the last sample:
// positions past it are used by no stored output. The usual case is one block of loads with
// scalar starts: a choice per channel, or starts in vector registers, made the compiler wait
// for earlier loads between them. The scalar unit serves all of a CU's wavefronts, one
// instruction a clock, so the starts are kept to a few operations.
template <int DT>
__device__ __forceinline__ void load_row(const ShParams& P, const Rec& k, uint32_t wbase, uint32_t lane16, Row<DT>& r) {
  constexpr int VC = dd::sh_row_chunks(DT);
  constexpr int EB = kEB<DT>;
  r.dst = k.dst;
  r.slot = k.slot;
  r.c0 = k.c0;
  r.c1 = k.c1;
  r.row = k.row & 255;
  r.sh = 0;
  if (k.row < 256) return;  // no channels
  // channels run up from `chan`, or down from it
  const uint64_t stride = (uint64_t)P.row_stride * EB, step = k.row & 4096 ? 0 - stride : stride;
  const uint32_t s0 = wbase + (uint32_t)k.off, s1 = s0 - P.ring, s = s1 < s0 ? s1 : s0;
  const bool whole = s + (uint32_t)k.reach <= P.limit;
  const uint64_t first = (uint64_t)P.in + (uint64_t)(uint32_t)k.chan * stride + (uint64_t)s * EB;
  const uint32_t vo = (uint32_t)(r.row * VC) * (4 * kDw<DT>) + lane16 / (4 / kDw<DT>);
  uint64_t base[4];
  uint32_t at[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    base[j] = first + j * step;
    at[j] = j ? (uint32_t)k.d[j - 1] : 0;
    if (DT != DD_F32) {
      at[j] += (uint32_t)base[j] & 3u;
      base[j] &= ~(uint64_t)3;
      r.sh |= (at[j] & 3u) << (2 * j);
      at[j] &= ~3u;
    }
  }
  if (whole && (k.row & 1024)) {  // four channels
#pragma unroll
    for (int j = 0; j < 4; ++j) load_words<DT>((gptr_t)base[j], vo + at[j], r.v[j]);
  } else {
    const int m = (k.row >> 8) & 7;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j >= m) {
#pragma unroll
        for (int i = 0; i < kRawN<DT>; ++i) r.v[j][i] = 0;
      } else if (whole) {
        load_words<DT>((gptr_t)base[j], vo + at[j], r.v[j]);
      } else {
        // a window starts before the last sample of its channel, so lim is not negative
        const uint64_t end = (uint64_t)P.in + (uint64_t)(uint32_t)k.chan * stride + (uint64_t)j * step +
                             (uint64_t)(P.nvalid * EB - 1);
        const uint32_t lim = (uint32_t)((end & ~(uint64_t)3) - base[j]);
#pragma unroll
        for (int i = 0; i < kRawN<DT>; ++i) {
          const uint32_t o = vo + at[j] + (DT == DD_U8 ? i * dd::kShWords : 4 * i);
          r.v[j][i] = *(const DD_GLOBAL uint32_t*)((gptr_t)base[j] + (o < lim ? o : lim));
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
// write and a jump to the next pattern's block, by its number in the low byte of q; number 64
// is past the table. A jump leaves more than the two instructions a DPP operand has to be
// older than.
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
  "s_and_b32 %[t], s80, 0xff\n\t"                \
  "s_lshr_b64 s[80:81], s[80:81], 8\n\t"         \
  "s_mulk_i32 %[t], %c[block]\n\t"               \
  "s_add_u32 vcc_lo, %[tlo], %[t]\n\t"           \
  "s_addc_u32 vcc_hi, %[thi], 0\n\t"             \
  "s_setpc_b64 vcc\n\t"
#define DD_FORM(n)                                                                                 \
  asm volatile(                                                                                    \
      "s_mov_b32 s80, %[c0]\n\t"                                                                   \
      "s_mov_b32 s81, %[c1]\n\t"                                                                   \
      "s_getpc_b64 vcc\n"                                                                          \
      "Ldd_pc_%=:\n\t"                                                                             \
      "s_add_u32 %[tlo], vcc_lo, Ldd_tab_%=-Ldd_pc_%=\n\t"                                         \
      "s_addc_u32 %[thi], vcc_hi, 0\n\t"                                                           \
      DD_FORM_GO                                                                                   \
      "Ldd_tab_%=:\n\t"                                                                            \
      ".irp e3, 0, 1, 2, 3\n\t"                                                                    \
      ".irp e2, 0, 1, 2, 3\n\t"                                                                    \
      ".irp e1, 0, 1, 2, 3\n\t"                                                                    \
      DD_FORM_ADD(n, "\\e1", "%4", "%5", "%6", "%7", "%8", "%9", "%10", "%11")                    \
      DD_FORM_ADD(n, "\\e2", "v112", "v113", "v114", "v115", "%12", "%13", "%14", "%15")           \
      DD_FORM_ADD(n, "\\e3", "v112", "v113", "v114", "v115", "%16", "%17", "%18", "%19")           \
      "ds_write_b128 %[dst], v[112:115]\n\t"                                                       \
      "v_add_u32_e32 %[dst], %[step], %[dst]\n\t"                                                  \
      DD_FORM_GO                                                                                   \
      ".endr\n\t"                                                                                  \
      ".endr\n\t"                                                                                  \
      ".endr\n"                                                                                    \
      "Ldd_end_%=:\n\t"                                                                            \
      ".if Ldd_end_%=-Ldd_tab_%= != 64*%c[block]\n\t.error \"block size\"\n\t.endif"               \
      : [dst] "+v"(dst), [t] "=&s"(t), [tlo] "=&s"(tlo), [thi] "=&s"(thi)                          \
      : "v"(w[0][0]), "v"(w[0][1]), "v"(w[0][2]), "v"(w[0][3]), "v"(w[1][0]), "v"(w[1][1]),        \
        "v"(w[1][2]), "v"(w[1][3]), "v"(w[2][0]), "v"(w[2][1]), "v"(w[2][2]), "v"(w[2][3]),        \
        "v"(w[3][0]), "v"(w[3][1]), "v"(w[3][2]), "v"(w[3][3]), [c0] "s"(c0), [c1] "s"(c1),        \
        [step] "v"(step), [block] "i"(dd::kShBlock)                                                \
      : "scc", "vcc", "memory", "s80", "s81", "v112", "v113", "v114", "v115")
__device__ __forceinline__ void form(const float (&w)[4][4], uint32_t c0, uint32_t c1, uint32_t dst, uint32_t step) {
  uint32_t t, tlo, thi;
  DD_FORM("v_add_f32");
}
__device__ __forceinline__ void form(const uint32_t (&w)[4][4], uint32_t c0, uint32_t c1, uint32_t dst, uint32_t step) {
  uint32_t t, tlo, thi;
  DD_FORM("v_add_u32");
}

// Forms row r: the words of its channels, then the sums.
// Lanes without a window chunk of their own write to the spare slot.
template <int DT>
__device__ __forceinline__ void form_row(const Row<DT>& r, uint32_t lane16, uint32_t lds) {
  using T = typename Word<DT>::T;
  constexpr int VC = dd::sh_row_chunks(DT);
  T w[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) words<DT>(r, j, w[j]);
  const uint32_t at = (uint32_t)(16 * VC * r.row) + lane16;
  const bool mine = lane16 < 16 * VC && at < (uint32_t)r.slot;
  form(w, r.c0, r.c1, lds + (mine ? r.dst + at : lane16), mine ? r.slot : 0);
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
#define DD_READ0 "ds_read_b128 v[112:115], %[va]\n\t"
#define DD_READ1 "ds_read_b128 v[116:119], %[va] offset:1008\n\t"
#define DD_READ2 "ds_read_b128 v[120:123], %[va] offset:2016\n\t"
#define DD_READ3 "ds_read_b128 v[124:127], %[va] offset:3024\n\t"
#define DD_WAIT(c) "s_waitcnt lgkmcnt(" #c ")\n\t"
#define DD_ROWS(SH, n, ...) DD_ROWS_(SH, n, __VA_ARGS__)
#define DD_ROWS_(SH, n, A0, A1, A2, A3, A4, A5, A6, A7, A8, A9, A10, A11, A12, A13, A14, A15) \
  DD_WAIT(3) SH(n, A0, A1, A2, A3, 112, 113, 114, 115) DD_READ0                               \
  DD_WAIT(3) SH(n, A4, A5, A6, A7, 116, 117, 118, 119) DD_READ1                               \
  DD_WAIT(3) SH(n, A8, A9, A10, A11, 120, 121, 122, 123) DD_READ2                             \
  DD_WAIT(3) SH(n, A12, A13, A14, A15, 124, 125, 126, 127) DD_READ3
// The last unit: nothing left to read.
#define DD_LAST_ROWS(SH, n, ...) DD_LAST_ROWS_(SH, n, __VA_ARGS__)
#define DD_LAST_ROWS_(SH, n, A0, A1, A2, A3, A4, A5, A6, A7, A8, A9, A10, A11, A12, A13, A14, A15) \
  DD_WAIT(3) SH(n, A0, A1, A2, A3, 112, 113, 114, 115)                                             \
  DD_WAIT(2) SH(n, A4, A5, A6, A7, 116, 117, 118, 119)                                             \
  DD_WAIT(1) SH(n, A8, A9, A10, A11, 120, 121, 122, 123)                                           \
  DD_WAIT(0) SH(n, A12, A13, A14, A15, 124, 125, 126, 127)
// The four ways of unit K, whose shift is bits 2 K, 2 K + 1 of %[sh].
#define DD_WAYS(K, L, ROWS, n, ...)             \
  "s_bitcmp1_b32 %[sh], 2*" #K "+1\n\t"         \
  "s_cbranch_scc1 Ldd_" #L #K "c_%=\n\t"        \
  "s_bitcmp1_b32 %[sh], 2*" #K "\n\t"           \
  "s_cbranch_scc1 Ldd_" #L #K "b_%=\n\t"        \
  ROWS(DD_SH0, n, __VA_ARGS__)                  \
  "s_branch Ldd_" #L #K "e_%=\n"                \
  "Ldd_" #L #K "b_%=:\n\t"                      \
  ROWS(DD_SH1, n, __VA_ARGS__)                  \
  "s_branch Ldd_" #L #K "e_%=\n"                \
  "Ldd_" #L #K "c_%=:\n\t"                      \
  "s_bitcmp1_b32 %[sh], 2*" #K "\n\t"           \
  "s_cbranch_scc1 Ldd_" #L #K "d_%=\n\t"        \
  ROWS(DD_SH2, n, __VA_ARGS__)                  \
  "s_branch Ldd_" #L #K "e_%=\n"                \
  "Ldd_" #L #K "d_%=:\n\t"                      \
  ROWS(DD_SH3, n, __VA_ARGS__)                  \
  "Ldd_" #L #K "e_%=:\n\t"
#define DD_U0 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15
#define DD_U1 16, 17, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31
// Unit K reads ahead the window at %[aN] (unit K + 1's); a bundle's second unit is the last one
// if %[end] says so.
#define DD_UNIT(K, N, n, ...) "v_add_u32 %[va], %[a" #N "], %[base]\n\t" DD_WAYS(K, u, DD_ROWS, n, __VA_ARGS__)
#define DD_END(K, n)                            \
  "s_cmp_eq_u32 %[end], " #K "\n\t"               \
  "s_cbranch_scc0 Ldd_go" #K "_%=\n\t"          \
  DD_WAYS(K, l, DD_LAST_ROWS, n, DD_U1)         \
  "s_branch Ldd_out_%=\n"                       \
  "Ldd_go" #K "_%=:\n\t"
// A stage's bundles: units (bundle, trial) in order, unit K's window at LDS offset %[aK] and
// its shift in %[sh]; %[end] is the last unit. All of the window registers' reads end in here:
// one asm block, so that nothing else touches them while a read is in flight.
#define DD_STAGE(n)                                                                                       \
  asm volatile("v_add_u32 %[va], %[a0], %[base]\n\t" DD_READ0 DD_READ1 DD_READ2 DD_READ3                  \
               DD_UNIT(0, 1, n, DD_U0) DD_END(1, n) DD_UNIT(1, 2, n, DD_U1)                               \
               DD_UNIT(2, 3, n, DD_U0) DD_END(3, n) DD_UNIT(3, 4, n, DD_U1)                               \
               DD_UNIT(4, 5, n, DD_U0) DD_WAYS(5, l, DD_LAST_ROWS, n, DD_U1)                              \
               "Ldd_out_%=:"                                                                              \
               : DD_ACC(0), DD_ACC(1), [va] "=&v"(va)                                                     \
               : [base] "v"(base), [end] "s"(k.last & 255), [sh] "s"(k.sh), [a0] "s"(k.a[0]), [a1] "s"(k.a[1]),   \
                 [a2] "s"(k.a[2]), [a3] "s"(k.a[3]), [a4] "s"(k.a[4]), [a5] "s"(k.a[5])                   \
               : "scc", "memory", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", \
                 "v121", "v122", "v123", "v124", "v125", "v126", "v127")
#define DD_ACC(g)                                                                                          \
  "+v"(acc[g][0]), "+v"(acc[g][1]), "+v"(acc[g][2]), "+v"(acc[g][3]), "+v"(acc[g][4]), "+v"(acc[g][5]),    \
      "+v"(acc[g][6]), "+v"(acc[g][7]), "+v"(acc[g][8]), "+v"(acc[g][9]), "+v"(acc[g][10]),                \
      "+v"(acc[g][11]), "+v"(acc[g][12]), "+v"(acc[g][13]), "+v"(acc[g][14]), "+v"(acc[g][15])

// An add record (dd_internal.h) in scalar registers.
struct Adds {
  int a[6], sh, last;  // last: the last unit | fold << 8
};
__device__ __forceinline__ Adds load_adds(ci32_t p) {
  Adds k;
#pragma unroll
  for (int i = 0; i < 6; ++i) k.a[i] = p[i];
  k.sh = p[6];
  k.last = p[7];
  return k;
}

static_assert(dd::kShG == 2 && dd::kShMaxBundles == 3, "a stage's code walks two trials of up to three bundles");
__device__ __forceinline__ void add_stage(float (&acc)[2][16], const Adds& k, uint32_t base) {
  uint32_t va;
  DD_STAGE("v_add_f32");
}
__device__ __forceinline__ void add_stage(uint32_t (&acc)[2][16], const Adds& k, uint32_t base) {
  uint32_t va;
  DD_STAGE("v_add_u32");
}

// Blocks of up to kShFold channels (FP32) or 256 channels (8-bit codes: 255 x 256 < 2^16) close into
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

// Q: where P was read from.
template <int DT>
__device__ __forceinline__ void unit(const ShParams& P, cparams_t Q, int64_t tile, int grp, char* smem) {
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
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  ci32_t tab = (ci32_t)P.tab;
  const int nst = tab[2 * grp + 1];
  const uint32_t wbase = (uint32_t)(P.ring ? (P.win0 + t0) % P.ring : t0);
  const uint32_t lds = dd::lds_addr(smem);
  const uint32_t lane16 = 16 * (threadIdx.x & 63);  // the spare slot comes first in the LDS
  // Every wavefront alternates adding a stage with forming the next one. Between two barriers
  // the two are independent; half of a SIMD's wavefronts form first (their barrier comes
  // between the adds and the forming, one stage further on), so that the LDS reads of some run
  // beside the LDS writes of others. The first row of a stage's raw samples is loaded when the
  // stage before has been formed. Records before the first stage and past the last one are
  // readable and go unused.
  const int ints = dd::sh_stage_ints(P.nw);
  ci32_t group = tab + tab[2 * grp];
  const int form_first = (wv >> 2) & 1;
  int s = -1 - form_first;
  asm volatile("" : "+s"(s));  // one copy of the loop body: no peeled first iteration
  Row<DT> r;
  int more;
  {
    const Rec k = load_rec(group + dd::kShRecInts * wv + dd::kShAddInts);
    load_row<DT>(P, k, wbase, lane16, r);
    more = k.more;
  }
  ci32_t rec = group + dd::kShRecInts * wv + (s + 1) * ints;  // stage s + 1's record
  const int form_at = (1 + form_first) * ints + dd::kShAddInts;  // from there to the form record after next
  Adds adds = load_adds(rec);  // waited on here, not in the loop
  asm volatile("" : "+s"(adds.a[0]), "+s"(adds.a[1]), "+s"(adds.a[2]), "+s"(adds.a[3]), "+s"(adds.a[4]),
               "+s"(adds.a[5]), "+s"(adds.sh), "+s"(adds.last));
#pragma nounroll
  for (; s < nst; ++s) {
    if (s >= 0) {
      add_stage(acc, adds, lds + lane16);
      if (adds.last >> 8) {
#pragma unroll
        for (int g = 0; g < G; ++g) fold(tot[g], acc[g]);
      }
    }
    if (form_first && s >= -1) stage_barrier();
    // the next records: after the adds, whose waits for LDS reads would take these loads in, and
    // back by the time the rows have been formed
    const Adds ahead = load_adds(rec);
    const Rec k = load_rec(rec + form_at);
    rec += ints;
    if (s + 1 + form_first < nst) {
      // this wavefront's row of the stage, further ones by links, then the next stage's first
      form_row<DT>(r, lane16, lds);
      while (more) {
        const Rec x = load_rec(group + more);
        load_row<DT>(P, x, wbase, lane16, r);
        more = x.more;
        form_row<DT>(r, lane16, lds);
      }
      load_row<DT>(P, k, wbase, lane16, r);
      more = k.more;
    }
    adds = ahead;
    if (!form_first) stage_barrier();
  }

  // outputs, and FP64 sums of the tile's outputs per trial (a fixed tree). The parameters are
  // read again here, so that they take no registers in the loop.
  asm volatile("" : "+s"(Q));
  uint32_t l16 = lane16;
  asm volatile("" : "+v"(l16));
  const int lane = (int)(l16 >> 4);
  float* const out = Q->out;
  double* const part = Q->part;
  const int64_t nout = Q->nout;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int d = grp * Q->per_group + wv * G + g;
    if (d >= Q->ndm) break;
    float* row = out + (int64_t)d * Q->out_stride;
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
          if (t + 4 <= nout && vec) {
            *reinterpret_cast<float4*>(row + t) = make_float4(v[0], v[1], v[2], v[3]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (t + e < nout) row[t + e] = v[e];
          }
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (t + e < nout) {
              const double x = (double)v[e];
              s1 += x;
              s2 += x * x;
            }
        }
      }
    if (part) {
      s1 = dd::wave_sum_lane0(s1);
      s2 = dd::wave_sum_lane0(s2);
      if (lane == 0) {
        double* q = part + ((int64_t)d * Q->ntile + tile) * 2;
        q[0] = s1;
        q[1] = s2;
      }
    }
  }
}

// One unit per workgroup; XCD x (workgroups x, x + 8, ...) takes a contiguous run of units,
// tile-major, so the DM groups of a tile share that XCD's L2.
template <int DT>
__global__ __launch_bounds__(64 * dd::kShWaves) void dedisp_shared(ShParams P) {
  extern __shared__ __align__(16) char smem[];
  const int64_t lin = blockIdx.x;
  const int64_t per = (P.nitems + 7) / 8;
  const int64_t item = (lin & 7) * per + (lin >> 3);
  if ((lin >> 3) >= per || item >= P.nitems) return;  // uniform for the workgroup, before any barrier
  const int64_t tile = item / P.ngroups;
  unit<DT>(P, (cparams_t)__builtin_amdgcn_kernarg_segment_ptr(), tile, (int)(item - tile * P.ngroups), smem);
}

// The same units over several items of one input type and workgroup size: XCD x takes an eighth of
// each item's units in turn, run[x][i] units of items 0 .. i - 1 before item i's. An item's own
// launch ends with a round of units that fills the chip in part, and a small item is no more than
// that. Batches of 32 8-bit items of 256 channels x 4000 samples x 200 trials and of 16 of 128
// channels x 2278 x 64 took 2.70 and 0.92 ms with a launch an item, 0.26 and 0.13 ms in one.
template <int DT>
__global__ __launch_bounds__(64 * dd::kShWaves) void shared_sum_batch(const ShParams* __restrict__ items,
                                                                      const int64_t* __restrict__ run, int n) {
  extern __shared__ __align__(16) char smem[];
  typedef const __attribute__((address_space(4))) int64_t* ci64_t;
  const int64_t lin = blockIdx.x;
  const int x = (int)(lin & 7);
  const ci64_t rx = (ci64_t)(run + (int64_t)x * (n + 1));
  const int64_t k = lin >> 3;
  if (k >= rx[n]) return;  // uniform for the workgroup, before any barrier
  int lo = 0, hi = n - 1;  // the last item whose run starts at or before k
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (rx[mid] <= k) lo = mid;
    else hi = mid - 1;
  }
  const cparams_t Q = (cparams_t)(items + lo);
  // wave-uniform copy of the item's record through scalar loads
  const ci64_t src = (ci64_t)Q;
  int64_t word[sizeof(ShParams) / 8];
#pragma unroll
  for (int j = 0; j < (int)(sizeof(ShParams) / 8); ++j) word[j] = src[j];
  ShParams P;
  __builtin_memcpy(&P, word, sizeof(P));
  const int64_t item = (P.nitems * x) / 8 + (k - rx[lo]);
  const int64_t tile = item / P.ngroups;
  unit<DT>(P, Q, tile, (int)(item - tile * P.ngroups), smem);
}

}  // namespace

namespace dd {

namespace {

using Kernel = void (*)(ShParams);
using BatchKernel = void (*)(const ShParams*, const int64_t*, int);

int prepare(const dd_plan* p, const InView& in, const int32_t* d_table, int64_t nout, float* out, int64_t out_stride,
            double* part, ShParams* P) {
  if (in.nvalid >= (int64_t)1 << 30 || in.ring_len >= (int64_t)1 << 30)
    return fail(DD_ERR_UNSUPPORTED, "windows of 2^30 samples or more per channel are not supported");
  *P = ShParams{};
  P->in = in.ptr;
  P->row_stride = in.row_stride;
  P->nvalid = in.nvalid;
  P->win0 = in.win0;
  P->ring = (uint32_t)in.ring_len;
  // a ring row goes on past its length far enough for every window
  P->limit = in.ring_len > 0 ? 0x7fffffffu : (uint32_t)in.nvalid;
  P->tab = d_table;
  P->out = out;
  P->part = part;
  P->out_stride = out_stride;
  P->nout = nout;
  P->ntile = stat_tiles(p, nout);
  P->nitems = P->ntile * p->ngroups;
  P->ngroups = p->ngroups;
  P->ndm = p->ndm;
  P->per_group = p->dms_per_group;
  P->nw = p->sh.nw;
  return DD_OK;
}

int allow_lds(const void* k, int64_t lds) {
  if (lds <= 65536) return DD_OK;
  const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return fail(DD_ERR_HIP, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
  return DD_OK;
}

int launch(const dd_plan* p, const ShParams& P, hipStream_t st) {
  const int64_t nblocks = (P.nitems + 7) / 8 * 8;
  if (nblocks > 0x7fffffff) return fail(DD_ERR_UNSUPPORTED, "too many work items");
  const Kernel k = p->dtype == DD_F32   ? dedisp_shared<DD_F32>
                   : p->dtype == DD_F16 ? dedisp_shared<DD_F16>
                                        : dedisp_shared<DD_U8>;
  const int rc = allow_lds((const void*)k, p->sh.lds);
  if (rc) return rc;
  hipLaunchKernelGGL(k, dim3((unsigned)nblocks), dim3(64 * P.nw), (size_t)p->sh.lds, st, P);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(DD_ERR_HIP, std::string("dedisp_shared launch: ") + hipGetErrorString(e));
  return DD_OK;
}

}  // namespace

int launch_shared(const dd_plan* p, const InView& in, const int32_t* d_table, int64_t nout, float* out,
                  int64_t out_stride, double* part, void* stream) {
  ShParams P;
  const int rc = prepare(p, in, d_table, nout, out, out_stride, part, &P);
  return rc ? rc : launch(p, P, static_cast<hipStream_t>(stream));
}

int64_t shared_batch_desc_bytes(int32_t n) {
  // the records, then per launch the XCD runs [8][items + 1] (at most n launches)
  return align_up((int64_t)n * (int64_t)sizeof(ShParams)) + align_up((int64_t)8 * 8 * 2 * n);
}

int launch_shared_batch(const std::vector<SharedItem>& items, void* d_desc, int64_t desc_bytes, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int32_t n = (int32_t)items.size();
  if (n == 0) return DD_OK;
  if (desc_bytes < shared_batch_desc_bytes(n)) return fail(DD_ERR_WORKSPACE, "batch workspace too small");
  std::vector<ShParams> all((size_t)n);
  std::vector<int32_t> order((size_t)n);
  for (int32_t i = 0; i < n; ++i) {
    const SharedItem& it = items[i];
    const int rc = prepare(it.plan, it.in, it.table, it.nout, it.out, it.out_stride, it.part, &all[i]);
    if (rc) return rc;
    order[i] = i;
  }
  // the longest units first: the shortest fill the last round
  std::stable_sort(order.begin(), order.end(),
                   [&](int32_t a, int32_t b) { return items[a].plan->sh.stages > items[b].plan->sh.stages; });
  // one launch per input type and workgroup size, in the order of their longest units
  struct Group {
    const dd_plan* plan;
    int32_t first, count;
    int64_t run_at, longest;
  };
  std::vector<Group> groups;
  std::vector<ShParams> rec;
  std::vector<int64_t> run;
  for (int32_t i : order) {
    const dd_plan* p = items[i].plan;
    auto like = [&](const dd_plan* q) { return q->dtype == p->dtype && q->sh.nw == p->sh.nw && q->sh.lds == p->sh.lds; };
    if (std::any_of(groups.begin(), groups.end(), [&](const Group& g) { return like(g.plan); })) continue;
    Group gr{p, (int32_t)rec.size(), 0, (int64_t)run.size(), 0};
    for (int32_t j : order)
      if (like(items[j].plan)) rec.push_back(all[j]), ++gr.count;
    for (int x = 0; x < 8; ++x) {
      int64_t k = 0;
      run.push_back(0);
      for (int32_t j = 0; j < gr.count; ++j) {
        const int64_t u = rec[(size_t)(gr.first + j)].nitems;
        k += (u * (x + 1)) / 8 - (u * x) / 8;  // XCD x's eighth of item j
        run.push_back(k);
      }
      gr.longest = std::max(gr.longest, k);
    }
    if (8 * gr.longest > 0x7fffffff) return fail(DD_ERR_UNSUPPORTED, "too many work items");
    groups.push_back(gr);
  }
  char* bw = static_cast<char*>(d_desc);
  ShParams* d_rec = reinterpret_cast<ShParams*>(bw);
  int64_t* d_run = reinterpret_cast<int64_t*>(bw + align_up((int64_t)n * (int64_t)sizeof(ShParams)));
  if (std::any_of(groups.begin(), groups.end(), [](const Group& g) { return g.count > 1; })) {
    hipError_t e = hipMemcpyAsync(d_rec, rec.data(), rec.size() * sizeof(ShParams), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(d_run, run.data(), run.size() * 8, hipMemcpyHostToDevice, st);
    if (e != hipSuccess)
      return fail(DD_ERR_HIP, std::string("hipMemcpyAsync (batch descriptors): ") + hipGetErrorString(e));
  }
  for (const Group& gr : groups) {
    if (gr.count == 1) {  // its own launch needs no descriptors
      const int rc = launch(gr.plan, rec[(size_t)gr.first], st);
      if (rc) return rc;
      continue;
    }
    const BatchKernel k = gr.plan->dtype == DD_F32   ? shared_sum_batch<DD_F32>
                          : gr.plan->dtype == DD_F16 ? shared_sum_batch<DD_F16>
                                                     : shared_sum_batch<DD_U8>;
    const int rc = allow_lds((const void*)k, gr.plan->sh.lds);
    if (rc) return rc;
    hipLaunchKernelGGL(k, dim3((unsigned)(8 * gr.longest)), dim3(64 * gr.plan->sh.nw), (size_t)gr.plan->sh.lds, st,
                       (const ShParams*)(d_rec + gr.first), (const int64_t*)(d_run + gr.run_at), (int)gr.count);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(DD_ERR_HIP, std::string("shared_sum_batch launch: ") + hipGetErrorString(e));
  }
  return DD_OK;
}

}  // namespace dd
