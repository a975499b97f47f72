// Launch planning of the matrix-core pair kernel: which products of shifted
// time series a launch forms, and where frames lie in its LDS planes.
// Host-only, no HIP dependency.
//
// The kernel holds every coefficient of a mode's time series as a whole number
// of 31 bits at most in four signed bytes, one byte plane per digit, and forms
//   C_lag = sum_t q[t] q[t - lag]
// by 16 x 16 x 64 byte matrix products: the 16 rows are the older series
// shifted back by four 16-frame blocks times 4 digits, the 16 columns the
// target series shifted by 4 c + j, j = 0..3 (c: the column class) times 4
// digits, the inner index is time. One product (a "tile": a row set of four
// blocks b and a class c) covers the 16 delays 16 b + 4 c + j with all their
// digit products; the four tiles of a row set cover its 64 delays from one
// read of the rows.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "pair_plan.hpp"

namespace nfs {

// Tasks, row sets and delays of one launch at most: the tables travel in the
// kernel's arguments (4 KB at most).
constexpr int kMxTasks = 24;
constexpr int kMxRows = 96;
constexpr int kMxLags = 512;
constexpr int kMxChunks = kMxLags / 64 + kMxTasks;
// Whole row sets of a task at most; with the scattered ones it accumulates up
// to 4 * (kMxSets + 1) tiles of 4 registers.
constexpr int kMxSets = 4;
constexpr int kMxTiles = 4 * (kMxSets + 1);
constexpr int kMxWaves = 4;
constexpr int kMxRounds = 5;  // of octets that a thread loads at most
// Bytes of a digit plane at most (4 modes per workgroup, two workgroups per
// CU); a longer window is cut.
constexpr int kMxPlane = 2240;
// LDS of one workgroup, half a CU's.
constexpr int kMxLds = 80 * 1024;
// Scale 2^mx_exponent of a mode whose squares over a launch's frames sum to E, with
// the bits of the normal FP32 number kMxRoom * E: it takes E to 0.94 * 2^60 .. 0.94 * 2^62,
// so that a sum of squared differences, at most four times that, stays below 2^64
// whatever the signs, and the numbers below 2^31 - 2^24.
constexpr float kMxRoom = 1.0625f;
constexpr int mx_exponent(uint32_t bits) { return (188 - int(bits >> 23 & 255)) >> 1; }
// Energies that this is right for: of squares that FP32 holds.
constexpr float kMxMost = 3.4028235e38f;
constexpr float kMxFew = 0x1p-100f;
// Sums below this many steps^2 of a mode's whole numbers are formed again from
// its coefficients. Rounding them moves a sum of P pairs by 0.82 / sqrt(S) of
// itself (rms; at most 2.9 sqrt(P / S)): 2^-24 at the line, the rounding of one
// FP32 term.
constexpr unsigned long long kMxLeast = 1ull << 48;
// Delays of one launch span at most this many frames when a window has to be
// cut, so that its two frame ranges leave room for targets.
constexpr int kMxSpan = 600;

// Tiles a wave accumulates together: `sets` whole row sets (with column
// classes 0..3: tiles 4 * set + class) and, if `scattered`, one row set per
// class (tile 4 * sets + class).
struct MxTask {
  int16_t sets;
  int16_t scattered;
  int16_t rows0;   // first row set
  int16_t start;   // targets from 16 * start frames after the first target on
  int16_t first;   // its delays that are in no run: order[first .. first + count)
  int16_t count;
  int16_t chunk0;  // tiles of its delays, 64 at a time: chunk[chunk0 ..]
  int16_t run0;    // runs of its whole sets: run[run0 ..]
};

// Tables of one launch (by value in the kernel's arguments).
struct MxTables {
  int32_t n_tasks = 0, n_rows = 0;
  int32_t n_paired = 0;               // delays of the group below t1
  int32_t lag0 = 0;                   // blocks are relative to this delay (a multiple of 16)
  MxTask task[kMxTasks];
  uint32_t chunk[kMxChunks];          // bit s: row set s (sets: scattered) has a delay of the chunk
  uint16_t block[kMxRows][4];         // of a row set
  uint32_t run[kMxRows / 2];          // of a whole set (by order of the sets), see mx_run
  // The other delays task by task, see mx_order.
  uint32_t order[kMxLags];
};

// Index in the group's list, row set of the task (sets: the scattered ones),
// row of it, and the delay less lag0.
constexpr uint32_t mx_order(int lag_index, int set, int row, int64_t tau) {
  return uint32_t(lag_index) | uint32_t(set) << 9 | uint32_t(row) << 13 | uint32_t(tau) << 15;
}
// A whole set whose delays are consecutive: list index of the first, and the
// first's and last's place among the set's 64 delays. 0: none.
constexpr uint32_t mx_run(int lag_index, int64_t first, int64_t last) {
  return 1u << 31 | uint32_t(lag_index) | uint32_t(first) << 9 | uint32_t(last) << 15;
}
constexpr int kMxMinRun = 24;         // delays of a run at least
constexpr int kMxMaxSpan = 120000;    // of a group's delays: order holds 17 bits
static_assert(kMxLags <= 1 << 9 && kMxSets < 16, "mx_order's fields");
static_assert(kMxTiles <= 32, "chunk masks");
static_assert(sizeof(MxTables) <= 3600, "kernel arguments");

// Delays lags[first .. first + count) handled together.
struct MxGroup {
  int first = 0, count = 0;
};

// Frames and LDS places of one launch: targets [t0, t1), older frames
// [olo, olo + olen). A plane byte at x < split holds older frame
// olo + x - obase, at x >= split target t0 + x - tbase; `split` = pl when
// one range holds both (then tbase = obase + t0 - olo). Bytes that are no
// frame's are zero.
struct MxShape {
  int64_t t0 = 0, t1 = 0, olo = 0;
  int olen = 0, obase = 0, tbase = 0, split = 0;
  int pl = 0;      // bytes per plane
  int aoff = 0;    // older row of plane place k, delay 0: k + aoff
  int amin = 0;    // lowest place an older row is read from (16 zero bytes)
  int km = 0;      // modes per workgroup
  size_t lds = 0;  // dynamic LDS bytes
};

// Groups of delays for windows that fit one launch (span 0) or are cut
// (span kMxSpan).
std::vector<MxGroup> mx_groups(const std::vector<int32_t>& lags, int span);

// Place of targets [t0, t1) and their older frames for delays [ta, tb].
MxShape mx_shape(int64_t t0, int64_t t1, int64_t ta, int64_t tb);

// End of the next launch's targets from t0 on, at most t1: near-equal cuts
// that fit kMxPlane.
int64_t mx_cut(int64_t t0, int64_t t1, int64_t ta, int64_t tb);

// Modes per workgroup and LDS bytes of a shape for `modes` modes.
void mx_workgroup(MxShape* s, int64_t modes);

// Whether the kernel may read rows of `row` bytes by 32-bit offsets from the
// first row of each range: neither range wraps in the ring, and no place of the
// plane is 4 GiB or more from it. Places that are no frame's, up to 207 past the
// last one, then lie past the range's descriptor and read as 0.
bool mx_direct(const MxShape& s, int64_t capacity, int64_t row);

// Tables for the group's delays below t1 and the targets [t0, t1).
void mx_tables(const std::vector<int32_t>& lags, const MxGroup& g, int64_t t0, int64_t t1,
               MxTables* out);

// Whether the matrix-core kernel is expected to sum the targets [t0, t1) of
// all delays sooner than the explicit one (its groups: `groups`).
bool mx_wins(const std::vector<int32_t>& lags, const std::vector<LagGroup>& groups,
             const std::vector<MxGroup>& mx, int64_t t0, int64_t t1);

// 16-frame steps of a task's four time quarters: targets from
// tbase - 16 + 16 * start on.
inline int mx_steps(int targets, int start) {
  const int blocks = (targets + 16 - 16 * start + 15) / 16;
  return (blocks + 3) / 4;
}

}  // namespace nfs
