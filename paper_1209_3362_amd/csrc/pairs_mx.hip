// Lag-pair sums on the matrix cores. For every stored mode and delay
//   S_tau = sum_t |a_t - a_{t-tau}|^2
//         = sum_t |a_t|^2 + sum_t |a_{t-tau}|^2 - 2 Re sum_t a_t conj(a_{t-tau})
// is formed in integers: a mode's coefficients in the window are scaled by one
// power of two and rounded to whole numbers, and all sums are exact modulo 2^64.
// The scale makes the sum of their squares, E, less than 2^62, so every S_tau, at
// most 4 E, is held itself, and every number has 31 bits at most (mx_exponent). So
// nothing cancels: equal frames give exactly 0, and the only rounding is that
// of the coefficients: for 1000 of like size about 2^-26 of theirs. A sum that
// this rounding reaches is summed again from the coefficients themselves: below
// kMxLeast steps^2 (few pairs, slow modes, or one frame far larger than the
// others), and all sums of a mode with a value that is not finite.
//
// The cross terms are byte products on MFMA (see pair_matrix.hpp): a
// 16 x 16 x 64 product gives 16 delays over 64 frames with all 16 digit
// products. The explicit form costs four FP32 instructions per pair and mode
// on the vector units; here 16 delays of a dense list cost 16 matrix cycles
// per 32 frames and mode. Time is cut into four quarters, one per 16-lane
// group of the operands, and walked in 16-frame steps, so the older rows of
// the next 16 delays are those read one step before: a wave keeps them in
// registers and reads two operands from LDS for up to eight products.
//
// One workgroup owns km modes (16, 8 or 4) and reads each of their
// coefficients once: all frames of the window are loaded into registers,
// corrected by the reference transform, scaled and written as byte planes;
// prefix sums of |a|^2 every 8 frames give the energies, the frames between
// them from the planes by byte dot products, or for 64 consecutive delays by a
// sum over the lanes. 4-wave workgroups, two per CU (80 KB of LDS, some 240
// registers per lane): one's loads run under the other's products.
//
// Measured against the explicit kernel (pair stage, MI355X): 2048 frames of
// 512 x 512 with all 2047 delays 63.6 -> 9.2 ms; 900 frames of 1024 x 1024,
// delays 1..400, BF16 spectra, 23.0 -> 5.7 ms, of which the products take 3.1
// (the matrix units' own time is 2.4: 18.5 cycles per product at 2.4 GHz), the
// digits 0.8 and the energies 1.3. Bound by instruction issue at two waves per
// SIMD: a step of four row sets is 16 products and 23 vector instructions.
// The small sums and the test for them take 0.45 of the 9.2 ms (the last delays
// have few pairs) and 0.1 of the 5.7. 300 frames of 512 x 512 with 250 delays take
// 0.58 ms, with a frame 10^4 times the others, where the sums of 100
// delays are small, 1.42; the explicit kernel takes 1.51.
// 8-wave workgroups of 128 registers (four waves per SIMD, two row sets per
// task) took as long on dense delays and 10 % longer on the 2047.
#include <algorithm>

#include "nfs_device.hpp"
#include "nfs_kernels.hpp"
#include "pair_matrix.hpp"

namespace nfs {
namespace {
using dev::kSpecBF16;
using dev::kSpecF16;
using dev::kSpecF32;

typedef int v4i __attribute__((ext_vector_type(4)));

struct MxArgs {
  const char* ring;
  const float2* refspec;
  const float4* fscale;
  float* acc;
  float* comp;
  const int32_t* lags;
  unsigned long long* work;
  int64_t n_modes, mode_stride, t0, t1;
  int32_t capacity, slot_old, slot_new;  // ring slots of frames olo and t0
  int32_t olen, obase, tbase, split, pl, aoff, amin, km_log2;
  int64_t olo;
  int32_t n_lags, acc_pitch, assign;
  int32_t zero_from;  // delays from this one on have no pair: set to 0 with `assign`
  int32_t direct;     // buffer loads (see mx_direct)
  MxTables tab;
};

extern __shared__ char smem[];

// LDS address of a pointer into it, and 16 bytes at an address + PLUS.
using LdsByte = __attribute__((address_space(3))) char;
__device__ __forceinline__ int lds_address(char* p) {
  return int(reinterpret_cast<uintptr_t>((LdsByte*)(p)));
}
template <int PLUS = 0>
__device__ __forceinline__ v4i lds16(int at) {
  const auto* p = reinterpret_cast<const LdsByte*>(static_cast<uintptr_t>(static_cast<unsigned>(at)));
  return *reinterpret_cast<const __attribute__((address_space(3))) v4i*>(p + PLUS);
}

typedef int v6i __attribute__((ext_vector_type(6)));

// Byte-shifted target words: w[i] = bytes [4 (FROM + i) + j, + 4) of the 32
// bytes (q, next). Column class c is four words from c on; operands start at
// even registers, so the even and the odd classes get six words of their own.
template <int FROM>
__device__ __forceinline__ v6i shifted_words(v4i q, v4i next, unsigned j) {
  const int d[8] = {q.x, q.y, q.z, q.w, next.x, next.y, next.z, next.w};
  v6i w;
#pragma unroll
  for (int i = 0; i < 6; ++i) w[i] = __builtin_amdgcn_alignbyte(d[FROM + i + 1], d[FROM + i], j);
  asm volatile("" : "+v"(w));  // kept together
  return w;
}

template <int CTRL>
__device__ __forceinline__ unsigned long long quad_perm(unsigned long long x) {
  const unsigned lo = __builtin_amdgcn_mov_dpp(int(unsigned(x)), CTRL, 0xf, 0xf, true);
  const unsigned hi = __builtin_amdgcn_mov_dpp(int(unsigned(x >> 32)), CTRL, 0xf, 0xf, true);
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// Sums over the four lanes of a quad, of x[r] in lane r of it.
__device__ __forceinline__ unsigned long long quad_sums(const unsigned long long (&x)[4]) {
  const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
  const unsigned long long y0 = (b0 ? x[1] : x[0]) + quad_perm<0xB1>(b0 ? x[0] : x[1]);
  const unsigned long long y1 = (b0 ? x[3] : x[2]) + quad_perm<0xB1>(b0 ? x[2] : x[3]);
  return (b1 ? y1 : y0) + quad_perm<0x4E>(b1 ? y0 : y1);
}

// Inclusive sum over the wave's lanes.
__device__ __forceinline__ unsigned long long wave_scan(unsigned long long v) {
  auto step = [&](auto CTRL, auto ROWS) {
    constexpr int c = decltype(CTRL)::value, rows = decltype(ROWS)::value;
    const unsigned lo = __builtin_amdgcn_update_dpp(0, int(unsigned(v)), c, rows, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, int(unsigned(v >> 32)), c, rows, 0xf, false);
    v += (static_cast<unsigned long long>(hi) << 32) | lo;
  };
  using std::integral_constant;
  step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});  // row_shr:1
  step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});  // row_shr:2
  step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});  // row_shr:4
  step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});  // row_shr:8
  step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});  // row_bcast:15
  step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});  // row_bcast:31
  return v;
}

// Cross sums of a task's tiles: W whole row sets, tiles 4 i + class, and with
// X one row set per class, tiles 4 W + class. planes: LDS address of the mode's byte planes,
// [component][digit][pl]; kst: place of the first step's first frame (16-byte
// boundary); off[i]: this lane's row's place offset in row set i. Lane (row or
// column l % 16: digit l % 4, row or shift (l / 4) % 4; time quarter l / 16).
// first: the 16 places before the first target hold older frames, no targets.
// Rows and columns are read one step ahead of their products.
template <int W, bool X>
__device__ __forceinline__ void cross_sums(v4i (&acc)[kMxTiles], const int (&off)[W + (X ? 4 : 0)],
                                           int planes, int pl, int kst, int steps, int amin,
                                           bool first) {
  constexpr int NR = W + (X ? 4 : 0);
  const int lane = threadIdx.x & 63;
  const unsigned j = (lane >> 2) & 3;
  const int quarter = lane >> 4;
#pragma unroll 1
  for (int comp = 0; comp < 2; ++comp) {
    const int base = planes + (comp * 4 + (lane & 3)) * pl;
    int at = base + kst + quarter * 16 * steps;
    // Rows below place amin are all zeros there; `low` bounds a read at +0,
    // low16 one at +16.
    const int low = base + amin;
    const int low16 = low - 16;
    int row_at[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) row_at[i] = at + off[i];
    v4i q0 = lds16(at), q1 = lds16<16>(at);
    if (first && quarter == 0) q0 = v4i{0, 0, 0, 0};
    v4i rows0[NR], rows1[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) rows0[i] = lds16(max(row_at[i], low));
    // Opaque to the optimiser, which would turn a loop-carried load back into
    // a load at its use.
    asm volatile("" : "+v"(q0), "+v"(q1));
#pragma unroll
    for (int i = 0; i < NR; ++i) asm volatile("" : "+v"(rows0[i]));
    // Products of one step.
    auto step = [&](v4i cur, v4i next, const v4i (&rows)[NR]) {
      const v6i even = shifted_words<0>(cur, next, j);
      unsigned j2 = j;
      asm volatile("" : "+v"(j2));
      const v6i odd = shifted_words<1>(cur, next, j2);
      const v4i col[4] = {__builtin_shufflevector(even, even, 0, 1, 2, 3),
                          __builtin_shufflevector(odd, odd, 0, 1, 2, 3),
                          __builtin_shufflevector(even, even, 2, 3, 4, 5),
                          __builtin_shufflevector(odd, odd, 2, 3, 4, 5)};
#pragma unroll
      for (int i = 0; i < W; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          acc[4 * i + c] =
              __builtin_amdgcn_mfma_i32_16x16x64_i8(rows[i], col[c], acc[4 * i + c], 0, 0, 0);
      if constexpr (X) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          acc[4 * W + c] =
              __builtin_amdgcn_mfma_i32_16x16x64_i8(rows[W + c], col[c], acc[4 * W + c], 0, 0, 0);
      }
    };
    int s = 0;
#pragma unroll 1
    for (; s + 1 < steps; s += 2) {
#pragma unroll
      for (int i = 0; i < NR; ++i)
        rows1[i] = lds16<16>(max(row_at[i], low16));
      const v4i q2 = lds16<32>(at);
      step(q0, q1, rows0);
      at += 32;
      asm volatile("" : "+v"(at));
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        row_at[i] += 32;
        asm volatile("" : "+v"(row_at[i]));  // kept, not formed again from a base
        rows0[i] = lds16(max(row_at[i], low));
      }
      const v4i q3 = lds16<16>(at);
      step(q1, q2, rows1);
      q0 = q2;
      q1 = q3;
    }
    if (s < steps) step(q0, q1, rows0);
  }
}

// Energy (sum of q^2) of both components over the frames of x's octet before
// plane place x, by byte dot products of the masked digits.
__device__ __forceinline__ unsigned long long energy_in_octet(const char* planes, int pl, int x) {
  const int r = x & 7;
  const char* p = planes + (x - r);
  const unsigned m0 = r >= 4 ? ~0u : (1u << (8 * r)) - 1u;
  const unsigned m1 = r <= 4 ? 0u : (1u << (8 * (r - 4))) - 1u;
  int same[4] = {0, 0, 0, 0};         // digit i with itself: 2^(16 i)
  int cross[6] = {0, 0, 0, 0, 0, 0};  // digits i < k, i + k = 1 .. 5: 2 * 2^(8 (i + k))
#pragma unroll
  for (int comp = 0; comp < 2; ++comp) {
    int lo[4], hi[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const uint2 w = *reinterpret_cast<const uint2*>(p + (comp * 4 + d) * pl);
      lo[d] = int(w.x & m0);
      hi[d] = int(w.y & m1);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      same[i] = __builtin_amdgcn_sdot4(lo[i], lo[i], same[i], false);
      same[i] = __builtin_amdgcn_sdot4(hi[i], hi[i], same[i], false);
#pragma unroll
      for (int k = i + 1; k < 4; ++k) {
        cross[i + k] = __builtin_amdgcn_sdot4(lo[i], lo[k], cross[i + k], false);
        cross[i + k] = __builtin_amdgcn_sdot4(hi[i], hi[k], cross[i + k], false);
      }
    }
  }
  // Product sums are at most 16 * 2^14, two of them in cross[3]; of the last line
  // the low 32 bits count.
  const int e0 = same[0] + cross[1] * (1 << 9);
  const int e16 = 2 * cross[2] + same[1] + cross[3] * (1 << 9);
  const unsigned e32 = 2 * unsigned(cross[4]) + unsigned(same[2]) + (unsigned(cross[5]) << 9) +
                       (unsigned(same[3]) << 16);
  return static_cast<unsigned long long>(static_cast<long long>(e0)) +
         (static_cast<unsigned long long>(static_cast<long long>(e16)) << 16) +
         (static_cast<unsigned long long>(e32) << 32);
}

// Energy of the frame at plane place x.
__device__ __forceinline__ unsigned long long energy_at(const char* planes, int pl, int x) {
  unsigned long long e = 0;
#pragma unroll
  for (int comp = 0; comp < 2; ++comp) {
    const signed char* p = reinterpret_cast<const signed char*>(planes) + comp * 4 * pl + x;
    const int q = p[0] + (p[pl] * (1 << 8)) + (p[2 * pl] * (1 << 16)) + (p[3 * pl] * (1 << 24));
    e += static_cast<unsigned long long>(static_cast<long long>(q) * q);
  }
  return e;
}

// Prefix of the energies at the octet of plane place x.
__device__ __forceinline__ unsigned long long prefix_at(const char* planes, int pl, int x) {
  return *reinterpret_cast<const unsigned long long*>(planes + 8 * pl + (x & ~7));
}

// Ring slot of plane place x, or -1 where no frame lies.
__device__ __forceinline__ int slot_at(const MxArgs& a, int x) {
  const bool old = x < a.split;
  const int f = x - (old ? a.obase : a.tbase);
  const int n = old ? a.olen : int(a.t1 - a.t0);
  uint32_t s = uint32_t(old ? a.slot_old : a.slot_new) + uint32_t(f);
  if (s >= uint32_t(a.capacity)) s -= uint32_t(a.capacity);
  return f >= 0 && f < n ? int(s) : -1;
}

// Stored words of a mode, and their value: decoded, scaled by 2^-e (16-bit
// storage) and corrected by d times the reference transform.
template <int SPEC>
using MxWord = std::conditional_t<SPEC == kSpecF32, float2, uint32_t>;
template <int SPEC>
__device__ __forceinline__ float2 decode(MxWord<SPEC> w, float d, float inv, float2 ref) {
  float2 v;
  if constexpr (SPEC == kSpecF32) {
    v = w;
  } else {
    v = SPEC == kSpecBF16 ? dev::unpack_bf16(w) : dev::unpack_f16(w);
    v.x *= inv;
    v.y *= inv;
  }
  return make_float2(fmaf(d, ref.x, v.x), fmaf(d, ref.y, v.y));
}

// A launch's sum of delay index l into the running sum.
__device__ __forceinline__ void add_sum(const MxArgs& a, int64_t mode, int l, float val) {
  float* sum = a.acc + mode * a.acc_pitch + l;
  if (a.comp) {
    // With Kahan compensation.
    float* comp = a.comp + mode * a.acc_pitch + l;
    if (a.assign) {
      *sum = val;
      *comp = 0.f;
    } else {
      const float was = *sum;
      const float y = val - *comp;
      const float t = was + y;
      *comp = (t - was) - y;
      *sum = t;
    }
  } else {
    *sum = a.assign ? val : *sum + val;
  }
}

// LDS after the planes, the rounds' totals and the sums of squares: the first delay
// with a small sum in the workgroup, then the small sums, a bit per mode and
// delay index.
__device__ __forceinline__ int* first_small_of(int km, int pl) {
  return reinterpret_cast<int*>(smem + km * (9 * pl + kMxRounds * kMxWaves * 8 + kMxWaves * 4));
}

// The kernel's arguments, read again: kept from its beginning on they would take
// the registers of its loops.
__device__ __forceinline__ const MxArgs& kernel_args() {
  auto* p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const MxArgs*)(p);
}

// The workgroup's small sums from the coefficients themselves, which take the
// planes' room: a wave a mode's delays on its lanes, FP32 terms into an FP64 sum.
template <int SPEC>
__device__ __forceinline__ void sum_small(const MxArgs& a, int64_t m0) {
  constexpr int THREADS = 64 * kMxWaves;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int km = 1 << a.km_log2, pl = a.pl, mode_lds = 9 * pl;
  const int tn = int(a.t1 - a.t0);
  const int* first_small = first_small_of(km, pl);
  const auto* small = reinterpret_cast<const unsigned*>(first_small + 1);
  // Their targets begin at place x0, their older frames end at x1.
  const int64_t least_lag = a.lags[*first_small];
  const int x0 = a.tbase + int(max(least_lag - a.t0, int64_t(0)));
  const int x1 = a.obase + int(a.t1 - least_lag - a.olo);
  const int lm = tid & (km - 1);
  const float2 ref = a.refspec[m0 + lm];
  const auto* ring = reinterpret_cast<const MxWord<SPEC>*>(a.ring) + m0 + lm;
  auto* values = reinterpret_cast<float2*>(smem + lm * mode_lds);
  for (int oct = tid >> a.km_log2; oct < pl >> 3; oct += THREADS >> a.km_log2) {
    if (8 * oct + 8 <= x0 && 8 * oct >= x1) continue;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int slot = slot_at(a, 8 * oct + i);
      const float4 f = a.fscale[max(slot, 0)];
      const float2 v = decode<SPEC>(ring[max(slot, 0) * a.mode_stride], f.y, f.z, ref);
      values[8 * oct + i] = slot >= 0 ? v : make_float2(0.f, 0.f);
    }
  }
  __syncthreads();
  for (int mm = wave; mm < km; mm += kMxWaves) {
    if (m0 + mm >= a.n_modes) continue;
    const auto* z = reinterpret_cast<const float2*>(smem + mm * mode_lds);
    for (int l0 = 0; l0 < a.tab.n_paired; l0 += 64) {
      const unsigned* bits = small + mm * (kMxLags / 32) + (l0 >> 5);
      const unsigned long long mask = (static_cast<unsigned long long>(bits[1]) << 32) | bits[0];
      if (!mask) continue;
      const bool mine = mask >> lane & 1;
      const int64_t lag0 = a.lags[l0 + __builtin_ctzll(mask)];
      const int64_t lag1 = a.lags[l0 + 63 - __builtin_clzll(mask)];
      const int64_t tau = mine ? int64_t(a.lags[l0 + lane]) : lag0;
      // Targets t0 + r, r >= first, and the older frames' places. From r1 on every
      // delay has pairs.
      const int first = int(max(tau - a.t0, int64_t(0)));
      const int r1 = int(max(lag1 - a.t0, int64_t(0)));
      const float2* target = z + a.tbase;
      const int older = int(a.t0 - tau - a.olo) + a.obase;
      double sum = 0.0;
      auto square = [&](int r, float2 o) {
        const float dx = target[r].x - o.x, dy = target[r].y - o.y;
        return double(fmaf(dx, dx, dy * dy));
      };
      int r = int(max(lag0 - a.t0, int64_t(0)));
      for (; r < r1; ++r) {
        const double d = square(r, z[max(older + r, 0)]);
        if (r >= first) sum += d;
      }
      for (; r + 8 <= tn; r += 8) {
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += square(r + i, z[older + r + i]);
      }
      for (; r < tn; ++r) sum += square(r, z[older + r]);
      if (mine) add_sum(a, m0 + mm, l0 + lane, float(sum));
    }
  }
}

template <int SPEC>
__global__ __launch_bounds__(64 * kMxWaves, 2) void pair_mx_kernel(const MxArgs a) {
  constexpr int THREADS = 64 * kMxWaves, ROUNDS = kMxRounds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int km = 1 << a.km_log2, pl = a.pl;
  const int mode_lds = 9 * pl;
  const int lds0 = lds_address(smem);
  auto* tot = reinterpret_cast<unsigned long long*>(smem + km * mode_lds);  // [rounds][waves][km]
  auto* squares = reinterpret_cast<float*>(tot + ROUNDS * kMxWaves * km);    // [waves][km]
  int* first_small = first_small_of(km, pl);
  auto* small = reinterpret_cast<unsigned*>(first_small + 1);
  if (tid == 0) *first_small = kMxLags;
  for (int e = tid; e < kMxLags / 32 * km; e += THREADS) small[e] = 0;

  // Workgroups are dispatched round robin over the 8 XCDs; neighbouring
  // workgroups, whose modes share lines of the ring, stay on one XCD's L2.
  const int per_xcd = int(gridDim.x) / 8;
  const int64_t m0 = int64_t((int(blockIdx.x) % 8) * per_xcd + int(blockIdx.x) / 8) << a.km_log2;
  if (m0 >= a.n_modes) return;

  // Delays without a pair in this window start at 0.
  if (a.assign && a.zero_from < a.n_lags) {
    for (int e = tid; e < (a.n_lags - a.zero_from) << a.km_log2; e += THREADS) {
      const int64_t m = m0 + (e & (km - 1));
      const int l = a.zero_from + (e >> a.km_log2);
      if (m < a.n_modes) {
        a.acc[m * a.acc_pitch + l] = 0.f;
        if (a.comp) a.comp[m * a.acc_pitch + l] = 0.f;
      }
    }
  }
  // Work counter: the (target, delay) pairs summed by this launch.
  if (a.work && blockIdx.x == 0) {
    unsigned long long n = 0;
    for (int l = tid; l < a.n_lags; l += THREADS) {
      const int64_t from = a.t0 > a.lags[l] ? a.t0 : int64_t(a.lags[l]);
      if (a.t1 > from) n += static_cast<unsigned long long>(a.t1 - from);
    }
    if (n) atomicAdd(a.work, n);
  }
  if (a.tab.n_tasks == 0) return;

  // ---- load: a thread's items are octets of 8 plane places of one mode ----
  const int lm = tid & (km - 1);
  const int64_t m = m0 + lm;
  const float2 R = a.refspec[m];
  const int octets = pl >> 3;
  const int step = THREADS >> a.km_log2;  // octets per round
  const int oct0 = tid >> a.km_log2;
  constexpr int MODE_BYTES = SPEC == kSpecF32 ? 8 : 4;
  const char* ring_m = a.ring + m * MODE_BYTES;
  const int64_t slot_bytes = a.mode_stride * MODE_BYTES;
  using Word = MxWord<SPEC>;
  // The frames' {d, 2^-e} by plane place ({0, 0} where none lies), in the room
  // that the planes take later.
  float* tab_d = reinterpret_cast<float*>(smem);
  float* tab_s = tab_d + pl;
  for (int x = tid; x < pl; x += THREADS) {
    const int slot = slot_at(a, x);
    const float4 f = a.fscale[max(slot, 0)];
    tab_d[x] = slot >= 0 ? f.y : 0.f;
    if constexpr (SPEC != kSpecF32) tab_s[x] = slot >= 0 ? f.z : 0.f;
  }
  Word raw[ROUNDS][8];
  if (a.direct) {
    // Rows before or past a range are out of the descriptor's bounds and
    // read as 0.
    const int64_t n_new = a.t1 - a.t0;
    const dev::BufferRsrc old_rows =
        dev::make_buffer(const_cast<char*>(a.ring + a.slot_old * slot_bytes),
                         uint32_t(a.olen * slot_bytes));
    const dev::BufferRsrc new_rows =
        dev::make_buffer(const_cast<char*>(a.ring + a.slot_new * slot_bytes),
                         uint32_t(n_new * slot_bytes));
    const uint32_t row = uint32_t(slot_bytes), col = uint32_t(m) * uint32_t(MODE_BYTES);
    auto load = [&](const dev::BufferRsrc& rs, int x0, Word (&w)[8]) {
      uint32_t off = uint32_t(x0) * row + col;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if constexpr (SPEC == kSpecF32) {
          const auto q = __builtin_amdgcn_raw_buffer_load_b64(rs, int(off), 0, 0);
          w[i] = make_float2(__uint_as_float(q[0]), __uint_as_float(q[1]));
        } else {
          w[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, int(off), 0, 0);
        }
        off += row;
      }
    };
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int oct = oct0 + r * step;
      if (oct < octets) {
        if (8 * oct < a.split)
          load(old_rows, 8 * oct - a.obase, raw[r]);
        else
          load(new_rows, 8 * oct - a.tbase, raw[r]);
      }
    }
  } else {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int oct = oct0 + r * step;
      if (oct < octets) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int slot = slot_at(a, 8 * oct + i);
          const Word w = *reinterpret_cast<const Word*>(ring_m + max(slot, 0) * slot_bytes);
          raw[r][i] = slot >= 0 ? w : Word{};
        }
      }
    }
  }
  __syncthreads();  // the table
  float2 v[ROUNDS][8];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int oct = oct0 + r * step;
    if (oct < octets) {
      float d[8], inv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        d[i] = tab_d[8 * oct + i];
        inv[i] = SPEC == kSpecF32 ? 0.f : tab_s[8 * oct + i];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) v[r][i] = decode<SPEC>(raw[r][i], d[i], inv[i], R);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[r][i] = make_float2(0.f, 0.f);
    }
  }
  float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
    for (int i = 0; i < 8; ++i)
      part[i & 3] = fmaf(v[r][i].x, v[r][i].x, fmaf(v[r][i].y, v[r][i].y, part[i & 3]));
  float square = (part[0] + part[1]) + (part[2] + part[3]);
  for (int o = km; o < 64; o <<= 1) square += __shfl_xor(square, o, 64);
  if (lane < km) squares[wave * km + lane] = square;
  __syncthreads();

  // The mode's sum of squares, which gives its scale 2^exponent. A mode whose
  // squares pass FP32, or lie where it loses them, becomes 0 here: all its sums
  // are small.
  static_assert(kMxWaves == 4, "a sum of four");
  auto squares_of = [&](int mode) -> float {
    return (squares[mode] + squares[km + mode]) + (squares[2 * km + mode] + squares[3 * km + mode]);
  };
  auto exponent = [](float e) -> int { return mx_exponent(__float_as_uint(kMxRoom * e)); };
  const float energy = squares_of(lm);
  if (!(energy <= kMxMost) || (energy < kMxFew && energy != 0.f)) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
      for (int i = 0; i < 8; ++i) v[r][i] = make_float2(0.f, 0.f);
  }
  const int ex = exponent(energy);
  unsigned long long sums[ROUNDS];
  char* const planes_m = smem + lm * mode_lds;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int oct = oct0 + r * step;
    unsigned long long e = 0;
    if (oct < octets) {
#pragma unroll
      for (int comp = 0; comp < 2; ++comp) {
        unsigned x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int q = int(rintf(ldexpf(comp ? v[r][i].y : v[r][i].x, ex)));
          e += static_cast<unsigned long long>(static_cast<long long>(q) * q);
          x[i] = unsigned(q) + 0x00808080u;
        }
        // Balanced base-256 digits: the bytes of q + 0x808080 with the low
        // three moved back by 128 each. Byte transposes of four words: plane d
        // takes byte d of each.
        unsigned out[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const unsigned* w = x + 4 * h;
          const unsigned a01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);
          const unsigned b01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
          const unsigned a23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
          const unsigned b23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
          out[h][0] = __builtin_amdgcn_perm(a23, a01, 0x05040100u) ^ 0x80808080u;
          out[h][1] = __builtin_amdgcn_perm(a23, a01, 0x07060302u) ^ 0x80808080u;
          out[h][2] = __builtin_amdgcn_perm(b23, b01, 0x05040100u) ^ 0x80808080u;
          out[h][3] = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
        }
#pragma unroll
        for (int d = 0; d < 4; ++d)
          *reinterpret_cast<uint2*>(planes_m + (comp * 4 + d) * pl + 8 * oct) =
              make_uint2(out[0][d], out[1][d]);
      }
    }
    sums[r] = e;
    if (r * step >= octets) continue;
    // Inclusive sum over the wave's octets of the mode (lanes km apart).
    for (int o = km; o < 64; o <<= 1) {
      const unsigned long long up =
          (static_cast<unsigned long long>(unsigned(__shfl_up(int(sums[r] >> 32), o, 64))) << 32) |
          unsigned(__shfl_up(int(unsigned(sums[r])), o, 64));
      if (lane >= o) sums[r] += up;
    }
    if (lane >= 64 - km) tot[(r * kMxWaves + wave) * km + lm] = sums[r];
    sums[r] -= e;  // exclusive
  }
  __syncthreads();
  {
    unsigned long long run = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      if (r * step >= octets) continue;
#pragma unroll
      for (int w = 0; w < kMxWaves; ++w) {
        if (w == wave) sums[r] += run;
        run += tot[(r * kMxWaves + w) * km + lm];
      }
      const int oct = oct0 + r * step;
      if (oct < octets)
        *reinterpret_cast<unsigned long long*>(planes_m + 8 * pl + 8 * oct) = sums[r];
    }
  }
  __syncthreads();

  // ---- products: waves take modes, and tasks when there are more waves ----
  const int tn = int(a.t1 - a.t0);
  const int share = km < kMxWaves ? kMxWaves / km : 1;
  for (int t = share > 1 ? wave >> a.km_log2 : 0; t < a.tab.n_tasks; t += share) {
    const MxTask task = a.tab.task[t];
    const int kst = a.tbase - 16 + 16 * task.start;
    const int steps = ((tn + 16 - 16 * task.start + 15) / 16 + 3) / 4;  // mx_steps
    // The task's tables, once for all modes: this lane's row of each row set,
    // and the first delays.
    int off[kMxSets + 4];
#pragma unroll
    for (int i = 0; i < kMxSets + 4; ++i)
      off[i] = a.aoff - a.tab.lag0 -
               16 * int(a.tab.block[min(task.rows0 + i, kMxRows - 1)][(lane >> 2) & 3]);
    unsigned codes[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
      codes[k] = a.tab.order[task.first + min(64 * k + lane, max(int(task.count) - 1, 0))];

    for (int mm = wave & (km - 1); mm < km; mm += kMxWaves) {
      const char* planes = smem + mm * mode_lds;
      const int back = -2 * exponent(squares_of(mm));
      const bool stored = m0 + mm < a.n_modes;

      // Energies of a delay: targets [from, t1) and older frames [from - tau,
      // t1 - tau), from = max(t0, tau). The prefix at t1 is the total; that at
      // t0 is wanted by delays up to t0 only.
      const unsigned long long total = prefix_at(planes, pl, pl - 8);
      unsigned long long at_t0 = 0;
      if (a.t0 > 0) at_t0 = prefix_at(planes, pl, a.tbase);
      // S of delay index l into the running sums, or to the small ones. A mode
      // of zeros has no small sums.
      static_assert(kMxLeast << 32 == 0, "the high word decides");
      const unsigned least = squares_of(mm) == 0.f ? 0 : unsigned(kMxLeast >> 32);
      auto put = [&](int l, unsigned long long S) {
        if (unsigned(S >> 32) < least) {
          atomicOr(&small[mm * (kMxLags / 32) + (l >> 5)], 1u << (l & 31));
          atomicMin(first_small, l);
          return;
        }
        add_sum(a, m0 + mm, l, float(ldexp(double(S), back)));
      };
      // Four tiles' sums (lane: delay place lane / 4, target digit lane % 4) to
      // cross sums modulo 2^64: class lane % 4 of place lane / 4.
      auto cross_of = [&](const v4i* c) -> unsigned long long {
        unsigned long long x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          long long y = c[k].x;
          y += static_cast<long long>(c[k].y) * (1 << 8);
          y += static_cast<long long>(c[k].z) * (1 << 16);
          y += static_cast<long long>(c[k].w) * (1 << 24);
          x[k] = static_cast<unsigned long long>(y) << (8 * (lane & 3));
        }
        return quad_sums(x);
      };
      auto from_lane = [](unsigned long long v, int l) -> unsigned long long {
        const unsigned lo = unsigned(__shfl(int(unsigned(v)), l, 64));
        const unsigned hi = unsigned(__shfl(int(unsigned(v >> 32)), l, 64));
        return (static_cast<unsigned long long>(hi) << 32) | lo;
      };
      auto clamped = [&](int x) { return min(max(x, 0), pl - 1); };
      auto prefix = [&](int x) { return prefix_at(planes, pl, x) + energy_in_octet(planes, pl, x); };
      // The sums of a task's sets: runs of consecutive delays with the energies
      // by a sum over the lanes, the other delays 64 at a time.
      auto finish = [&](const unsigned long long (&cross)[kMxSets + 1]) {
        unsigned long long next_e = 0;
        int next_lag = -1;
        dev::static_for<kMxSets>([&](auto I) {
          constexpr int i = decltype(I)::value;
          if (i >= task.sets) return;
          const unsigned run = a.tab.run[task.run0 + i];
          if (!run) return;
          const int l0 = int(a.tab.lag0) + 16 * a.tab.block[task.rows0 + i][0];
          const bool late = l0 + int(run >> 9 & 63) >= a.t0;  // a pair's first target is frame tau
          // Place of the older range's end, and of the first target (late) or
          // the older range's start, for delay l0.
          const int xe = int(a.t1 - a.olo) + a.obase - l0;
          const int xs = late ? l0 - int(a.t0) + a.tbase : int(a.t0 - a.olo) + a.obase - l0;
          if (next_lag != l0)
            next_e = (late ? total : total - at_t0) + prefix(clamped(xe)) - prefix(clamped(xs));
          // One more delay drops the last older frame, and the first target or
          // (early) takes in an older frame more.
          unsigned long long drop = energy_at(planes, pl, clamped(xe - 1 - lane));
          if (late)
            drop += energy_at(planes, pl, clamped(xs + lane));
          else
            drop -= energy_at(planes, pl, clamped(xs - 1 - lane));
          const unsigned long long sum = wave_scan(drop);
          const unsigned long long E = next_e - (sum - drop);
          const unsigned long long all =
              (static_cast<unsigned long long>(
                   unsigned(__builtin_amdgcn_readlane(int(unsigned(sum >> 32)), 63))) << 32) |
              unsigned(__builtin_amdgcn_readlane(int(unsigned(sum)), 63));
          next_e -= all;
          next_lag = l0 + 64 <= a.t0 || late ? l0 + 64 : -1;
          // Delay l0 + lane: row lane / 16, class (lane / 4) % 4, shift lane % 4.
          const unsigned long long c = from_lane(
              cross[i], (lane & 48) + 4 * (lane & 3) + ((lane >> 2) & 3));
          const int p0 = run >> 9 & 63, p1 = run >> 15 & 63;
          if (lane >= p0 && lane <= p1 && stored) put(int(run & 511) + lane - p0, E - 2 * c);
        });
        for (int k0 = 0; k0 < task.count; k0 += 64) {
          const bool mine = k0 + lane < task.count;
          const unsigned code = k0 == 0   ? codes[0]
                                : k0 == 64 ? codes[1]
                                           : a.tab.order[task.first + (mine ? k0 + lane : 0)];
          const int l = code & 511, set = (code >> 9) & 15, row = (code >> 13) & 3;
          const int tau = int(code >> 15) + a.tab.lag0;
          const int src = 16 * row + 4 * (tau & 3) + ((tau >> 2) & 3);
          const unsigned sets = a.tab.chunk[task.chunk0 + k0 / 64];
          unsigned long long c = 0;
          dev::static_for<kMxSets + 1>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if (!(sets >> i & 1)) return;
            const unsigned long long got = from_lane(cross[i], src);
            if (set == i) c = got;
          });
          const bool late = tau > a.t0;
          const int x0 = late ? int(tau - a.t0) + a.tbase : int(a.t0 - tau - a.olo) + a.obase;
          const int x1 = int(a.t1 - tau - a.olo) + a.obase;
          const unsigned long long E = (late ? total : total - at_t0) + prefix(x1) - prefix(x0);
          if (mine && stored) put(l, E - 2 * c);
        }
      };

      unsigned long long cross[kMxSets + 1] = {};
      auto go = [&](auto SETS, auto SCAT) {
        constexpr int W = decltype(SETS)::value;
        constexpr bool X = decltype(SCAT)::value;
        constexpr int NR = W + (X ? 4 : 0), T = 4 * (W + (X ? 1 : 0));
        if constexpr (NR > 0) {
          v4i acc[kMxTiles];
#pragma unroll
          for (int i = 0; i < T; ++i) acc[i] = v4i{0, 0, 0, 0};
          int rows[NR];
#pragma unroll
          for (int i = 0; i < NR; ++i) rows[i] = off[i];
          cross_sums<W, X>(acc, rows, lds0 + mm * mode_lds, pl, kst, steps, a.amin,
                           task.start == 0);
#pragma unroll
          for (int i = 0; i < T / 4; ++i) cross[i] = cross_of(acc + 4 * i);
        }
      };
      dev::static_for<kMxSets + 1>([&](auto SETS) {
        if (task.sets != decltype(SETS)::value) return;
        if (task.scattered)
          go(SETS, std::true_type{});
        else
          go(SETS, std::false_type{});
      });
      finish(cross);
    }
  }

  __syncthreads();
  if (*first_small != kMxLags) sum_small<SPEC>(kernel_args(), m0);
}

}  // namespace

hipError_t launch_pairs_mx(const void* ring, int spec, const float2* refspec,
                           const float4* fscale, int64_t n_modes, int64_t mode_stride,
                           int64_t capacity, const MxShape& s, const MxTables& tab,
                           const int32_t* lags, int n_lags, float* acc, float* comp,
                           int acc_pitch, bool assign, unsigned long long* work,
                           hipStream_t stream) {
  if (s.km != 4 && s.km != 8 && s.km != 16) return hipErrorInvalidValue;
  if (s.pl % 8 || (int64_t(s.pl) / 8) * s.km > kMxRounds * 64 * kMxWaves) return hipErrorInvalidValue;
  if (s.lds > size_t(kMxLds)) return hipErrorInvalidValue;
  MxArgs a;
  a.ring = static_cast<const char*>(ring);
  a.refspec = refspec;
  a.fscale = fscale;
  a.acc = acc;
  a.comp = comp;
  a.lags = lags;
  a.work = work;
  a.n_modes = n_modes;
  a.mode_stride = mode_stride;
  a.t0 = s.t0;
  a.t1 = s.t1;
  a.capacity = int32_t(capacity);
  a.slot_old = int32_t(s.olo % capacity);
  a.slot_new = int32_t(s.t0 % capacity);
  a.olen = s.olen;
  a.obase = s.obase;
  a.tbase = s.tbase;
  a.split = s.split;
  a.pl = s.pl;
  a.aoff = s.aoff;
  a.amin = s.amin;
  a.km_log2 = s.km == 16 ? 4 : s.km == 8 ? 3 : 2;
  a.olo = s.olo;
  a.n_lags = n_lags;
  a.acc_pitch = acc_pitch;
  a.assign = assign;
  a.zero_from = tab.n_paired;
  a.direct = mx_direct(s, capacity, mode_stride * (spec == kSpecF32 ? 8 : 4));
  a.tab = tab;
  const int64_t blocks = ((n_modes + s.km - 1) / s.km + 7) / 8 * 8;
#define NFS_MX_GO(SPECV)                                                                        \
  do {                                                                                          \
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&pair_mx_kernel<SPECV>),            \
                              hipFuncAttributeMaxDynamicSharedMemorySize, kMxLds);             \
    hipLaunchKernelGGL((pair_mx_kernel<SPECV>), dim3(unsigned(blocks)), dim3(64 * kMxWaves),   \
                       s.lds, stream, a);                                                      \
  } while (0)
  if (spec == kSpecF32)
    NFS_MX_GO(kSpecF32);
  else if (spec == kSpecBF16)
    NFS_MX_GO(kSpecBF16);
  else
    NFS_MX_GO(kSpecF16);
#undef NFS_MX_GO
  return hipGetLastError();
}

}  // namespace nfs
