// Pair sums of short windows: every frame that the window's pairs need fits the
// LDS of a workgroup at once, next to those of other workgroups of the CU.
//
// One workgroup owns K = 16 or 32 consecutive modes. It copies the window's
// frames and the max_lag frames before them to LDS in one go (all its loads are
// in flight together), waits once, and sums all its lags from there. The history
// form of the kernel walks the window in chunks of 32 frames with a barrier and a
// load that little covers in each; over a few chunks that chain, not the loads or
// the arithmetic, is its time: 96 frames of 2048 x 2048 with 16 lags 1021 us, of
// which the loads need 260 and the arithmetic 400; here 594.
//
// The sums of a workgroup are cut into tasks of (up to 4 lags) x (every
// n_slices-th block of 64 / K * 8 target frames); waves take them in turn. In a
// task a lane owns one mode and 8 consecutive target frames of each block, read
// once for the task's lags; per pair one LDS read of the older frame (lags that
// are consecutive integers share a register window of them), two subtractions
// and two FMAs, each sum a plain FP32 chain per lane. The lanes' and the tasks'
// sums are then added in a fixed order. Sets of 8 lags took 90 to 170 registers
// and with them the waves that hide the LDS latency (256 frames, 32 lags: 192
// against 168 us); bounded to 128 registers they spilled (382 us). The
// register bound asks for 3 waves per SIMD with K = 16 and 4 with K = 32: for the
// 96 frames above one wave more takes 661 us, two 1246.
#include "nfs_device.hpp"
#include "nfs_kernels.hpp"
#include "pair_plan.hpp"

namespace nfs {
namespace {
using dev::kSpecBF16;
using dev::kSpecF32;
using dev::unpack_bf16;
using dev::unpack_f16;

constexpr int RPT = 8;            // target rows per lane and block
constexpr int GUARD = kWinGuard;  // rows before the window that a masked lane may read
static_assert(GUARD == RPT - 1, "a run starts at most one row short of wholly outside");

template <int K, int P, int NW, bool F32>
__global__ __launch_bounds__(64 * NW, (K == 32 ? 4 : 3)) void pair_window_kernel(
    const char* __restrict__ ring, int spec, const float2* __restrict__ refspec,
    const float4* __restrict__ fscale, int64_t n_modes, int64_t mode_stride, int capacity,
    int slot0, int rows, int pre, const int32_t* __restrict__ lags, int n_lags, int n_sets,
    int n_slices, float* __restrict__ acc, int acc_pitch, bool assign,
    unsigned long long* __restrict__ work) {
  constexpr int BLK = 64 / K * RPT;  // target rows per block
  extern __shared__ float2 lds[];  // [GUARD + rows][K], then the tasks' sums
  float2* hist = lds + GUARD * K;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Neighbouring tiles share lines of 128 bytes where modes have 4 bytes: each
  // XCD (workgroups go round robin over the 8) takes a run of tiles.
  int tile = blockIdx.x;
  if (gridDim.x % 8 == 0) tile = (tile % 8) * int(gridDim.x / 8) + tile / 8;
  const int64_t m0 = int64_t(tile) * K;

  // Row r: the frame in ring slot slot0 + r. A thread always copies the same
  // 16 bytes of a row (2 FP32 modes or 4 of 16 bits), so their reference values
  // stay in registers.
  {
    constexpr int PER = F32 ? 2 : 4;   // modes per load
    constexpr int COLS = K / PER;
    constexpr int STEP = 64 * NW / COLS;  // rows per pass of the workgroup
    constexpr int U = 4;
    const int col = tid % COLS;
    const int64_t mode_bytes = F32 ? 8 : 4;
    const char* base = ring + (m0 + col * PER) * mode_bytes;
    const int64_t slot_bytes = mode_stride * mode_bytes;
    float2 R[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) R[i] = refspec[m0 + col * PER + i];
    for (int r0 = tid / COLS; r0 < rows; r0 += U * STEP) {
      float4 raw[U], sc[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = min(r0 + u * STEP, rows - 1);
        int slot = slot0 + r;
        if (slot >= capacity) slot -= capacity;
        raw[u] = *reinterpret_cast<const float4*>(base + slot * slot_bytes);
        sc[u] = fscale[slot];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * STEP;
        if (r >= rows) continue;
        float2* dst = hist + r * K + col * PER;
        const float d = sc[u].y, s = sc[u].z;
        float2 v[PER];
        if constexpr (F32) {
          v[0] = make_float2(raw[u].x, raw[u].y);
          v[1] = make_float2(raw[u].z, raw[u].w);
        } else {
          const float w[4] = {raw[u].x, raw[u].y, raw[u].z, raw[u].w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t b = __float_as_uint(w[i]);
            const float2 a = spec == kSpecBF16 ? unpack_bf16(b) : unpack_f16(b);
            v[i] = make_float2(a.x * s, a.y * s);
          }
        }
#pragma unroll
        for (int i = 0; i < PER; ++i)
          v[i] = make_float2(fmaf(d, R[i].x, v[i].x), fmaf(d, R[i].y, v[i].y));
#pragma unroll
        for (int i = 0; i < PER; i += 2)
          *reinterpret_cast<float4*>(dst + i) = make_float4(v[i].x, v[i].y, v[i + 1].x, v[i + 1].y);
      }
    }
  }
  __syncthreads();

  float* sums = reinterpret_cast<float*>(hist + rows * K);  // [n_slices][K][n_lags]
  const int m = lane % K, g = lane / K;
  const float2* mine = hist + g * RPT * K + m;
  const int blocks = (rows - pre + BLK - 1) / BLK;
  const int base = n_lags / n_sets, extra = n_lags % n_sets;
  for (int task = (wave + blockIdx.x) % NW; task < n_sets * n_slices; task += NW) {
    const int set = task % n_sets, slice = task / n_sets;
    const int l0 = set * base + min(set, extra);
    const int count = base + (set < extra ? 1 : 0);  // P or P - 1
    int tau[P];
#pragma unroll
    for (int s = 0; s < P; ++s)
      tau[s] = __builtin_amdgcn_readfirstlane(lags[l0 + min(s, count - 1)]);
    const bool consecutive = P > 2 && count == P && tau[P - 1] - tau[0] == P - 1;
    float ax[P], ay[P];
#pragma unroll
    for (int s = 0; s < P; ++s) ax[s] = ay[s] = 0.f;
    for (int b = slice; b < blocks; b += n_slices) {
      // Blocks end at the window's last row, so only their beginning can lie
      // outside: targets before `pre` or without a partner.
      const int r0 = rows - (b + 1) * BLK;
      const int t0 = r0 + g * RPT;
      float2 cur[RPT];
      {
        const float2* src = hist + max(t0, -GUARD) * K + m;
#pragma unroll
        for (int i = 0; i < RPT; ++i) cur[i] = src[i * K];
      }
      if (r0 >= max(pre, tau[P - 1])) {
        auto add = [&](const float2* old, auto S) {
          constexpr int s = decltype(S)::value;
#pragma unroll
          for (int i = 0; i < RPT; ++i) {
            const float dx = cur[i].x - old[i].x, dy = cur[i].y - old[i].y;
            ax[s] = fmaf(dx, dx, ax[s]);
            ay[s] = fmaf(dy, dy, ay[s]);
          }
        };
        if (consecutive) {
          constexpr int WL = RPT + P - 1;
          float2 win[WL];
          const float2* src = mine + (r0 - tau[P - 1]) * K;
#pragma unroll
          for (int i = 0; i < WL; ++i) win[i] = src[i * K];
          dev::static_for<P>([&](auto S) { add(win + (P - 1 - decltype(S)::value), S); });
        } else {
          dev::static_for<P>([&](auto S) {
            constexpr int s = decltype(S)::value;
            if (s + 1 < P || count == P) {
              float2 old[RPT];
              const float2* src = mine + (r0 - tau[s]) * K;
#pragma unroll
              for (int i = 0; i < RPT; ++i) old[i] = src[i * K];
              add(old, S);
            }
          });
        }
      } else {
        // Targets outside count 0: a lane's run starts at most GUARD rows
        // before the window, or wholly outside.
        dev::static_for<P>([&](auto S) {
          constexpr int s = decltype(S)::value;
          const int from = max(pre, tau[s]);
          if ((s + 1 < P || count == P) && r0 + BLK > from) {
            const float2* src = hist + max(t0 - tau[s], -GUARD) * K + m;
            const int lo = from - t0;
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
              const float2 o = src[i * K];
              const float dx = i >= lo ? cur[i].x - o.x : 0.f;
              const float dy = i >= lo ? cur[i].y - o.y : 0.f;
              ax[s] = fmaf(dx, dx, ax[s]);
              ay[s] = fmaf(dy, dy, ay[s]);
            }
          }
        });
      }
    }
#pragma unroll
    for (int s = 0; s < P; ++s) {
      float v = ax[s] + ay[s];
#pragma unroll
      for (int o = K; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
      if (g == 0 && s < count) sums[(slice * K + m) * n_lags + l0 + s] = v;
    }
  }
  __syncthreads();
  const int64_t kmax = n_modes - m0 < K ? n_modes - m0 : K;
  for (int e = tid; e < int(kmax) * n_lags; e += 64 * NW) {
    float v = sums[e];
    for (int q = 1; q < n_slices; ++q) v += sums[q * K * n_lags + e];
    const int64_t at = (m0 + e / n_lags) * acc_pitch + e % n_lags;
    acc[at] = assign ? v : acc[at] + v;
  }
  // Work counter: the (target, lag) pairs summed.
  if (work && blockIdx.x == 0 && wave == 0) {
    unsigned long long pairs = 0;
    for (int l = lane; l < n_lags; l += 64) pairs += max(0, rows - max(pre, lags[l]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) pairs += __shfl_xor(pairs, o, 64);
    if (lane == 0) atomicAdd(work, pairs);
  }
}

}  // namespace

hipError_t launch_pairs_window(const void* ring, int spec, const float2* refspec,
                               const float4* fscale, int64_t n_modes, int64_t mode_stride,
                               int64_t capacity, int64_t T0, int64_t T1, const int32_t* lags,
                               const WindowShape& w, float* acc, int acc_pitch, bool assign,
                               unsigned long long* work, hipStream_t s) {
  const int per = (w.n_lags + w.sets - 1) / w.sets;
  const int slot0 = int((T0 - w.pre) % capacity);
  const int rows = w.pre + int(T1 - T0);
  const dim3 grid(unsigned((n_modes + w.modes - 1) / w.modes)), block(unsigned(64 * w.waves));
  const char* r = static_cast<const char*>(ring);
#define NFS_WIN_GO(KK, PP, NWW, F32V)                                                         \
  do {                                                                                        \
    (void)hipFuncSetAttribute(                                                                \
        reinterpret_cast<const void*>(&pair_window_kernel<KK, PP, NWW, F32V>),                \
        hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);                               \
    hipLaunchKernelGGL((pair_window_kernel<KK, PP, NWW, F32V>), grid, block, w.lds, s, r,     \
                       spec, refspec, fscale, n_modes, mode_stride, int(capacity), slot0,     \
                       rows, w.pre, lags, w.n_lags, w.sets, w.slices, acc, acc_pitch, assign, \
                       work);                                                                 \
  } while (0)
#define NFS_WIN_SPEC(KK, PP, NWW)                                                             \
  if (spec == kSpecF32) NFS_WIN_GO(KK, PP, NWW, true); else NFS_WIN_GO(KK, PP, NWW, false)
#define NFS_WIN_CASE(PP)                                                                      \
  case PP:                                                                                    \
    if (w.modes == 32) NFS_WIN_SPEC(32, PP, 4);                                               \
    else if (w.waves == 4) NFS_WIN_SPEC(16, PP, 4);                                           \
    else NFS_WIN_SPEC(16, PP, 8);                                                             \
    break;
  if (!(w.modes == 16 && (w.waves == 4 || w.waves == 8)) && !(w.modes == 32 && w.waves == 4))
    return hipErrorInvalidValue;
  static_assert(kWinLags == 4, "a case for each number of lags");
  switch (per) {
    NFS_WIN_CASE(1)
    NFS_WIN_CASE(2)
    NFS_WIN_CASE(3)
    NFS_WIN_CASE(4)
    default: return hipErrorInvalidValue;
  }
#undef NFS_WIN_CASE
#undef NFS_WIN_SPEC
#undef NFS_WIN_GO
  return hipGetLastError();
}

}  // namespace nfs
