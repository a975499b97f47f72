// Azimuthal average of the per-lag sums into rings of |q| (text after
// Eq. 1 and Fig. 1e-f), and the average over pairs per delay (processing
// section: the average for every delay is stored).
//
// Ring b is the set of modes with lo_b <= |k|^2 < hi_b. Each half-plane
// mode stands for itself and its mirror -k (weight 2) except on k_x = 0,
// where both k and -k are stored (weight 1). The plan lists the slots of
// every ring's stored modes with their weights (the binning table) and cuts
// each ring's list into segments of at most kSegModes modes.
//
// The sums are mode-major per slot, so each mode's lag sums are one
// contiguous read. One workgroup sums one segment for a chunk of up to 64 lags:
// each wave takes 64 table entries (one per lane), then walks them with the
// lags on LG = 8, 16, 32 or 64 lanes and 64 / LG entries side by side, eight
// reads in flight; the entries' sums meet by shuffles and in LDS. Where every
// ring is one segment (up to kSegModes modes: n <= 128 with rings of width 1)
// that is its sum; elsewhere a second kernel adds the segments of each ring in
// order. (A workgroup for each ring of any size leaves the chip idle: 23
// against 13 + 5 us with rings of up to 402 modes, 32 lags; 68 against 40 + 5
// with up to 1608, 50 lags.) All sums are FP64 in a fixed order, so D is
// bitwise reproducible.
//
// Bound by the gather of n_lags * 4 bytes per mode. A workgroup per segment
// that walked the lag chunks one after the other, then always the second
// kernel, took 970 + 8 us on 512 x 512 modes with 2047 lags (0.84 GB: 600
// workgroups, each with 32 chunks in a row), 121 + 7 us on 2048 x 2048 with 16
// and 22 + 4 us on 128 x 128 with 5 lags (16 and 5 of 64 lanes at work); now
// 321 + 8 us (2.6 TB/s), 43 + 7 us and 8 us. 1024 x 1024 with 50 lags stays at
// 40 + 5 us.
#include "nfs.h"
#include "nfs_device.hpp"
#include "nfs_host.hpp"
#include "nfs_kernels.hpp"

namespace nfs {
namespace {

constexpr int kSegThreads = 256;
static_assert(kSegModes == kSegThreads, "one table entry per thread of a segment");

// Outputs of a ring: D, its modes, and with ring 0 the pairs and the status.
struct BinOut {
  const int32_t* lags;
  int64_t n_frames;
  const int32_t* status;
  double* D;
  int64_t* counts;
  int64_t* pairs;
  int32_t* status_out;
};

__device__ __forceinline__ void write_bin(const BinOut& o, int nb, int b, int l, double sum,
                                          long long C) {
  const int64_t np = o.n_frames - o.lags[l] > 0 ? o.n_frames - o.lags[l] : 0;
  o.D[int64_t(l) * nb + b] =
      (np > 0 && C > 0) ? sum / (double(C) * double(np)) : __builtin_nan("");
  if (l == 0 && o.counts) o.counts[b] = C;
  if (b == 0) {
    if (o.pairs) o.pairs[l] = np;
    if (l == 0 && o.status_out)
      o.status_out[0] = (o.status[0] & 2)   ? NFS_E_TIMEOUT
                        : (o.status[0] & 1) ? NFS_E_DEGENERATE_FRAME
                                            : NFS_OK;
  }
}

// Block x: segment x, which without PART is all of ring x; with PART its sums go
// to part and part_cnt. Block y: lags LG * y .. .
template <int LG, bool PART>
__global__ void bin_sum_kernel(const float* __restrict__ acc, int n_lags,
                               const int32_t* __restrict__ bin_slots,
                               const int32_t* __restrict__ seg_first, double* __restrict__ part,
                               long long* __restrict__ part_cnt, int nb, BinOut out) {
  constexpr int EPS = 64 / LG;  // entries side by side
  constexpr int U = 8;
  constexpr int kWaves = kSegThreads / 64;
  __shared__ double red[kWaves][LG];
  __shared__ int redc[kWaves];
  const int x = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i0 = seg_first[x] + wave * 64;
  const int cnt = max(0, min(64, seg_first[x + 1] - i0));  // wave-uniform
  const int l = blockIdx.y * LG + lane % LG;
  const bool lag_ok = l < n_lags;
  const int code = lane < cnt ? bin_slots[i0 + lane] : 0;
  int wsum = lane < cnt ? (code & 1) + 1 : 0;
  double s = 0.0;
  for (int j = 0; j < cnt; j += U * EPS) {
    float v[U];
    int c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = j + u * EPS + lane / LG;
      c[u] = LG == 64 ? __builtin_amdgcn_readlane(code, (j + u) & 63) : __shfl(code, e & 63, 64);
      v[u] = (e < cnt && lag_ok) ? acc[int64_t(c[u] >> 1) * n_lags + l] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s += ((c[u] & 1) ? 2.0 : 1.0) * double(v[u]);
  }
#pragma unroll
  for (int o = LG; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) wsum += __shfl_xor(wsum, o, 64);
  if (lane < LG) red[wave][lane] = s;
  if (lane == 0) redc[wave] = wsum;
  __syncthreads();
  if (threadIdx.x >= LG || !lag_ok) return;
  double t = 0.0;
  long long C = 0;
  for (int w = 0; w < kWaves; ++w) {
    t += red[w][lane];
    C += redc[w];
  }
  if constexpr (PART) {
    part[int64_t(x) * n_lags + l] = t;
    if (l == 0) part_cnt[x] = C;
  } else {
    write_bin(out, nb, x, l, t, C);
  }
}

__global__ void bin_final_kernel(int nb, int n_lags, const double* __restrict__ part,
                                 const long long* __restrict__ part_cnt,
                                 const int32_t* __restrict__ bin_seg0, BinOut out) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= int64_t(nb) * n_lags) return;
  const int b = int(i / n_lags), l = int(i % n_lags);
  const int s0 = bin_seg0[b], s1 = bin_seg0[b + 1];
  double sum = 0.0;
  long long C = 0;
  for (int s = s0; s < s1; ++s) {
    sum += part[int64_t(s) * n_lags + l];
    C += part_cnt[s];
  }
  write_bin(out, nb, b, l, sum, C);
}

template <int LG>
void bins_go(int n_bins, const float* acc, int n_lags, const int32_t* bin_slots,
             const int32_t* seg_first, int n_segs, const int32_t* bin_seg0, double* part,
             long long* part_cnt, const BinOut& out, hipStream_t s) {
  const dim3 grid(unsigned(n_segs), unsigned((n_lags + LG - 1) / LG));
  if (n_segs == n_bins) {  // every ring has at least one segment
    hipLaunchKernelGGL((bin_sum_kernel<LG, false>), grid, dim3(kSegThreads), 0, s, acc, n_lags,
                       bin_slots, seg_first, part, part_cnt, n_bins, out);
    return;
  }
  hipLaunchKernelGGL((bin_sum_kernel<LG, true>), grid, dim3(kSegThreads), 0, s, acc, n_lags,
                     bin_slots, seg_first, part, part_cnt, n_bins, out);
  const int64_t items = int64_t(n_bins) * n_lags;
  hipLaunchKernelGGL(bin_final_kernel, dim3(unsigned((items + 255) / 256)), dim3(256), 0, s,
                     n_bins, n_lags, part, part_cnt, bin_seg0, out);
}

}  // namespace

hipError_t launch_bins(int n_bins, const float* acc, int n_lags, const int32_t* bin_slots,
                       const int32_t* seg_first, int n_segs, const int32_t* bin_seg0,
                       double* part, long long* part_cnt, const int32_t* lags,
                       int64_t n_frames, const int32_t* status, double* D, int64_t* counts,
                       int64_t* pairs, int32_t* status_out, hipStream_t s) {
  const BinOut out{lags, n_frames, status, D, counts, pairs, status_out};
#define NFS_BINS_GO(LG)                                                                     \
  bins_go<LG>(n_bins, acc, n_lags, bin_slots, seg_first, n_segs, bin_seg0, part, part_cnt, \
              out, s)
  if (n_lags <= 8)
    NFS_BINS_GO(8);
  else if (n_lags <= 16)
    NFS_BINS_GO(16);
  else if (n_lags <= 32)
    NFS_BINS_GO(32);
  else
    NFS_BINS_GO(64);
#undef NFS_BINS_GO
  return hipGetLastError();
}

}  // namespace nfs
