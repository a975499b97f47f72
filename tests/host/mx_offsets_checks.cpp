// Byte offsets of the matrix-core pair kernel's buffer loads: for rows of real
// plans and windows around the sizes where a window's rows reach 4 GiB, every
// place of every launch that may use them is formed as the kernel does, in 32
// bits. Places of frames have to give that frame's bytes, all others an offset
// past the descriptor, which reads as 0.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "nfs_host.hpp"
#include "pair_matrix.hpp"

using namespace nfs;

namespace {

long long g_places = 0, g_direct = 0, g_wrong = 0;

void check_launch(const MxShape& s, int64_t row, int64_t mode_bytes, const char* what) {
  // One range's descriptor as the kernel makes it: `n` rows from its first.
  auto range = [&](int from, int to, int base, int64_t n) {
    const uint32_t records = uint32_t(n * row);
    for (int oct = from / 8; oct < to / 8; ++oct)
      for (int64_t col : {int64_t(0), row - mode_bytes}) {
        uint32_t off = uint32_t(8 * oct - base) * uint32_t(row) + uint32_t(col);
        for (int i = 0; i < 8; ++i, off += uint32_t(row)) {
          const int64_t f = 8 * oct + i - base;
          const bool inside = uint64_t(off) + uint64_t(mode_bytes) <= records;
          const bool good = f >= 0 && f < n ? inside && int64_t(off) == f * row + col : !inside;
          ++g_places;
          if (!good && ++g_wrong <= 10)
            std::printf("FAIL %s: targets [%lld, %lld), row %lld of %lld at offset %u of %u\n", what,
                        (long long)s.t0, (long long)s.t1, (long long)f, (long long)n, off, records);
        }
      }
  };
  range(0, s.split, s.obase, s.olen);
  if (s.split < s.pl) range(s.split, s.pl, s.tbase, s.t1 - s.t0);
}

void check_stack(const Layout& L, const std::vector<int32_t>& lags, int64_t frames) {
  char what[128];
  std::snprintf(what, sizeof what, "n %d %s %d bytes, %lld frames, %zu delays", L.n,
                L.full ? "full" : "ring", int(L.mode_bytes), (long long)frames, lags.size());
  const int64_t row = L.mode_stride * int64_t(L.mode_bytes);
  for (int span : {0, kMxSpan})
    for (const MxGroup& g : mx_groups(lags, span)) {
      int last = g.first + g.count;
      while (last > g.first && lags[size_t(last - 1)] >= frames) --last;
      if (last == g.first) continue;
      const int64_t ta = lags[size_t(g.first)], tb = lags[size_t(last - 1)];
      if (!span && mx_shape(ta, frames, ta, tb).pl > kMxPlane) continue;
      for (int64_t t = ta; t < frames;) {
        const int64_t e = mx_cut(t, frames, ta, tb);
        const MxShape s = mx_shape(t, e, ta, tb);
        if (mx_direct(s, frames, row)) {
          ++g_direct;
          check_launch(s, row, int64_t(L.mode_bytes), what);
        }
        t = e;
      }
    }
}

}  // namespace

int main() {
  for (int n : {512, 1024, 2048, 4096})
    for (int full : {0, 1})
      for (int spec : {NFS_SPEC_F32, NFS_SPEC_BF16}) {
        const int32_t one = 1;
        nfs_desc d{};
        d.n = n;
        d.n_bins = 1;
        d.lags = &one;
        d.n_lags = 1;
        d.spec_dtype = spec;
        d.full_spectra = full;
        d.capacity = 2;
        Layout L;
        std::string err;
        if (full && spec != NFS_SPEC_F32) continue;
        if (make_layout(&d, 0, &L, &err, true) != NFS_OK) {
          std::printf("FAIL layout: %s\n", err.c_str());
          return 1;
        }
        const int64_t fit = (int64_t(1) << 32) / (L.mode_stride * int64_t(L.mode_bytes));
        for (int64_t N = std::max<int64_t>(20, fit - 300); N <= fit + 20 && N <= 2600; N += 7)
          for (int64_t top : {int64_t(64), N / 2, N - 1}) {
            std::vector<int32_t> lags;
            for (int64_t t = 1; t <= std::min(top, N - 1); ++t) lags.push_back(int32_t(t));
            check_stack(L, lags, N);
          }
        // Far below 4 GiB the buffer loads are taken.
        std::vector<int32_t> lags;
        for (int t = 1; t < 20; ++t) lags.push_back(t);
        const long long before = g_direct;
        if (fit > 256) {
          check_stack(L, lags, std::min<int64_t>(fit / 4, 1000));
          if (g_direct == before) {
            std::printf("FAIL no buffer loads for n %d\n", n);
            ++g_wrong;
          }
        }
      }
  std::printf("%lld places of %lld launches, %lld failures\n", g_places, g_direct, g_wrong);
  return g_wrong ? 1 : 0;
}
