// Launch planning of the matrix-core pair kernel (see pair_matrix.hpp).
#include "pair_matrix.hpp"

#include <algorithm>

namespace nfs {
namespace {

// One 16-delay block of a delay list: delays [first, last) of it, and how
// many of its four column classes they touch.
struct Block {
  int64_t b;
  int first, last, classes;
};

std::vector<Block> blocks_of(const std::vector<int32_t>& lags, int first, int last) {
  std::vector<Block> out;
  for (int i = first; i < last;) {
    Block k{lags[size_t(i)] / 16, i, i, 0};
    int64_t quarter = -1;
    while (k.last < last && lags[size_t(k.last)] / 16 == k.b) {
      if (lags[size_t(k.last)] / 4 != quarter) {
        quarter = lags[size_t(k.last)] / 4;
        ++k.classes;
      }
      ++k.last;
    }
    out.push_back(k);
    i = k.last;
  }
  return out;
}

// Blocks from i on that one row set of four consecutive blocks sums whole:
// those within 64 delays, when together they touch at least kMxDense of its
// 16 (block, class) quarters; else 0. A whole row set costs one row read and
// up to four products per step, a scattered one of four quarters of a class
// one read and one product.
constexpr int kMxDense = 6;
// Blocks of a group: scattered they make a task each four.
constexpr int kMxBlocks = std::min(kMxRows - 8, 4 * (kMxTasks - 2));
size_t dense_run(const std::vector<Block>& v, size_t i) {
  size_t e = i;
  int q = 0;
  while (e < v.size() && v[e].b < v[i].b + 4) q += v[e++].classes;
  return q >= kMxDense ? e - i : 0;
}

}  // namespace

std::vector<MxGroup> mx_groups(const std::vector<int32_t>& lags, int span) {
  std::vector<MxGroup> out;
  const int L = int(lags.size());
  int i = 0;
  while (i < L) {
    MxGroup g;
    g.first = i;
    // At most one row set and a quarter of a task per block (a whole row set
    // takes two blocks or more), and the rounding up of the last.
    int blocks = 0;
    for (const Block& b : blocks_of(lags, i, L)) {
      if (g.count > 0 &&
          (blocks + 1 > kMxBlocks || g.count + (b.last - b.first) > kMxLags ||
           lags[size_t(b.last - 1)] - lags[size_t(g.first)] > (span ? span : kMxMaxSpan)))
        break;
      g.count += b.last - b.first;
      ++blocks;
    }
    out.push_back(g);
    i += g.count;
  }
  return out;
}

MxShape mx_shape(int64_t t0, int64_t t1, int64_t ta, int64_t tb) {
  MxShape s;
  s.t0 = t0;
  s.t1 = t1;
  const int tn = int(t1 - t0);
  s.olo = t0 - tb > 0 ? t0 - tb : 0;
  // Targets are read in 16-frame steps of four quarters from 16 places before
  // the first (for the shifts), and two steps ahead.
  const int reach = 64 * ((tn + 16 + 63) / 64) + 32;
  // 64 mod 128: rows of four neighbouring blocks and four digit planes lie on
  // distinct banks.
  auto plane = [](int64_t bytes) { return int((bytes - 64 + 127) / 128 * 128 + 64); };
  const int64_t before = t0 - s.olo;
  // One range [olo, t1).
  const int ob = 32 + int((16 - before % 16) % 16);
  const int64_t joined = int64_t(ob) + before - 16 + reach;
  // Two ranges, [olo, t1 - ta) and [t0, t1).
  const int64_t older = t1 - ta - s.olo > 0 ? t1 - ta - s.olo : 0;
  const int64_t tb2 = (ob + older + 15) / 16 * 16 + 16;
  const int64_t apart = tb2 - 16 + reach;
  s.obase = ob;
  if (joined <= apart) {
    s.olen = int(t1 - s.olo);
    s.tbase = int(ob + before);
    s.pl = plane(joined);
    s.split = s.pl;
    s.aoff = 0;
  } else {
    s.olen = int(older);
    s.tbase = int(tb2);
    s.pl = plane(apart);
    s.split = s.tbase - 16;
    s.aoff = int(before + ob - tb2);
  }
  s.amin = (s.obase - 16) / 16 * 16;  // 16 or more
  return s;
}

int64_t mx_cut(int64_t t0, int64_t t1, int64_t ta, int64_t tb) {
  for (int64_t parts = 1;; ++parts) {
    const int64_t n = (t1 - t0 + parts - 1) / parts;
    // The first cut may hold fewer older frames than the next ones.
    const int64_t far = t1 - n > t0 ? t1 - n : t0;
    if (n <= 16 || (mx_shape(t0, t0 + n, ta, tb).pl <= kMxPlane &&
                    mx_shape(far, far + n, ta, tb).pl <= kMxPlane))
      return t0 + n < t1 ? t0 + n : t1;
  }
}

void mx_workgroup(MxShape* s, int64_t modes) {
  auto lds = [&](int km) {
    return size_t(km) * (9 * size_t(s->pl) + kMxRounds * kMxWaves * 8 + kMxWaves * 4 +
                         kMxLags / 8) + 16;
  };
  int km = 16;
  // As many modes as two workgroups per CU leave LDS for, fewer while the
  // launch would not give every CU two workgroups.
  while (km > 4 && (lds(km) > kMxLds || modes / km < 512)) km /= 2;
  s->km = km;
  s->lds = lds(km);
}

bool mx_direct(const MxShape& s, int64_t capacity, int64_t row) {
  // Offsets go from -tbase rows (modulo 2^32) to fewer than pl rows, and a range
  // and its places before its first frame are within pl rows.
  return s.olo % capacity + s.olen <= capacity && s.t0 % capacity + (s.t1 - s.t0) <= capacity &&
         int64_t(s.pl) * row <= int64_t(1) << 32;
}

void mx_tables(const std::vector<int32_t>& lags, const MxGroup& g, int64_t t0, int64_t t1,
               MxTables* out) {
  MxTables& o = *out;
  o.n_tasks = o.n_rows = 0;
  int last = g.first + g.count;
  while (last > g.first && lags[size_t(last - 1)] >= t1) --last;
  o.n_paired = last - g.first;
  o.lag0 = lags[size_t(g.first)] / 16 * 16;
  const int64_t b0 = o.lag0 / 16;
  const std::vector<Block> blocks = blocks_of(lags, g.first, last);
  // Whole row sets, and the quarters of the other blocks by class.
  struct Set {
    int64_t b;
    int first, last;
  };
  std::vector<Set> whole, of_class[4];
  for (size_t i = 0; i < blocks.size();) {
    const size_t n = dense_run(blocks, i);
    if (n) {
      whole.push_back({blocks[i].b, blocks[i].first, blocks[i + n - 1].last});
      i += n;
      continue;
    }
    for (int l = blocks[i].first; l < blocks[i].last; ++l) {
      std::vector<Set>& v = of_class[lags[size_t(l)] / 4 % 4];
      if (v.empty() || v.back().b != blocks[i].b) v.push_back({blocks[i].b, l, l});
      v.back().last = l + 1;
    }
    ++i;
  }
  size_t scattered = 0;  // groups of four scattered rows per class
  for (const auto& v : of_class) scattered = std::max(scattered, (v.size() + 3) / 4);
  // Tasks: near-equal shares of the whole sets, with a scattered group each
  // while there are any (they share the columns).
  const int tasks = std::max(int((whole.size() + kMxSets - 1) / kMxSets), int(scattered));
  int ordered = 0, chunks = 0, runs = 0;
  for (int k = 0; k < tasks; ++k) {
    const size_t a = whole.size() * size_t(k) / size_t(tasks);
    const size_t z = whole.size() * size_t(k + 1) / size_t(tasks);
    MxTask& t = o.task[o.n_tasks++];
    t.sets = int16_t(z - a);
    t.scattered = size_t(k) < scattered;
    t.rows0 = int16_t(o.n_rows);
    t.first = int16_t(ordered);
    t.chunk0 = int16_t(chunks);
    t.run0 = int16_t(runs);
    int64_t lag = t1;
    auto put = [&](int l, int set, int row) {
      const int n = ordered - t.first;
      if (n % 64 == 0) o.chunk[chunks++] = 0;
      o.chunk[chunks - 1] |= 1u << set;
      o.order[ordered++] = mx_order(l - g.first, set, row, lags[size_t(l)] - o.lag0);
      lag = std::min(lag, int64_t(lags[size_t(l)]));
    };
    for (size_t i = a; i < z; ++i) {
      uint16_t* rows = o.block[o.n_rows++];
      for (int r = 0; r < 4; ++r) rows[r] = uint16_t(whole[i].b - b0 + r);
      const int64_t l0 = 16 * whole[i].b, n = whole[i].last - whole[i].first;
      const int64_t first = lags[size_t(whole[i].first)], last = lags[size_t(whole[i].last - 1)];
      lag = std::min(lag, first);
      o.run[runs] = 0;
      if (n >= kMxMinRun && last - first == n - 1 && (first >= t0 || last <= t0))
        o.run[runs] = mx_run(whole[i].first - g.first, first - l0, last - l0);
      else
        for (int l = whole[i].first; l < whole[i].last; ++l)
          put(l, int(i - a), int(lags[size_t(l)] / 16 - whole[i].b));
      ++runs;
    }
    if (t.scattered)
      for (const std::vector<Set>& v : of_class) {
        uint16_t* rows = o.block[o.n_rows++];
        for (size_t r = 0; r < 4; ++r) {
          const size_t at = 4 * size_t(k) + r;
          // A row without a quarter repeats the last of its class.
          rows[r] = v.empty() ? 0 : uint16_t(v[std::min(at, v.size() - 1)].b - b0);
          if (at >= v.size()) continue;
          for (int l = v[at].first; l < v[at].last; ++l) put(l, t.sets, int(r));
        }
      }
    t.count = int16_t(ordered - t.first);
    // From the first target that has a partner on, in whole groups of four
    // 16-frame blocks from the end.
    const int64_t late = (t0 > lag ? t0 : lag) - t0;
    const int64_t n = (t1 - t0 + 16 + 15) / 16;
    const int64_t s = n - (n - (late + 1) / 16 + 3) / 4 * 4;
    t.start = int16_t(s > 0 ? s : 0);
  }
}

// Cost in microseconds per 104,000 modes (512 x 512 frames), fitted to both
// kernels over 24 to 2600 frames and 4 to 1000 delays. A matrix launch takes
// about 200 plus 0.4 per frame it reads (load, digits, prefix sums) and 50 +
// 0.075 per target for every set of 64 delays or scattered group (products
// and energies); the explicit kernel 1.8 + 0.0095 per pair for each delay
// (2.2 + 0.0133 from 57 delays a group on, whose waves hold eight), and per
// frame 0.1, or 0.4 / 0.55 where its history leaves one workgroup per CU
// with 16 / 8 modes; its long-delay kernel reads a pair in 0.17. At 1000
// frames, matrix against explicit: delays 1..400 1.55 against 5.73 ms, 1..96
// 0.73 against 1.38, 1..56 0.61 against 0.64, 50 log-spaced ones up to 500
// 0.83 against 0.67; at 128 frames delays 1..64 0.36 against 0.26. The short-window
// kernel, other frame sizes, storage types and Kahan sums are not in the fit:
// over 258 stacks of 16 x 16 to 512 x 512 frames (130 to 1500 of them, 48 delays
// to all, every storage type) a whole pass took at most 0.98 of what it took
// before there was this kernel and the short-window one.
bool mx_wins(const std::vector<int32_t>& lags, const std::vector<LagGroup>& groups,
             const std::vector<MxGroup>& mx, int64_t t0, int64_t t1) {
  double plain = 0.0;
  for (const LagGroup& g : groups) {
    int count = 0;
    double pairs = 0.0;
    for (int l = g.first; l < g.first + g.count; ++l) {
      const int64_t from = std::max<int64_t>(t0, lags[size_t(l)]);
      if (from >= t1) continue;
      ++count;
      pairs += double(t1 - from);
    }
    if (g.modes == 0) {
      plain += 0.17 * pairs;
      continue;
    }
    const double frames = double(t1 - std::max<int64_t>(0, t0 - g.max_lag));
    plain += count < 57 ? 1.8 * count + 0.0095 * pairs : 2.2 * count + 0.0133 * pairs;
    plain += frames * (g.modes == 8 ? 0.55 : 2 * g.lds > size_t(kLdsBytes) ? 0.4 : 0.1);
  }
  double matrix = 0.0;
  for (const MxGroup& g : mx) {
    int last = g.first + g.count;
    while (last > g.first && lags[size_t(last - 1)] >= t1) --last;
    if (last == g.first) continue;
    const int64_t ta = lags[size_t(g.first)], tb = lags[size_t(last - 1)];
    const std::vector<Block> blocks = blocks_of(lags, g.first, last);
    int whole = 0, classes = 0;
    for (size_t i = 0; i < blocks.size();) {
      const size_t n = dense_run(blocks, i);
      whole += n > 0;
      if (!n) classes += blocks[i].classes;
      i += std::max<size_t>(n, 1);
    }
    const int sets = whole + (classes + 15) / 16;
    for (int64_t t = std::max(t0, ta); t < t1;) {
      const int64_t e = mx_cut(t, t1, ta, tb);
      const MxShape s = mx_shape(t, e, ta, tb);
      const double frames = s.split == s.pl ? double(s.olen) : double(s.olen) + double(e - t);
      matrix += 200.0 + 0.4 * frames + sets * (50.0 + 0.075 * double(e - t));
      t = e;
    }
  }
  return 1.08 * matrix < plain;  // the fits are within a few percent
}

}  // namespace nfs
