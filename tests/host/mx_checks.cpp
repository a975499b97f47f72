// Host model of the matrix-core pair kernel's index arithmetic: for many
// windows and delay lists it places random integer series in byte planes as
// the kernel does, walks every task's lanes and steps with the kernel's
// addresses (each read checked against the plane), and compares the sums of
// squared differences with the plain definition, exactly.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "pair_matrix.hpp"

using namespace nfs;

static int g_fail = 0, g_checks = 0;
#define CHECK(c, ...)                             \
  do {                                            \
    ++g_checks;                                   \
    if (!(c)) {                                   \
      std::printf("FAIL %s:%d: ", #c, __LINE__);  \
      std::printf(__VA_ARGS__);                   \
      std::printf("\n");                          \
      if (++g_fail > 20) std::exit(1);            \
    }                                             \
  } while (0)

namespace {

struct Model {
  std::vector<int64_t> q;  // frame -> value (one component; up to 2^25)
  std::vector<int8_t> plane[4];
  std::vector<uint64_t> prefix;
  MxShape s;

  void place() {
    for (auto& p : plane) p.assign(size_t(s.pl), 0);
    prefix.assign(size_t(s.pl) + 1, 0);
    for (int x = 0; x < s.pl; ++x) {
      const bool old = x < s.split;
      const int f = x - (old ? s.obase : s.tbase);
      const int n = old ? s.olen : int(s.t1 - s.t0);
      int64_t v = 0;
      if (f >= 0 && f < n) v = q[size_t((old ? s.olo : s.t0) + f)];
      const uint32_t w = (uint32_t(int32_t(v)) + 0x808080u) ^ 0x808080u;
      int64_t back = 0;
      for (int d = 0; d < 4; ++d) {
        plane[d][size_t(x)] = int8_t(w >> (8 * d));
        back += int64_t(plane[d][size_t(x)]) * (int64_t(1) << (8 * d));
      }
      CHECK(back == v, "digits of %lld", (long long)v);
      prefix[size_t(x) + 1] = prefix[size_t(x)] + uint64_t(v * v);
    }
  }

  // 16 bytes of plane d from place x (4-byte boundary), bounds checked.
  const int8_t* read(int d, int x, int align) {
    CHECK(x >= 0 && x + 16 <= s.pl && x % align == 0, "read at %d of %d (align %d)", x, s.pl,
          align);
    if (x < 0 || x + 16 > s.pl) std::exit(1);
    return &plane[d][size_t(x)];
  }
};

int64_t sum_at(const std::vector<int64_t>& v, int i) { return v[size_t(i)]; }

void run_window(Model& M, const std::vector<int32_t>& lags, const MxGroup& g, int64_t t0,
                int64_t t1, int64_t modes) {
  int64_t tb = -1;
  for (int l = g.first; l < g.first + g.count; ++l)
    if (lags[size_t(l)] < t1) tb = lags[size_t(l)];
  if (tb < 0) return;
  const int64_t ta = lags[size_t(g.first)];
  M.s = mx_shape(t0, t1, ta, tb);
  mx_workgroup(&M.s, modes);
  const MxShape& s = M.s;
  CHECK(s.lds <= size_t(kMxLds), "lds %zu", s.lds);
  CHECK(s.pl % 128 == 64 && s.amin >= 16 && s.amin % 16 == 0 && s.amin + 16 <= s.obase, "shape");
  CHECK((s.pl / 8) * s.km <= kMxRounds * 64 * kMxWaves, "items %d", (s.pl / 8) * s.km);
  CHECK(s.tbase % 16 == 0 && s.aoff % 16 == 0 && s.split % 8 == 0, "bases");
  CHECK(s.tbase + (t1 - t0) <= s.pl, "targets inside");
  M.place();
  static MxTables T;
  mx_tables(lags, g, t0, t1, &T);
  CHECK(T.n_rows <= kMxRows && T.n_tasks <= kMxTasks, "tables %d %d", T.n_rows, T.n_tasks);
  std::vector<int64_t> got(size_t(g.count), -1);
  for (int t = 0; t < T.n_tasks; ++t) {
    const MxTask& task = T.task[t];
    const int sets = task.sets + (task.scattered ? 4 : 0);
    CHECK(task.sets <= kMxSets && task.rows0 + sets <= T.n_rows && sets > 0, "task");
    const int kst = s.tbase - 16 + 16 * task.start;
    const int steps = mx_steps(int(t1 - t0), task.start);
    CHECK(steps >= 1, "steps");
    std::vector<int64_t> sum_v(size_t(kMxTiles) * 16, 0);
    for (int quarter = 0; quarter < 4; ++quarter)
      for (int rr = 0; rr < 4; ++rr) {
        const int kb = kst + quarter * 16 * steps;
        for (int d = 0; d < 4; ++d) M.read(d, kb + 16 * (steps + 1), 16);  // read ahead
        for (int st = 0; st < steps; ++st) {
          // target values of the step and the next
          int64_t tv[32];
          for (int e = 0; e < 32; ++e) {
            tv[e] = 0;
            for (int d = 0; d < 4; ++d) {
              const int8_t* p = M.read(d, kb + 16 * (st + (e >= 16)), 16);
              tv[e] += int64_t(p[e % 16]) * (int64_t(1) << (8 * d));
            }
            if (task.start == 0 && quarter == 0 && st == 0 && e < 16) tv[e] = 0;
          }
          for (int i = 0; i < sets; ++i) {
            const int off = s.aoff - T.lag0 - 16 * int(T.block[task.rows0 + i][rr]);
            int at = kb + off + 16 * st;
            if (at < s.amin) at = s.amin;
            int64_t ov[16] = {0};
            for (int d = 0; d < 4; ++d) {
              const int8_t* p = M.read(d, at, 16);
              for (int e = 0; e < 16; ++e) ov[e] += int64_t(p[e]) * (int64_t(1) << (8 * d));
            }
            for (int c = 0; c < 4; ++c) {
              if (i >= task.sets && c != i - task.sets) continue;
              const int tile = i < task.sets ? 4 * i + c : 4 * task.sets + c;
              for (int j = 0; j < 4; ++j)
                for (int e = 0; e < 16; ++e)
                  sum_v[size_t(tile) * 16 + 4 * rr + j] += ov[e] * tv[e + 4 * c + j];
            }
            // the row read ahead of the last step
            at = kb + off + 16 * (st + 1);
            M.read(0, at < s.amin ? s.amin : at, 16);
          }
        }
      }
    auto P = [&](int64_t x) -> uint64_t {
      CHECK(x >= 0 && x < s.pl, "prefix at %lld", (long long)x);
      return M.prefix[size_t(x)];
    };
    CHECK(P(t1 - t0 + s.tbase) == P(s.pl - 8), "total");
    CHECK(s.tbase % 8 == 0, "energy at t0");
    const uint64_t total = P(s.pl - 8), at_t0 = t0 > 0 ? P(s.tbase) : 0;
    auto clamped = [&](int64_t x) { return x < 0 ? 0 : x > s.pl - 1 ? int64_t(s.pl) - 1 : x; };
    auto energy_at = [&](int64_t x) { return M.prefix[size_t(clamped(x)) + 1] - M.prefix[size_t(clamped(x))]; };
    // Runs of consecutive delays.
    uint64_t next_e = 0;
    int64_t next_lag = -1;
    for (int i = 0; i < task.sets; ++i) {
      const uint32_t run = T.run[task.run0 + i];
      CHECK(task.run0 + i < kMxRows / 2, "runs");
      if (!run) continue;
      const int64_t l0 = T.lag0 + 16 * T.block[task.rows0 + i][0];
      const int p0 = run >> 9 & 63, p1 = run >> 15 & 63;
      const bool late = l0 + p0 >= t0;
      const int64_t xe = t1 - s.olo + s.obase - l0;
      const int64_t xs = late ? l0 - t0 + s.tbase : t0 - s.olo + s.obase - l0;
      if (next_lag != l0)
        next_e = (late ? total : total - at_t0) + P(clamped(xe)) - P(clamped(xs));
      uint64_t sum = 0;
      for (int k = 0; k < 64; ++k) {
        const int64_t tau = l0 + k;
        if (k >= p0 && k <= p1) {
          const int l = int(run & 511) + k - p0;
          CHECK(l < g.count && lags[size_t(g.first + l)] == tau, "run");
          CHECK(got[size_t(l)] == -1, "delay %d twice", l);
          const int o = 16 * (4 * i + (k >> 2 & 3)) + 4 * (k >> 4) + (k & 3);
          got[size_t(l)] = int64_t(next_e - sum - 2 * uint64_t(sum_at(sum_v, o)));
        }
        uint64_t drop = energy_at(xe - 1 - k);
        drop += late ? energy_at(xs + k) : 0 - energy_at(xs - 1 - k);
        sum += drop;
      }
      next_e -= sum;
      next_lag = l0 + 64 <= t0 || late ? l0 + 64 : -1;
    }
    for (int k = 0; k < task.count; ++k) {
      const uint32_t code = T.order[task.first + k];
      const int l = code & 511, set = code >> 9 & 15, row = code >> 13 & 3;
      const int64_t tau = int64_t(code >> 15) + T.lag0;
      CHECK(l < g.count && tau == lags[size_t(g.first + l)], "order");
      const int c = int(tau / 4 % 4), i = 4 * set + c, o = 4 * row + int(tau % 4);
      CHECK(set <= task.sets && (T.chunk[task.chunk0 + k / 64] >> set & 1), "chunk");
      CHECK(task.chunk0 + k / 64 < kMxChunks, "chunks");
      const int rs = task.rows0 + (set < task.sets ? set : set + c);
      CHECK(tau == T.lag0 + 16 * T.block[rs][row] + 4 * c + tau % 4, "delay of tile %d", i);
      const bool late = tau > t0;
      const uint64_t e = (late ? total : total - at_t0) + P(t1 - tau - s.olo + s.obase) -
                         P(late ? tau - t0 + s.tbase : t0 - tau - s.olo + s.obase);
      CHECK(got[size_t(l)] == -1, "delay %d twice", l);
      got[size_t(l)] = int64_t(e - 2 * uint64_t(sum_at(sum_v, 16 * i + o)));
    }
  }
  for (int l = 0; l < g.count; ++l) {
    const int64_t tau = lags[size_t(g.first + l)];
    if (tau >= t1) {
      CHECK(got[size_t(l)] == -1, "delay without pairs");
      continue;
    }
    int64_t want = 0;
    for (int64_t t = t0 > tau ? t0 : tau; t < t1; ++t) {
      const int64_t d = M.q[size_t(t)] - M.q[size_t(t - tau)];
      want += d * d;
    }
    CHECK(got[size_t(l)] == want, "window [%lld, %lld) tau %lld", (long long)t0, (long long)t1,
          (long long)tau);
  }
}

// Targets [T0, T1) of a ring that keeps what the delays need.
void run(std::mt19937_64& rng, const std::vector<int32_t>& lags, int64_t T0, int64_t T1) {
  Model M;
  M.q.resize(size_t(T1));
  for (auto& v : M.q) v = int64_t(rng() % ((1u << 26) + 1)) - (1 << 25);
  std::vector<MxGroup> groups = mx_groups(lags, 0);
  bool whole = true;
  for (int pass = 0; pass < 2; ++pass) {
    int next = 0;
    for (const MxGroup& g : groups) {
      CHECK(g.first == next && g.count >= 1 && g.count <= kMxLags, "groups in order");
      next = g.first + g.count;
      int64_t tb = -1;
      for (int l = g.first; l < next; ++l)
        if (lags[size_t(l)] < T1) tb = lags[size_t(l)];
      if (tb < 0) continue;
      const int64_t ta = lags[size_t(g.first)], t0 = T0 > ta ? T0 : ta;
      if (pass == 0) {
        whole &= mx_shape(t0, T1, ta, tb).pl <= kMxPlane;
        continue;
      }
      for (int64_t t = t0; t < T1;) {
        const int64_t e = mx_cut(t, T1, ta, tb);
        run_window(M, lags, g, t, e, 100000);
        t = e;
      }
    }
    CHECK(next == int(lags.size()), "all delays");
    if (pass == 0 && !whole) groups = mx_groups(lags, kMxSpan);
  }
}

std::vector<int32_t> random_lags(std::mt19937_64& rng, int top, int count) {
  std::vector<char> take(size_t(top) + 1, 0);
  for (int i = 0; i < count; ++i) {
    const double u = double(rng() % 100000) / 100000;
    const int64_t v = rng() % 2 ? int64_t(rng() % (uint64_t(top) + 1)) : int64_t(u * u * u * top);
    take[size_t(v)] = 1;
    if (rng() % 4 == 0)
      for (int64_t k = v; k <= top && k < v + int64_t(rng() % 40); ++k) take[size_t(k)] = 1;
  }
  std::vector<int32_t> out;
  for (int v = 0; v <= top; ++v)
    if (take[size_t(v)]) out.push_back(v);
  return out;
}

}  // namespace

int main() {
  std::mt19937_64 rng(7);
  auto all = [](int a, int b) {
    std::vector<int32_t> v;
    for (int i = a; i <= b; ++i) v.push_back(i);
    return v;
  };
  run(rng, {0}, 0, 1);
  run(rng, {1}, 0, 2);
  run(rng, {0, 1, 5, 9, 12}, 0, 9);
  run(rng, all(1, 31), 0, 32);
  run(rng, {1, 2, 4, 8, 16}, 0, 64);
  run(rng, all(0, 400), 0, 900);
  run(rng, all(1, 700), 500, 760);
  run(rng, all(1, 2047), 0, 2048);
  run(rng, all(1, 600), 900, 3000);
  run(rng, {1, 5, 700, 2401, 3000, 3999, 4000}, 0, 4000);
  run(rng, {1, 5, 700, 2401, 3000}, 3000, 3100);
  for (int it = 0; it < 400; ++it) {
    const int top = 1 + int(rng() % (it % 10 == 0 ? 3000 : 300));
    const std::vector<int32_t> lags = random_lags(rng, top, 1 + int(rng() % 30));
    const int64_t T0 = rng() % 3 ? int64_t(rng() % 700) : 0;
    run(rng, lags, T0, T0 + 1 + int64_t(rng() % 260));
  }
  std::printf("%d checks, %d failures\n", g_checks, g_fail);
  return g_fail ? 1 : 0;
}
