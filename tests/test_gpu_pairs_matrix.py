"""The matrix-core pair kernel (csrc/pairs_mx.hip), which windows with many
delays run: D against the FP64 oracle at the edges of its tables and planes,
exact zeros, values that are not finite, and the same sums from cut windows."""
import numpy as np
import pytest
import torch

import gen
import oracle
from gpu_util import assert_D_close, require_gpu, run_plan, say

pytestmark = pytest.mark.gpu

# FP32 transforms of fluctuation-sized values: about 1e-7 of a mode's largest
# coefficient per value; sums are exact, so the slowest modes' shortest
# differences, some 30 times smaller, are within 1e-5.
RTOL = 1e-5


@pytest.mark.parametrize("n,N,lags,kw", [
    (32, 200, list(range(0, 100)), {}),                        # lag 0, consecutive runs
    (64, 1000, list(range(1, 401)), {}),                       # 8 modes per workgroup
    (32, 2047, list(range(1, 2047)), {}),                      # several launches
    (16, 2600, list(range(1, 400)), {}),                       # a window cut in two
    (16, 3100, list(range(1, 300)) + list(range(2401, 2700, 2)), {}),  # far delays
    (32, 301, [t for t in range(1, 290) if t % 3], {}),        # no consecutive run
    (32, 400, list(range(5, 130)) + [200, 300, 399, 400, 500], {}),    # delays without pairs
    (32, 700, list(range(1, 200)), dict(capacity=450)),        # windows of a shorter ring
    (32, 700, list(range(1, 200)), dict(capacity=450, accum="kahan")),
    (64, 333, list(range(1, 129)), dict(chunk=50)),
    (64, 900, list(range(1, 257)), dict(in_dtype="u16")),
])
def test_dense_delays_match_oracle(n, N, lags, kw):
    kw = dict(kw)
    u16 = kw.pop("in_dtype", "f32") == "u16"
    cfg = gen.config("c2" if u16 else "c1", n=n, N=N, n_bins=n // 2)
    say(f"matrix pairs: {N} frames {n}x{n}, {len(lags)} delays up to {lags[-1]}, {kw}")
    f = gen.make_stack(cfg, 21)
    ref = oracle.structure_function(f.numpy().astype(np.float64), lags, n // 2)
    D, C, P, st = run_plan(f, lags, n // 2, "u16" if u16 else "f32", **kw)
    assert st == 0 and np.array_equal(P, ref["pairs"]) and np.array_equal(C, ref["counts"])
    print("worst", assert_D_close(D, ref["D"], rtol=RTOL))


@pytest.mark.parametrize("spec", ["bf16", "f16"])
def test_sixteen_bit_spectra(spec):
    """The same D as the explicit kernel sums from the same ring (few delays
    at a time), within the FP32 sums of that one."""
    n, N = 64, 700
    cfg = gen.config("c2", n=n, N=N, n_bins=n // 2)
    say(f"matrix pairs on {spec} spectra: {N} frames {n}x{n}")
    f = gen.make_stack(cfg, 22)
    lags = list(range(1, 257))
    D, _, _, st = run_plan(f, lags, n // 2, "u16", spec=spec)
    assert st == 0
    for part in (lags[:8], lags[124:132], lags[248:]):
        E = run_plan(f, part, n // 2, "u16", spec=spec, capacity=N)[0]
        assert_D_close(D[part[0] - 1:part[-1]], E, rtol=2e-6)


def test_equal_frames_give_exact_zero():
    """A stack that alternates between two frames: even delays are exactly 0
    and odd ones all equal."""
    n, N = 32, 301
    cfg = gen.config("c1", n=n, N=2, n_bins=n // 2)
    say("matrix pairs: two frames alternating")
    two = gen.make_stack(cfg, 23)
    f = two[torch.arange(N) % 2]
    lags = list(range(1, 200))
    D = run_plan(f, lags, n // 2, "f32")[0]
    assert np.all(D[1::2] == 0.0)
    assert np.all(D[0::2, 1:] > 0.0)
    assert_D_close(D[0::2], np.repeat(D[:1], 100, axis=0), rtol=1e-6)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("k", [0, 120])
def test_values_that_are_not_finite(bad, k):
    """A pixel that is not finite spoils exactly the delays with a pair of its
    frame; the others are those of the stack without it."""
    n, N = 32, 240
    cfg = gen.config("c1", n=n, N=N, n_bins=n // 2)
    say(f"matrix pairs: a pixel {bad} in frame {k}")
    f = gen.make_stack(cfg, 24)
    lags = list(range(1, 236))
    clean = run_plan(f, lags, n // 2, "f32")[0]
    g = f.clone()
    g[k, 3, 5] = bad
    D, _, _, st = run_plan(g, lags, n // 2, "f32")
    assert st != 0
    for i, t in enumerate(lags):
        # Frame 0 is subtracted from every frame.
        spoilt = k == 0 or k - t >= 0 or k + t < N
        if spoilt:
            assert not np.isfinite(D[i, 1:]).any(), t
        else:
            assert_D_close(D[i:i + 1], clean[i:i + 1], rtol=1e-6)


def test_work_counter_and_power_spectra():
    import paper_1209_3362_amd as nfs
    require_gpu()
    n, N, lags = 32, 260, list(range(1, 150)) + [259, 260, 300]
    cfg = gen.config("c1", n=n, N=N, n_bins=n // 2)
    say("matrix pairs: counter and 2D spectra")
    f = gen.make_stack(cfg, 25)
    ref = oracle.structure_function(f.numpy(), lags, n // 2, return_power=True)
    plan = nfs.Plan(n, lags, n // 2, in_dtype="f32", capacity=N + 60, full_spectra=True)
    plan.push(f.cuda())
    S = plan.power_spectra().cpu().numpy()
    assert plan.work_counters() == (N, sum(max(0, N - t) for t in lags))
    plan.close()
    ok = [i for i, t in enumerate(lags) if t < N]
    o = ref["P"][ok][:, :, : n // 2 + 1]
    assert np.all(np.abs(S[ok] - o) <= 1e-4 * np.abs(o) + 1e-6 * np.abs(o).max(axis=(1, 2), keepdims=True))
    assert np.all(np.isnan(S[len(ok):]))
