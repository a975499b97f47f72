"""Matrix-core pair sums of modes whose values differ much in size: the sums that
the largest value does not enter are as exact per mode as the explicit kernels'
(the same ring, few delays at a time)."""
import pytest
import torch

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

# The explicit kernels add FP32 terms in chains of up to a quarter of the targets
# (at most 60 pairs here, two fused terms each): (2 + 30 + 3) * 2^-24. A matrix sum is
# within 2.9 sqrt(120) * 2^-24, or 5 * 2^-24 where it is formed from the coefficients.
RTOL = 4e-6


def spectra(f, lags, n, spec, accum, full, capacity, chunk):
    import paper_1209_3362_amd as nfs
    plan = nfs.Plan(n, lags, n // 2, in_dtype="f32", capacity=capacity, spec=spec, accum=accum,
                    full_spectra=full)
    for t in range(0, f.shape[0], chunk):
        plan.push(f[t:t + chunk])
    S = plan.power_spectra().cpu()
    plan.close()
    return S


def compare(f, lags, parts, n, spec="f32", accum="plain", full=True, capacity=0, chunk=0):
    """parts: slices of lags summed by themselves."""
    capacity, chunk = capacity or f.shape[0], chunk or f.shape[0]
    S = spectra(f, lags, n, spec, accum, full, capacity, chunk)
    for part in parts:
        E = spectra(f, lags[part], n, spec, accum, full, capacity, chunk)
        M = S[part]
        assert torch.equal(torch.isnan(M), torch.isnan(E))
        bad = (M - E).abs() > RTOL * E.abs()
        assert not bad.any(), (lags[part], ((M - E).abs() / E.abs())[bad].max())


@pytest.mark.parametrize("n,full", [(32, True), (64, True), (128, False), (128, True),
                                    (256, False)])  # 4, 4, 8, 16 and 16 modes per workgroup
@pytest.mark.parametrize("spec,accum", [("f32", "plain"), ("f32", "kahan"), ("bf16", "plain"),
                                        ("f16", "kahan")])
@pytest.mark.parametrize("dark", [30, 1000, 10000])
def test_one_dark_frame(n, full, spec, accum, dark):
    """Frame 120 of 240 is nearly dark: normalised by its mean, its fluctuations are `dark`
    times the others'. Delays above 120 have no pair of it."""
    require_gpu()
    say(f"matrix pairs: a frame {dark} times darker, n={n} full={full} {spec} {accum}")
    N = 240
    g = torch.Generator().manual_seed(n + dark)
    f = torch.randn((N, n, n), generator=g)
    f -= f.mean(dim=(1, 2), keepdim=True)
    f = 1000 + 100 * f
    f[120] = f[120] - 1000 + 1000 / dark
    lags = list(range(1, 236))
    compare(f.cuda(), lags, [slice(0, 3), slice(118, 124), slice(150, 158), slice(228, 235)], n,
            spec, accum, full)


def test_slow_modes_and_last_delays():
    """A first frame unlike all others, which hardly change, in a ring whose later windows no
    longer hold it; and the delays with one, two and three pairs of a long stack."""
    require_gpu()
    say("matrix pairs: slow modes, few pairs")
    n = 32
    g = torch.Generator().manual_seed(5)
    f = 1000 + 300 * torch.rand((700, n, n), generator=g)
    f[2:] = f[1] + 0.05 * (f[2:] - 1150)
    lags = list(range(1, 200))
    for accum in ("plain", "kahan"):
        compare(f.cuda(), lags, [slice(0, 3), slice(60, 64), slice(196, 199)], n, accum=accum,
                capacity=450, chunk=90)
    f = 1000 + 300 * torch.rand((1000, n, n), generator=g)
    lags = list(range(500, 1000))
    compare(f.cuda(), lags, [slice(495, 500)], n)


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 1e30])
def test_values_beyond_the_integers(value):
    """A pixel so large that squares overflow, or not finite: the same sums as the explicit
    kernels' for every delay, finite or not."""
    require_gpu()
    say(f"matrix pairs: a pixel {value}")
    n, N = 32, 240
    f = 1000 + 300 * torch.rand((N, n, n), generator=torch.Generator().manual_seed(6))
    f[120, 3, 5] = value
    f[120, 9, 9] -= 0 if value != 1e30 else 1e30
    lags = list(range(1, 236))
    S = spectra(f.cuda(), lags, n, "f32", "plain", True, N, N)
    for part in (slice(0, 3), slice(118, 124), slice(228, 235)):
        E = spectra(f.cuda(), lags[part], n, "f32", "plain", True, N, N)
        M = S[part]
        assert torch.equal(torch.isfinite(M), torch.isfinite(E))
        ok = torch.isfinite(E)
        assert torch.all((M - E).abs()[ok] <= RTOL * E.abs()[ok])
