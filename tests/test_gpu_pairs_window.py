"""The short-window pair kernel against the compensated sums of the history
kernel over the same spectra, mode by mode, at the edges of its shapes: windows
of 1 to 641 frames with and without a history, ring wraps, 1 to 50 lags
(consecutive, sparse, 0 and beyond the frames), every storage type."""
import numpy as np
import pytest
import torch

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

# (n, pushes, capacity, lags, spec); sums are taken after every push;
# smaller frames take the history kernel
CASES = [
    (256, [1], 8, [0, 1, 3], "f32"),
    (256, [2, 1, 5], 8, [1, 2], "f32"),
    (256, [15], 40, [0, 1, 2, 3, 7, 14, 15, 30], "f32"),
    (256, [33, 16, 17], 70, list(range(1, 14)), "bf16"),
    (256, [112], 112, list(range(1, 112, 4)), "f32"),
    (256, [113], 113, [1, 2, 4, 8, 112], "f16"),
    (256, [150], 150, list(range(1, 51)), "f32"),
    (256, [151, 40], 200, [1, 5, 25, 49], "f16"),
    (256, [100, 100, 100, 37], 180, [1, 2, 3, 4, 8, 13, 21, 34, 55, 80], "f32"),
    (256, [200, 64], 264, [3, 17, 50, 120], "bf16"),
    (256, [201], 201, list(range(1, 40)), "f32"),
    (256, [448], 448, list(range(10, 300, 8)), "f32"),
    (256, [640], 640, [1, 2, 3, 5, 9, 33, 65, 257, 600], "f32"),
    (256, [641], 641, [1, 2, 3, 5, 9, 33, 65, 257, 600], "f32"),
    (512, [9, 30], 39, [1, 4, 9, 16, 25], "f32"),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_window_sums(case):
    import paper_1209_3362_amd as nfs
    require_gpu()
    n, pushes, capacity, lags, spec = CASES[case]
    say(f"window sums n={n} pushes={pushes} capacity={capacity} lags={len(lags)} {spec}")
    g = torch.Generator().manual_seed(case)
    f = (torch.rand((sum(pushes), n, n), generator=g) * 900 + 50).cuda()
    got = []
    for accum in ("plain", "kahan"):
        plan = nfs.Plan(n, lags, n // 2, in_dtype="f32", capacity=capacity, spec=spec, accum=accum)
        t = 0
        for b in pushes:
            plan.push(f[t:t + b]).accumulate()
            t += b
        D, _, _, st = plan.structure_function()
        assert int(st.item()) == 0
        pairs = plan.work_counters()[1]
        assert pairs == sum(max(0, t - lag) for lag in lags)
        got.append((plan.power_spectra().cpu().numpy(), D.cpu().numpy()))
        plan.close()
    # Sums of the same FP32 terms, all >= 0: a lane adds at most 160 of them
    # one after the other (2^-24 each), a window and a few partial sums more.
    for a, b in zip(*got):
        assert np.array_equal(np.isnan(a), np.isnan(b))
        ok = ~np.isnan(b)
        assert np.all(np.abs(a[ok] - b[ok]) <= 1.2e-5 * np.abs(b[ok]))
