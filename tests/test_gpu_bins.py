"""The rings' sums against a float64 average of the same plan's per-mode power
spectra, at the edges of the binning kernel: numbers of lags around its lane
splits (8, 16, 32, 64) and chunks (64), rings of one segment (256 modes) and of
several, and one ring of all modes."""
import numpy as np
import pytest
import torch

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_bins", [(16, 8), (16, 1), (128, 64), (256, 128), (64, 1), (256, 3)])
def test_ring_sums(n, n_bins):
    import paper_1209_3362_amd as nfs
    require_gpu()
    g = torch.Generator().manual_seed(n + n_bins)
    f = torch.randint(0, 4096, (72, n, n), generator=g).to(torch.float32)
    for n_lags in (1, 2, 8, 9, 16, 17, 32, 33, 64, 65, 75):
        say(f"bins n={n} rings={n_bins} lags={n_lags}")
        lags = list(range(n_lags))
        plan = nfs.Plan(n, lags, n_bins, in_dtype="f32", capacity=80)
        plan.push(f.cuda())
        D, C, P, st = (x.cpu().numpy() for x in plan.structure_function())
        S = plan.power_spectra().cpu().numpy().astype(np.float64)[:, :, :n // 2]
        ring = plan.bin_map().cpu().numpy()
        plan.close()
        weight = np.where(np.arange(n // 2) > 0, 2.0, 1.0)[None, :] * np.ones((n, 1))
        counts = np.array([weight[ring == b].sum() for b in range(n_bins)])
        assert np.array_equal(C, counts.astype(np.int64))
        assert np.array_equal(P, np.maximum(0, 72 - np.array(lags)))
        for b in range(n_bins):
            m = ring == b
            for i in range(n_lags):
                if not counts[b] or P[i] == 0:
                    assert np.isnan(D[i, b])
                    continue
                want = (S[i][m] * weight[m]).sum() / counts[b]
                # The spectra are the sums over the pairs rounded once more to
                # float32 (2^-24); every term is positive.
                assert abs(D[i, b] - want) <= 1.2e-7 * want, (i, b)
