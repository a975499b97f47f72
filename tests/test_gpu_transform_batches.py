"""Transform batches of plans whose largest delay nearly fills the ring: they
borrow idle memory (the sums, the ring behind the batch) instead of
transforming frame by frame, and store the same spectra bit for bit."""
import numpy as np
import pytest

import gen
from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,N,lags,kw", [
    (32, 32, list(range(1, 32)), {}),                              # sums and ring
    (128, 90, [1, 89], {}),                                        # few sums: the ring
    (64, 150, list(range(0, 150)), dict(spec="f16")),              # row sums of |u| too
    (64, 70, [1, 5, 69], dict(full_spectra=True, spec="bf16")),    # k_x = n/2 values too
    (64, 200, [1, 2, 120], dict(capacity=130)),                    # the ring wraps
])
@pytest.mark.parametrize("chunk", [None, 29])
def test_spectra_do_not_depend_on_the_batches(n, N, lags, kw, chunk):
    import paper_1209_3362_amd as nfs
    require_gpu()
    kw = dict(kw)
    cap = kw.pop("capacity", N)
    cfg = gen.config("c2", n=n, N=N, n_bins=n // 2)
    say(f"batches: {N} frames {n}x{n}, delays up to {lags[-1]}, ring {cap}, {kw}, chunk {chunk}")
    f = gen.make_stack(cfg, 31).cuda()
    out = []
    # The second ring has room for whole batches beyond the largest delay.
    for c in (cap, N + lags[-1] + 64):
        plan = nfs.Plan(n, lags, n // 2, in_dtype="u16", capacity=c, **kw)
        for rep in range(2):  # after a reset the sums are idle again
            plan.reset()
            for i in range(0, N, chunk or N):
                plan.push(f[i:i + (chunk or N)])
        spec = [plan.spectrum(t).cpu().numpy() for t in range(N - cap, N)]
        D = plan.structure_function()[0].cpu().numpy()
        out.append((spec, D))
        plan.close()
    for a, b in zip(out[0][0], out[1][0]):
        assert np.array_equal(a, b)
    if cap == N:
        assert np.array_equal(out[0][1], out[1][1], equal_nan=True)
    else:
        ok = out[1][1] != 0
        assert np.all(np.abs(out[0][1] / np.where(ok, out[1][1], 1) - 1)[ok] < 1e-6)
