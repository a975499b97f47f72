"""D of a plan with full spectra is that of a plan with the ring modes only, bit for
bit, whichever kernel sums the pairs: launch shapes do not go by the number of modes
stored, 8 to 20 % more with full spectra."""
import pytest
import torch

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,N,lags", [
    (256, 100, [1, 2, 4, 8, 16, 32]),        # short windows
    (256, 255, [1, 2, 3, 5, 9, 17, 40, 90]),
    (256, 300, list(range(1, 31, 2))),
    (256, 313, list(range(1, 90, 2))),       # 45 delays: left to the history kernel
    (512, 75, [1, 3, 7, 30]),
    (512, 170, list(range(1, 42))),
    (128, 400, list(range(1, 201))),         # matrix cores
    (128, 64, [1, 2, 40]),                   # history kernel
    (256, 700, [1, 5, 25, 125, 600]),
])
def test_same_sums_as_ring_modes(n, N, lags):
    import paper_1209_3362_amd as nfs
    require_gpu()
    say(f"full spectra against ring modes: {N} frames {n}x{n}, {len(lags)} delays")
    g = torch.Generator(device="cuda")
    g.manual_seed(n + N)
    f = torch.rand((N, n, n), generator=g, device="cuda") * 900 + 50
    D = []
    for full in (False, True):
        plan = nfs.Plan(n, lags, n // 2, in_dtype="f32", capacity=N, full_spectra=full)
        D.append(plan.push(f).structure_function()[0].cpu())
        plan.close()
    assert torch.equal(D[0], D[1])
