"""Matrix-core pair sums of rings that nearly fill 4 GiB, where the kernel's
32-bit row offsets end, against the explicit kernel (few delays at a time)."""
import pytest
import torch

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,N,top,full", [
    (1024, 900, 100, True),    # 32-bit offsets would end 1021 rows on, its places 1032
    (2048, 250, 249, False),
    (1024, 1200, 400, False),
    (2048, 170, 169, True),
])
def test_rings_near_four_gigabytes(n, N, top, full):
    import paper_1209_3362_amd as nfs
    require_gpu()
    say(f"matrix pairs: {N} frames {n}x{n}, delays 1..{top}, full {full}")
    g = torch.Generator(device="cuda")
    g.manual_seed(n + N)
    f = torch.empty((N, n, n), dtype=torch.uint16, device="cuda")
    for t in range(0, N, 50):
        b = f[t:t + 50]
        b.copy_(torch.randint(1000, 3000, b.shape, generator=g, device="cuda").to(torch.uint16))
    out = []
    few = sorted({1, 2, top // 2, top - 1, top})
    for lags in (list(range(1, top + 1)), few):
        plan = nfs.Plan(n, lags, n // 2, in_dtype="u16", capacity=N, full_spectra=full)
        out.append(plan.push(f).structure_function()[0].cpu())
        plan.close()
    D, E = out[0][[t - 1 for t in few]], out[1]
    # Sums of FP32 terms in both, averaged over a ring's modes.
    assert torch.all((D - E).abs()[:, 1:] <= 2e-6 * E[:, 1:])
