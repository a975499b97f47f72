"""Matrix-core pair sums at the ends of their ranges, against the explicit kernel
(few delays at a time): rings that nearly fill 4 GiB, where the kernel's 32-bit
row offsets end, and the largest sums of the longest launch."""
import math

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


def test_longest_launch_alternating_at_full_scale():
    """A mode that alternates between +A and -A, both components just below a power of two,
    over the 2160 targets of one launch: every odd delay's pairs are as large as they can be."""
    import paper_1209_3362_amd as nfs
    require_gpu()
    say("matrix pairs: 2161 frames alternating")
    n, N = 32, 2161
    k = 2 * math.pi / n * torch.arange(n)
    wave = torch.cos(3 * k[None, :] + 2 * k[:, None] + math.pi / 4)
    # The coefficient of a wave of amplitude a is a n^2 / 2 at pi / 4.
    a = 128 * (1 - 2 ** -9) * math.sqrt(2) * 2 / n ** 2
    f = 1000 * (1 + a * wave * (1 - 2.0 * (torch.arange(N) % 2))[:, None, None])
    f[0] = 1000  # subtracted from every frame
    out = []
    lags = list(range(1, 200))
    for part in (lags, [1, 3, 101, 199]):
        plan = nfs.Plan(n, part, n // 2, in_dtype="f32", capacity=N)
        out.append(plan.push(f.cuda()).structure_function()[0].cpu())
        plan.close()
    D, E = out[0][[0, 2, 100, 198]], out[1]
    # The explicit sums add 540 equal FP32 terms in a row.
    assert torch.all((D - E).abs()[:, 3] <= 540 * 2.0 ** -24 * E[:, 3])
