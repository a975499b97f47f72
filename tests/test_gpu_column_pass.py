"""Differences of stored spectra against float64 transforms at the frame sizes of the
three-level column pass (2048 and 4096) and around the frames that one workgroup
of a pass takes in turn, with ring wraps, every storage type and full spectra."""
import pytest
import torch

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,frames,capacity,spec,full", [
    (2048, 2, 4, "f32", False), (2048, 11, 6, "f32", False), (2048, 5, 8, "f32", True),
    (2048, 4, 4, "bf16", False), (2048, 4, 4, "f16", True), (4096, 3, 3, "f32", False),
    (4096, 2, 2, "f16", False), (512, 65, 65, "f32", False), (128, 130, 130, "f32", False)])
def test_spectra(n, frames, capacity, spec, full):
    import paper_1209_3362_amd as nfs
    require_gpu()
    say(f"column pass n={n} frames={frames} capacity={capacity} {spec} full={full}")
    g = torch.Generator().manual_seed(n + frames)
    f = (torch.rand((frames, n, n), generator=g) * 3000 + 100).cuda()
    plan = nfs.Plan(n, [1], n // 2, in_dtype="f32", capacity=capacity, spec=spec,
                    full_spectra=full)
    plan.push(f)
    first = max(0, frames - capacity)
    stored = torch.ones((n, n // 2), dtype=torch.bool) if full else plan.bin_map().cpu() >= 0

    def both(t):
        u = f[t].double()
        return plan.spectrum(t).cpu(), torch.fft.rfft2(u / u.mean())[:, :n // 2].cpu()

    got0, want0 = both(first)
    for t in sorted({frames - 1, (first + frames) // 2} - {first}):
        got, want = both(t)
        for s in (got0, got):
            assert s[0, 0] == n * n
            assert torch.all(s[~stored] == 0)
        # FP32 transforms of what differs from the first frame: 2e-6 of the
        # largest coefficient; 16-bit storage rounds each to 8 or 11 bits.
        want, got = (want - want0)[stored], (got - got0)[stored]
        bound = 2e-6 * want.abs().max()
        if spec != "f32":
            bound = bound + 2.0 ** (-7 if spec == "bf16" else -10) * want.abs().max()
        assert torch.all((got - want).abs() <= bound)
    plan.close()
