"""Pushes larger than a transform batch into rings that wrap: frames from host and
from device memory, whose batches differ, are paired in the same windows, so D is
the same bit for bit."""
import pytest
import torch

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,capacity,top,N,chunks", [
    (64, 40, 16, 200, [200]),
    (64, 40, 16, 200, [70, 130]),
    (64, 96, 32, 400, [400]),
    (64, 450, 199, 700, [700]),
    (32, 33, 31, 150, [150]),      # batches of two
    (32, 32, 31, 150, [150]),      # of one
    (128, 300, 64, 700, [1, 699]),
    (256, 420, 300, 900, [900]),
    (1024, 140, 64, 300, [300]),   # the reference by itself
])
@pytest.mark.parametrize("spec,accum,full", [("f32", "plain", False), ("f16", "kahan", True)])
def test_host_and_device_pushes_pair_alike(n, capacity, top, N, chunks, spec, accum, full):
    import paper_1209_3362_amd as nfs
    require_gpu()
    say(f"push windows: {N} frames {n}x{n} in {chunks}, ring {capacity}, delays to {top}, {spec} {accum}")
    g = torch.Generator(device="cuda")
    g.manual_seed(n + N)
    f = torch.randint(500, 3000, (N, n, n), generator=g, device="cuda", dtype=torch.int32)
    f = f.to(torch.uint16)
    lags = sorted({1, 2, 3, 5, 8, top // 2, top - 1, top})
    out = []
    for host in (True, False):
        plan = nfs.Plan(n, lags, n // 2, in_dtype="u16", capacity=capacity, spec=spec, accum=accum,
                        full_spectra=full, host_staging=host)
        t = 0
        for c in chunks:
            part = f[t:t + c]
            plan.push(part.cpu().pin_memory() if host else part)
            t += c
        out.append([x.cpu() for x in plan.structure_function()])
        assert plan.work_counters() == (N, sum(max(0, N - k) for k in lags))
        plan.close()
    for a, b in zip(*out):
        assert torch.equal(torch.nan_to_num(a, nan=-1.0) if a.is_floating_point() else a,
                           torch.nan_to_num(b, nan=-1.0) if b.is_floating_point() else b)
