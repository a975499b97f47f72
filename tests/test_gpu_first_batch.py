"""The first batch of a sequence, which takes the reference frame along, against
the separate passes of the reference (a plan whose batches have no room for one
more frame): spectra bit for bit, counters and status after a reset, replays."""
import pytest
import torch

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16, 32, 64, 128, 256, 512])
@pytest.mark.parametrize("dtype,window,spec,full", [
    ("u16", False, "f32", False), ("f32", True, "f32", True), ("u16", True, "f16", False),
    ("f32", False, "bf16", True)])
def test_reference_along(n, dtype, window, spec, full):
    import paper_1209_3362_amd as nfs
    require_gpu()
    say(f"first batch n={n} {dtype} window={window} {spec} full={full}")
    g = torch.Generator().manual_seed(n)
    f = torch.rand((9, n, n), generator=g) * 4000 + 50
    f = f.to(torch.uint16 if dtype == "u16" else torch.float32)
    w = torch.rand((n, n), generator=g) + 0.5 if window else None
    kw = dict(in_dtype=dtype, window=w, spec=spec, full_spectra=full)
    apart = nfs.Plan(n, [1, 8], 3, capacity=10, host_staging=True, **kw)  # batches of 2
    along = nfs.Plan(n, [1, 8], 3, capacity=64, **kw)
    for _ in range(2):  # the second time after a reset
        apart.push(f.pin_memory())
        along.push(f.cuda())
        assert along.work_counters()[0] == apart.work_counters()[0] == 9
        for t in range(9):
            assert torch.equal(along.spectrum(t), apart.spectrum(t)), t
        a, b = along.structure_function(), apart.structure_function()
        assert int(a[3].item()) == int(b[3].item()) == 0
        assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
        assert torch.all((a[0] - b[0]).abs() <= 1e-6 * b[0].abs())  # few FP32 terms each
        apart.reset()
        along.reset()
        assert along.work_counters() == apart.work_counters() == (0, 0)
    # A reference without light, then a good sequence: the status of the first is cleared.
    z = torch.zeros((3, n, n), dtype=f.dtype)
    status = []
    for p, x in ((apart, z), (along, z.cuda())):
        status.append(int(p.push(x).structure_function()[3].item()))
        p.reset()
    assert status[0] == status[1] != 0
    along.push(f.cuda())
    assert int(along.structure_function()[3].item()) == 0
    apart.close()
    along.close()


def test_replays_clear_the_counters():
    import paper_1209_3362_amd as nfs
    require_gpu()
    say("first batch under capture")
    s = torch.cuda.Stream()
    f = (torch.rand((6, 64, 64), generator=torch.Generator().manual_seed(2)) * 900 + 50).cuda()
    plan = nfs.Plan(64, [1, 2], 8, in_dtype="f32", capacity=16, stream=s)
    out = plan.empty_outputs()
    with torch.cuda.stream(s):
        plan.push(f)
        plan.structure_function(out=out)
        want = [x.clone() for x in out]
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            plan.reset()
            plan.push(f)
            plan.structure_function(out=out, sync=False)
        for _ in range(3):
            for x in out:
                x.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert plan.work_counters() == (6, 9)
            assert all(torch.equal(x, y) for x, y in zip(out, want))
    plan.close()
