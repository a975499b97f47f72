"""nfs_reset outside a graph whose first node is the sequence's first push: counters
and status are cleared by the reset and by nothing else."""
import pytest
import torch

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


def frames(n, count, seed):
    g = torch.Generator().manual_seed(seed)
    return (torch.rand((count, n, n), generator=g) * 900 + 50).cuda()


@pytest.mark.parametrize("n", [64, 1024])  # reference in the first batch, and by itself
def test_reset_is_not_put_off_into_a_graph(n):
    import paper_1209_3362_amd as nfs
    require_gpu()
    say(f"reset, then a captured push, n={n}")
    s = torch.cuda.Stream()
    good = frames(n, 6, 2)
    f = good.clone()
    plan = nfs.Plan(n, [1, 2], 8, in_dtype="f32", capacity=16, stream=s)
    out = plan.empty_outputs()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        plan.push(f)
        plan.structure_function(out=out)
        assert plan.work_counters() == (6, 9)
        plan.reset()
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            plan.push(f)
            plan.structure_function(out=out, sync=False)
        # Nothing has run since the reset.
        assert plan.work_counters() == (0, 0)
        # A frame without light: the status stays until the next reset.
        f[3].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert plan.work_counters() == (6, 9) and int(out[3].item()) != 0
        f.copy_(good)
        graph.replay()
        torch.cuda.synchronize()
        assert plan.work_counters() == (12, 18) and int(out[3].item()) != 0
        for _ in range(3):
            plan.reset()
            graph.replay()
            torch.cuda.synchronize()
            assert plan.work_counters() == (6, 9) and int(out[3].item()) == 0
    plan.close()


def test_a_new_plan_starts_cleared(monkeypatch):
    """Workspace full of ones: counters and status of a plan before and after its first push."""
    import paper_1209_3362_amd as nfs
    require_gpu()
    say("a new plan's counters in used memory")
    empty = torch.empty

    def used(*args, **kw):
        t = empty(*args, **kw)
        return t.fill_(255) if t.dtype == torch.uint8 else t

    monkeypatch.setattr(torch, "empty", used)
    plan = nfs.Plan(64, [1, 2], 8, in_dtype="f32", capacity=16)
    monkeypatch.undo()
    assert int(plan.workspace.max().item()) == 255
    assert plan.work_counters() == (0, 0)
    out = plan.structure_function()
    assert int(out[3].item()) == 0 and torch.isnan(out[0]).all()
    plan.push(frames(64, 6, 3))
    assert int(plan.structure_function()[3].item()) == 0 and plan.work_counters() == (6, 9)
    plan.close()
