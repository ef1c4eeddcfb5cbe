"""What a launch of a recomputing adjoint waits on: windows in order wait ahead
on at most the 7 after their own, and a batch with a chain over more than 8
windows takes a spine pass and then the windows last to first.  Either way the
launch progresses where the device holds 8 of its workgroups at once.  The form
taken is read off the number of kernels a captured call holds."""
import ctypes

import numpy as np
import pytest

from tests.gpu_util import to_dev
from workloads import make_angles, offsets_from_lengths, random_sequence

pytestmark = pytest.mark.gpu


def _plan(model, lengths):
    import paper_1812_01108_amd as a2c
    off = offsets_from_lengths(lengths)
    R = int(off[-1])
    rng = np.random.Generator(np.random.PCG64(R))
    seq = random_sequence(rng, R) if model == "fullatom" else None
    plan = a2c.Plan(model, offsets=off, seq=seq)
    ang = to_dev(make_angles(rng, R, "mixture", plan.n_planes))
    return plan, ang


def _kernels(run):
    """Kernels a call enqueues (nodes of a graph captured over it)."""
    import torch
    from paper_1812_01108_amd import _lib
    run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        run()
    n = ctypes.c_size_t()
    count = _lib.load().hipGraphGetNodes
    count.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    assert count(graph.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    return n.value


def _calls(plan, ang):
    """The recomputing calls that hand frames and wrenches between windows."""
    import torch
    g = torch.ones((3, plan.n_atoms), device=ang.device)
    grad = torch.empty_like(ang)
    loss = torch.empty(1, device=ang.device)
    calls = {"mse_step": lambda: plan.mse_step(ang, g, grad_angles=grad, loss_out=loss)}
    if plan.model == "fullatom":
        calls["backward"] = lambda: plan.backward(ang, g, grad_angles=grad)
    return calls


@pytest.mark.parametrize("model", ["backbone", "fullatom"])
@pytest.mark.parametrize("K,W", [(1, 1), (2, 2)])
@pytest.mark.parametrize("windows", [8, 9, 32])
def test_windows_wait_on_at_most_seven_ahead(model, K, W, windows):
    cap = 64 * K * W
    # from residue 5 of window 0 into residue 0 of the last of `windows`
    plan, ang = _plan(model, [5, (windows - 1) * cap - 4, 3])
    plan.set_schedule(K, W)
    for name, call in _calls(plan, ang).items():
        assert _kernels(call) == (1 if windows <= 8 else 2), name


@pytest.mark.parametrize("model,lengths", [
    ("fullatom", [2000, 300] * 30), ("fullatom", [1793, 3500, 60]), ("backbone", [3500, 1800, 40])])
def test_default_schedules_need_no_spine_pass(model, lengths):
    """Chains over more than 8 windows of four waves, not of eight."""
    plan, ang = _plan(model, lengths)
    for name, call in _calls(plan, ang).items():
        assert _kernels(call) == 1, (name, plan.adjoint_schedule)
