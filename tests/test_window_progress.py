"""What a launch of a recomputing adjoint waits on: windows in order wait ahead
on at most the 7 after their own; in a batch with a chain over more than 8
windows the spine aggregates are published first, by as many workgroups of the
same launch (leads) or by a spine pass, and the windows go last to first.  Either
way the launch progresses where the device holds 8 of its workgroups at once.
The form taken is read off the kernels that a captured call holds."""
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


class _KernelNode(ctypes.Structure):
    """hipKernelNodeParams."""
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p),
                ("func", ctypes.c_void_p), ("grid", ctypes.c_uint32 * 3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def _kernels(run):
    """Workgroups of each kernel that a call enqueues, sorted (nodes of a graph
    captured over it)."""
    import torch
    from paper_1812_01108_amd import _lib
    run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        run()
    lib = _lib.load()
    nodes_of, node_params = lib.hipGraphGetNodes, lib.hipGraphKernelNodeGetParams
    nodes_of.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    node_params.argtypes = [ctypes.c_void_p, ctypes.POINTER(_KernelNode)]
    n = ctypes.c_size_t()
    assert nodes_of(graph.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert nodes_of(graph.raw_cuda_graph(), nodes, ctypes.byref(n)) == 0
    grids = []
    for node in nodes:
        p = _KernelNode()
        assert node_params(node, ctypes.byref(p)) == 0
        grids.append(p.grid[0])
    return sorted(grids)


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
@pytest.mark.parametrize("K,W", [(1, 1), (1, 4), (2, 2)])
@pytest.mark.parametrize("windows", [8, 9, 32, 514])
def test_windows_wait_on_at_most_seven_ahead(model, K, W, windows):
    cap = 64 * K * W
    # from residue 5 of window 0 into residue 0 of the last of at most 33 windows
    chains = [5, (min(windows, 33) - 1) * cap - 4, 3]
    plan, ang = _plan(model, chains + [cap] * (windows - min(windows, 33)))
    plan.set_schedule(K, W)
    want = ([windows] if windows <= 8                          # in order
            else [2 * windows] if K == 1 and windows <= 512    # leads
            else [windows, windows])                           # a spine pass
    for name, call in _calls(plan, ang).items():
        assert _kernels(call) == want, name


@pytest.mark.parametrize("model,lengths,waves", [
    # windows of four waves: a chain over more than 8, on few of them and many
    ("fullatom", [2000, 300] * 30, 4), ("fullatom", [2000, 300] * 80, 8),
    ("fullatom", [1793, 3500, 60], 4), ("backbone", [3500, 1800, 40], 4),
    # every chain within 8
    ("fullatom", [1700, 300] * 80, 4)])
def test_default_schedules_need_no_spine_pass(model, lengths, waves):
    plan, ang = _plan(model, lengths)
    assert plan.adjoint_schedule["waves_per_group"] == waves
    for name, call in _calls(plan, ang).items():
        assert len(_kernels(call)) == 1, name


@pytest.mark.parametrize("model,K,W", [("backbone", 1, 2), ("fullatom", 1, 4), ("fullatom", 2, 2)])
def test_replays_between_other_calls_on_the_same_words(model, K, W):
    """A captured call with leads (K = 1) or a spine pass, replayed between eager
    calls of every form, which move the tags of the same words on."""
    import torch
    cap = 64 * K * W
    plan, ang = _plan(model, [9, 10 * cap + 3, 70, cap])
    plan.set_schedule(K, W)
    target = torch.randn((3, plan.n_atoms), device=ang.device)
    coords, loss = plan.forward(ang), torch.empty(1, device=ang.device)
    grads = [torch.empty_like(ang) for _ in range(3)]

    def call(which):
        if which == 0:
            plan.mse_step(ang, target, grad_angles=grads[0], loss_out=loss)
        else:
            plan.backward(ang, target, coords=coords if which == 2 else None,
                          grad_angles=grads[which])
        torch.cuda.synchronize()
        return [grads[which].clone()] + ([loss.clone()] if which == 0 else [])

    want = [call(k) for k in range(3)]
    graphs = []
    for k in range(3):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            if k == 0:
                plan.mse_step(ang, target, grad_angles=grads[0], loss_out=loss)
            else:
                plan.backward(ang, target, coords=coords if k == 2 else None, grad_angles=grads[k])
        graphs.append(graph)
    for replayed, eager in [(0, 1), (1, 2), (2, 0), (0, 0), (1, 1), (0, 2), (0, 1)]:
        for g in grads:
            g.fill_(float("nan"))
        graphs[replayed].replay()
        torch.cuda.synchronize()
        assert torch.equal(grads[replayed], want[replayed][0])
        if replayed == 0:
            assert torch.equal(loss, want[0][1])
        for a, b in zip(call(eager), want[eager]):
            assert torch.equal(a, b)
