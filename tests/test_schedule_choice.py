"""The schedules a plan starts with, and what becomes of them: set again, they
are the same schedules, and the autotuner times them before any other."""
import os
import subprocess

import numpy as np
import pytest

from tests.gpu_util import to_dev
from workloads import make_angles, offsets_from_lengths, random_sequence, upstream_grad


def _a2c():
    import paper_1812_01108_amd as a2c
    return a2c


def _plan(model, lengths, seed=901, **kw):
    off = offsets_from_lengths(lengths)
    R = int(off[-1])
    rng = np.random.Generator(np.random.PCG64(seed))
    seq = random_sequence(rng, R) if model == "fullatom" else None
    plan = _a2c().Plan(model, offsets=off, seq=seq, **kw)
    return plan, to_dev(make_angles(rng, R, "mixture", plan.n_planes))


def _pair(sched):
    return sched["res_per_lane"], sched["waves_per_group"]


def _whole_chain_tiles(lengths, cap):
    """Tiles of whole chains packed in order: at most cap residues, a longer
    chain alone."""
    n, cur = 0, cap + 1
    for L in lengths:
        if L == 0:
            continue
        if cur + L > cap:
            n, cur = n + 1, 0
        cur += L
    return n


# chains a chunk of the recomputing adjoint's own holds whole (100 of 2000
# residues), and chains that it walks chunk by chunk
LONG_BATCHES = {"whole": [2000, 400, 400, 400] * 100,
                "walked": [6000, 1500, 2500, 400] * 20}


@pytest.mark.gpu
@pytest.mark.parametrize("batch", sorted(LONG_BATCHES))
@pytest.mark.parametrize("setter", ["set_adjoint_schedule", "set_schedule"])
def test_reported_adjoint_schedule_set_again(batch, setter):
    """A plan's own adjoint schedule, read and set again (at once, and after
    another one), runs every adjoint form as before, bit for bit."""
    import torch
    lengths = LONG_BATCHES[batch]
    plan, ang = _plan("backbone", lengths)
    g = to_dev(upstream_grad(5, plan.n_atoms))
    coords = plan.forward(ang)

    def results():
        return [plan.backward(ang, g), plan.backward(ang, g, coords=coords),
                plan.mse_step(ang, g)[1]]

    first, sched = results(), plan.adjoint_schedule
    K, W = _pair(sched)
    assert sched["n_tiles"] == _whole_chain_tiles(lengths, 64 * K * W)
    getattr(plan, setter)(K, W)
    for _ in range(2):
        assert plan.adjoint_schedule == sched
        for a, b in zip(first, results()):
            assert torch.equal(a, b)
        getattr(plan, setter)(4, 3)   # away and back
        plan.backward(ang, g)
        getattr(plan, setter)(K, W)


@pytest.mark.parametrize("default,present", [((1, 11), (1, 11)), ((2, 6), (1, 5)), ((4, 4), (8, 3)),
                                             ((1, 1), (1, 1))])
def test_autotuner_times_default_and_present_first(tmp_path, default, present):
    """The candidate list, compiled for the host: the plan's default schedule,
    its present one, then the grid; nothing twice."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src, exe = tmp_path / "list.cpp", tmp_path / "list"
    src.write_text('#include <cstdio>\n#include "schedule.h"\nint main() { for (a2c::Shape s : '
                   'a2c::tune_candidates({%d, %d}, {%d, %d})) std::printf("%%d %%d\\n", s.K, s.W); }\n'
                   % (*default, *present))
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(root, "paper_1812_01108_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    cands = [tuple(int(v) for v in ln.split()) for ln in out.splitlines()]
    assert cands[0] == default and present in cands[:2]
    assert len(set(cands)) == len(cands)
    assert {(k, w) for k in (1, 2, 4, 8) for w in (1, 2, 3, 4, 6, 8, 12, 16)} <= set(cands)


@pytest.mark.gpu
@pytest.mark.parametrize("length,waves", [(180, 3), (120, 2)])
def test_default_forward_counts_the_kernels_own_registers(length, waves):
    """The forward over whole chains runs seven workgroups of up to four waves a
    CU where their LDS allows it (glycines: four atoms), one more than the
    linked one: 6.6 chains a CU, one to a window, are one round."""
    import torch
    n = int(6.6 * torch.cuda.get_device_properties(0).multi_processor_count)
    from workloads import ALPHABET
    off = offsets_from_lengths([length] * n)
    plan = _a2c().Plan("fullatom", offsets=off,
                       seq=np.full(n * length, ALPHABET.index("G"), np.uint8))
    assert plan.schedule == {"res_per_lane": 1, "waves_per_group": waves, "n_tiles": n}


@pytest.mark.gpu
@pytest.mark.parametrize("past", [-1, 1])
def test_full_atom_adjoint_reads_coordinates_up_to_one_round(past):
    """At four waves, two workgroups of six staged planes a CU: up to two
    windows a CU the adjoint reads the coordinates it is given, beyond it
    recomputes the frames.  Linked windows, against the oracle."""
    import torch
    import oracle
    from tests.gpu_util import GRAD_TOL_REL, grad_rel_err
    from workloads import BACKBONE_GEOMETRY
    windows = 2 * torch.cuda.get_device_properties(0).multi_processor_count + past
    lengths = [700] * (windows * 256 // 700) + [windows * 256 % 700]
    off = offsets_from_lengths(lengths)
    rng = np.random.Generator(np.random.PCG64(911))
    seq, ang = random_sequence(rng, int(off[-1])), make_angles(rng, int(off[-1]), "mixture", 7)
    plan = _a2c().Plan("fullatom", offsets=off, seq=seq)
    plan.set_schedule(1, 4)
    a, g = to_dev(ang), upstream_grad(7, plan.n_atoms)
    grad = plan.backward(a, to_dev(g), coords=plan.forward(a))
    ref = oracle.fullatom_backward(off, seq, ang, BACKBONE_GEOMETRY, g)
    assert grad_rel_err(grad.cpu().numpy(), ref, off) <= GRAD_TOL_REL
    off_by = plan.backward(a, to_dev(g), coords=plan.forward(a) + 1.0)
    assert torch.equal(grad, off_by) == (past > 0)
