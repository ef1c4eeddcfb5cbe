"""Timed cases of the map from dihedral angles to coordinates.

Each case is one call, or one training step, as a program that uses this
package makes it: `prepare` builds the packed batch (plan, angles, upstream
gradient or target), `run` makes one pass through the public entry points,
`exact` gives the same outputs from plain torch in 64 bits, `work` the bytes
and operations the path cannot do without.  `listed` are fixed sizes (the
package's own workload shapes among them), `draw` makes more of the same
ranges.

A case's fields:
  model    "backbone" or "fullatom";
  op       "forward"  coordinates into a kept buffer (inference);
           "step"     forward and adjoint on kept buffers (a loop that holds
                      its own buffers and does without autograd);
           "train"    forward and backward through autograd, for an upstream
                      gradient of the coordinates;
           "lrmsd"    a training step on the superposition loss, through
                      autograd;
           "mse"      the fused training step on the squared distance;
           "inverse"  coordinates to angles;
  mode     what the adjoint works from: "coords", "recompute", "auto";
  chains, lo, hi, spread   the number of chains, and their lengths: all `lo`
           ("fixed"), uniform or log-uniform in [lo, hi];
  layout   the seed of the chain lengths and the sequence (the plan's shape;
           the angles, gradients and targets come from prepare's seed);
  tuned    the plan's schedules autotuned on the case's buffers beforehand,
           as a long training run on one batch shape does;
  graph    the step captured in a HIP graph, a pass is one replay.
"""
from __future__ import annotations

import json
import math
import os

import numpy as np
import torch

import paper_1812_01108_amd as a2c

ALPHABET = "ACDEFGHIKLMNPQRSTVWY"
# bond lengths (Angstrom) and bond angles (degrees) of the default backbone:
# transforms placing N (after C), CA (after N) and C (after CA)
SPINE_D = (1.329, 1.458, 1.525)
SPINE_THETA = tuple(math.pi - math.radians(a) for a in (116.2, 121.7, 111.2))


# ------------------------------------------------------------------- the cases

def _case(name, model, op, chains, lo, hi, spread="fixed", mode="auto", layout=0, tuned=False,
          graph=False):
    return {"name": name, "model": model, "op": op, "mode": mode, "chains": chains, "lo": lo,
            "hi": hi, "spread": spread, "layout": layout, "tuned": tuned, "graph": graph}


def listed():
    return [
        # structure of one predicted sequence: the smallest call, all latency
        _case("backbone_1x150_forward", "backbone", "forward", 1, 150, 150),
        # a training step on a small minibatch of peptides
        _case("backbone_16x64_train", "backbone", "train", 16, 64, 64),
        # the usual training shape: one minibatch of 700-residue chains
        _case("backbone_256x700_step", "backbone", "step", 256, 700, 700, mode="coords"),
        # a full backbone batch, ragged, one shape trained for long: tuned,
        # and captured in a graph
        _case("backbone_ragged_4096_train", "backbone", "train", 4096, 20, 1000, "uniform",
              "coords", layout=1003, tuned=True, graph=True),
        # the largest backbone batch, where the plan may keep nothing between
        # the passes (a memory budget of 0)
        _case("backbone_ragged_6000_recompute", "backbone", "train", 6000, 20, 1000, "uniform",
              "recompute", layout=11),
        # large complexes: few chains, each far longer than a workgroup's window
        _case("backbone_long_chains_mse", "backbone", "mse", 48, 1500, 6000, "loguniform",
              layout=12),
        # a training step on a small full-atom minibatch
        _case("fullatom_64x300_step", "fullatom", "step", 64, 300, 300),
        # full-atom training on the superposition loss, captured in a graph
        _case("fullatom_ragged_512_lrmsd", "fullatom", "lrmsd", 512, 50, 2000, "loguniform",
              "recompute", layout=1004, graph=True),
        # the fused full-atom training step, one shape trained for long
        _case("fullatom_ragged_512_mse", "fullatom", "mse", 512, 50, 2000, "loguniform",
              layout=1004, tuned=True),
        # rebuilding a large set of decoys: full-atom coordinates only
        _case("fullatom_decoys_2000x151_forward", "fullatom", "forward", 2000, 151, 151),
        # the largest full-atom training step
        _case("fullatom_ragged_4096_train", "fullatom", "train", 4096, 50, 2000, "loguniform",
              "recompute", layout=13),
        # angles of a set of known structures (targets, initial angles)
        _case("fullatom_ragged_3000_inverse", "fullatom", "inverse", 3000, 30, 1100, "uniform",
              layout=14),
    ]


def draw(rng):
    model = rng.choice(["backbone", "fullatom", "fullatom"])
    op = rng.choice(["forward", "step", "train", "lrmsd", "mse", "inverse"])
    mode = rng.choice(["auto", "coords", "recompute"]) if op in ("step", "train", "lrmsd") else "auto"
    # residues of the batch over the whole range; below the largest listed case
    total = math.exp(rng.uniform(math.log(100.0), math.log(1.5e6 if model == "backbone" else 9e5)))
    lo = int(math.exp(rng.uniform(math.log(20.0), math.log(min(3000.0, total)))))
    spread = rng.choice(["fixed", "uniform", "loguniform"])
    hi = lo if spread == "fixed" else int(lo * rng.uniform(1.3, 30.0)) + 1
    hi = min(hi, 6000)
    if hi <= lo:
        spread, hi = "fixed", lo
    mean = lo if spread == "fixed" else (lo + hi) / 2 if spread == "uniform" else \
        (hi - lo) / math.log(hi / lo)
    chains = max(1, min(8192, int(total / mean)))
    return {"model": model, "op": op, "mode": mode, "chains": chains, "lo": lo, "hi": hi,
            "spread": spread, "layout": rng.randrange(1, 1 << 20), "tuned": rng.random() < 0.2,
            "graph": op in ("train", "lrmsd") and rng.random() < 0.3}


def _lengths(case):
    rng = np.random.Generator(np.random.PCG64(case["layout"]))
    n, lo, hi = case["chains"], case["lo"], case["hi"]
    if case["spread"] == "fixed":
        return np.full(n, lo, dtype=np.int64)
    if case["spread"] == "uniform":
        return rng.integers(lo, hi + 1, size=n)
    return np.rint(np.exp(rng.uniform(math.log(lo), math.log(hi), n))).astype(np.int64)


def work(case):
    R = float(_lengths(case).sum())
    full = case["model"] == "fullatom"
    tab = _table()
    atoms = R * (float(np.mean(tab["n_atoms"])) if full else 3.0)
    chis = R * (float(np.mean(tab["n_chi"])) if full else 0.0)
    angles = 4.0 * (3.0 * R + chis)            # the angles the map depends on
    seq = R if full else 0.0
    grads = 4.0 * R * (7.0 if full else 3.0)   # every plane of the gradient
    xyz = 12.0 * atoms
    # a transform is 27 multiply-adds, an atom 9 to place and 9 for its
    # wrench; a scan and sin/cos of each angle on top (about 60 a transform)
    fwd = 2.0 * (60.0 * (3.0 * R + chis) + 9.0 * atoms)
    bwd = 2.0 * (20.0 * (3.0 * R + chis) + 9.0 * atoms)
    op = case["op"]
    if op == "forward":
        return {"bytes": angles + seq + xyz, "flops": fwd}
    if op == "inverse":
        used = R * (float(np.mean(tab["n_used"])) if full else 0.0)
        return {"bytes": 36.0 * R + 12.0 * used + seq + grads, "flops": 80.0 * (3.0 * R + chis)}
    if op == "mse":
        return {"bytes": angles + seq + 2.0 * xyz + grads, "flops": fwd + bwd}
    if op == "lrmsd":  # angles and target in; coordinates out, angle gradients out
        return {"bytes": angles + seq + 2.0 * xyz + grads, "flops": fwd + bwd + 80.0 * atoms}
    return {"bytes": angles + seq + 2.0 * xyz + grads, "flops": fwd + bwd}


# ------------------------------------------------------------------ the inputs

def _uniform(gen, n, lo=-math.pi, hi=math.pi):
    return lo + (hi - lo) * torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)


def _angles(case, R, gen):
    """Angles [K][R] in 64 bits: phi and psi half helix, four tenths sheet and
    a tenth anywhere, omega trans, chi anywhere.  For the inverse map every
    angle stays 2 degrees off +-pi, where two values stand for one angle."""
    normal = lambda mean, sd: math.radians(mean) + math.radians(sd) * torch.randn(  # noqa: E731
        R, generator=gen, device="cuda", dtype=torch.float64)
    pick = torch.rand(R, generator=gen, device="cuda", dtype=torch.float64)
    out = torch.empty((3 if case["model"] == "backbone" else 7, R), device="cuda",
                      dtype=torch.float64)
    for plane, (helix, sheet) in enumerate((((-63, 10), (-120, 15)), ((-43, 10), (130, 15)))):
        a, b, c = normal(*helix), normal(*sheet), _uniform(gen, R)
        out[plane] = torch.where(pick < 0.5, a, torch.where(pick < 0.9, b, c))
    out[2] = math.pi
    for plane in range(3, out.shape[0]):
        out[plane] = _uniform(gen, R)
    if case["op"] == "inverse":
        out[2] = math.pi - math.radians(2.0) - normal(0, 4).abs()
        out = out.clamp(-math.pi + math.radians(2.0), math.pi - math.radians(2.0))
    return torch.remainder(out + math.pi, 2 * math.pi).sub_(math.pi).to(torch.float32)


def _inputs(case, seed):
    """Everything a case starts from, on the GPU, from the seed alone."""
    gen = torch.Generator("cuda").manual_seed(int(seed))
    lengths = _lengths(case)
    offsets = np.concatenate([[0], np.cumsum(lengths)])
    R = int(offsets[-1])
    seq = None
    if case["model"] == "fullatom":
        seq = np.random.Generator(np.random.PCG64(case["layout"] + 1)).integers(
            0, len(ALPHABET), size=R).astype(np.uint8)
    shape = _Shape(offsets, seq)
    angles = _angles(case, R, gen)
    inp = {"shape": shape, "angles": angles}
    op = case["op"]
    if op == "inverse":
        inp["coords"] = _coords(shape, angles.double())[0].to(torch.float32)
    elif op in ("mse", "lrmsd"):
        # the structure of perturbed angles, for the superposition loss moved
        # rigidly as well
        pert = angles.double()
        noise = math.radians(20.0) * torch.randn(pert.shape, generator=gen, device="cuda",
                                                 dtype=torch.float64)
        noise[2] = 0.0
        t = _coords(shape, pert + noise)[0]
        if op == "lrmsd":
            n = len(lengths)
            q = torch.randn((n, 4), generator=gen, device="cuda", dtype=torch.float64)
            w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
            rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                               2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                               2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)],
                              dim=1).reshape(n, 3, 3)
            move = 10.0 * torch.randn((n, 3), generator=gen, device="cuda", dtype=torch.float64)
            c = shape.chain_of_atom
            t = torch.stack([(rot[c, i] * t.T).sum(1) + move[c, i] for i in range(3)])
        inp["target"] = t.to(torch.float32).contiguous()
    elif op != "forward":
        inp["grad"] = torch.randn((3, shape.A), generator=gen, device="cuda", dtype=torch.float32)
    return inp


def prepare(case, seed):
    inp = _inputs(case, seed)
    shape, angles, op = inp["shape"], inp["angles"], case["op"]
    plan = a2c.Plan(case["model"], offsets=shape.offsets, seq=shape.seq,
                    mem_budget_bytes=0 if case["mode"] == "recompute" else None)
    state = {"op": op, "mode": case["mode"], "plan": plan, "angles": angles}
    if case["tuned"]:
        plan.autotune(angles, inp.get("grad"), from_coords=case["mode"] != "recompute", reps=10,
                      mse_target=inp["target"] if op == "mse" else None)
    if op in ("train", "lrmsd"):
        state["angles"] = angles.requires_grad_(True)
    if op == "lrmsd":
        state["weights"] = torch.ones(plan.n_chains, device="cuda")
    if op in ("forward", "step", "mse"):
        state["coords"] = torch.empty((3, plan.n_atoms), device="cuda")
    if op in ("step", "mse"):
        state["grad_angles"] = torch.empty_like(angles)
    if op == "mse":
        state["loss"] = torch.empty(1, device="cuda")
    if op == "inverse":
        state["coords"], state["out"] = inp["coords"], torch.empty_like(angles)
    for k in ("grad", "target"):
        if k in inp:
            state[k] = inp[k]
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for _ in range(3):
                _pass(state)
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            outputs = _pass(state)
        state["graph"], state["outputs"] = graph, outputs
    return state


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["outputs"]
    return _pass(state)


def _pass(state):
    op, plan, angles = state["op"], state["plan"], state["angles"]
    if op == "forward":
        return {"coords": plan.forward(angles, state["coords"])}
    if op == "step":
        coords = plan.forward(angles, state["coords"])
        g = plan.backward(angles, state["grad"],
                          coords=coords if state["mode"] != "recompute" else None,
                          grad_angles=state["grad_angles"])
        return {"coords": coords, "grad": g}
    if op == "train":
        coords = a2c.angles_to_coords(angles, plan, mode=state["mode"])
        (g,) = torch.autograd.grad(coords, angles, state["grad"])
        return {"coords": coords.detach(), "grad": g}
    if op == "lrmsd":
        coords = a2c.angles_to_coords(angles, plan, mode=state["mode"])
        loss = a2c.lrmsd(coords, state["target"], plan)
        (g,) = torch.autograd.grad(loss, angles, state["weights"])
        return {"coords": coords.detach(), "lrmsd": loss.detach(), "grad": g}
    if op == "mse":
        loss, g = plan.mse_step(angles, state["target"], coords=state["coords"],
                                grad_angles=state["grad_angles"], loss_out=state["loss"])
        return {"coords": state["coords"], "loss": loss, "grad": g}
    return {"angles": plan.coords_to_angles(state["coords"], out=state["out"])}


# ------------------------------------------------- the same in 64 bits, in torch

def _transform(alpha, theta, d):
    """Ry(theta) Tx(d) Rx(alpha) as [n, 3, 4]; theta and d numbers or [n]."""
    n = alpha.shape[0]
    theta, d = (torch.as_tensor(v, device=alpha.device, dtype=torch.float64).expand(n)
                for v in (theta, d))
    ca, sa, ct, st = alpha.cos(), alpha.sin(), theta.cos(), theta.sin()
    zero = torch.zeros_like(alpha)
    return torch.stack([ct, sa * st, ca * st, d * ct, zero, ca, -sa, zero,
                        -st, sa * ct, ca * ct, -d * st], dim=1).reshape(n, 3, 4)


def _compose(a, b):
    r = (a[:, :, :3, None] * b[:, None, :, :]).sum(2)
    r[:, :, 3] += a[:, :, 3]
    return r


def _point(frames, p):
    return (frames[:, :, :3] * p[:, None, :]).sum(2) + frames[:, :, 3]


def _nerf(a, b, c, bond, angle, torsion):
    """The point at `bond` from c, at `angle` (b, c, .) and torsion (a, b, c, .)."""
    bc = (c - b) / np.linalg.norm(c - b)
    n = np.cross(b - a, bc)
    n /= np.linalg.norm(n)
    m = np.cross(n, bc)
    return c + bond * (-math.cos(angle) * bc + math.sin(angle) * math.cos(torsion) * m
                       + math.sin(angle) * math.sin(torsion) * n)


def _table():
    """The residue types as arrays: side frames, and each atom's frame and
    position in it (frames: 0 N, 1 CA, 2 C, 3.. the side frames)."""
    if _table.got is None:
        path = os.path.join(os.path.dirname(a2c.__file__), "data", "residues.json")
        with open(path) as f:
            spec = json.load(f)
        types = {r["code"]: r for r in spec["residues"].values()}
        n_types = len(ALPHABET)
        t = {"n_atoms": np.zeros(n_types, np.int64), "n_side": np.zeros(n_types, np.int64),
             "n_chi": np.zeros(n_types), "n_used": np.zeros(n_types),
             "chi": np.zeros((n_types, 4)), "theta": np.zeros((n_types, 4)),
             "d": np.zeros((n_types, 4)), "pre": np.zeros(n_types),
             "frame": np.zeros((n_types, 14), np.int64), "local": np.zeros((n_types, 14, 3)),
             "quad": np.full((n_types, 4, 4), -1, np.int64)}
        for k, code in enumerate(ALPHABET):
            frames, atoms = types[code]["frames"], spec["backbone_atoms"] + types[code]["atoms"]
            at = {"N": 0, "CA": 1, "C": 2, **{f["origin"]: 3 + i for i, f in enumerate(frames)}}
            slot = {a["name"]: i for i, a in enumerate(atoms)}
            before = {"C": "CA", **{f["origin"]: f["parent"] for f in frames}}
            bond = {"C": SPINE_D[2], **{f["origin"]: f["bond"] for f in frames}}
            t["n_atoms"][k], t["n_side"][k] = len(atoms), len(frames)
            for i, f in enumerate(frames):
                t["chi"][k, i], t["d"][k, i] = 1.0 if f["chi"] else 0.0, f["bond"]
                t["theta"][k, i] = math.pi - math.radians(f["angle"])
                if i == 0:
                    t["pre"][k] = math.radians(f["pre_rotation"])
                # the atom whose torsion is the frame's angle: the next
                # frame's origin, or the frame's atom at azimuth 0
                if f["chi"]:
                    last = [frames[i + 1]["origin"]] if i + 1 < len(frames) else \
                        [a["name"] for a in atoms if a["frame"] == f["origin"]
                         and a["kind"] == "azimuth" and a["azimuth"] == 0.0][:1]
                    up = before[f["parent"]] if f["parent"] != "CA" else "N"
                    t["quad"][k, i] = [slot[n] for n in (up, f["parent"], f["origin"], last[0])]
            t["n_chi"][k] = t["chi"][k].sum()
            t["n_used"][k] = t["n_chi"][k] + 1 if t["n_chi"][k] else 0
            local = {}
            for i, a in enumerate(atoms):
                f = a["frame"]
                if a["kind"] == "origin":
                    p = np.zeros(3)
                elif a["kind"] == "azimuth":
                    ang, z = math.radians(a["angle"]), math.radians(a["azimuth"])
                    p = a["bond"] * np.array([-math.cos(ang), math.sin(ang) * math.sin(z),
                                              -math.sin(ang) * math.cos(z)])
                else:
                    ref = [np.array([-bond[f], 0.0, 0.0]) if r == before.get(f) else local[f, r]
                           for r in a["refs"]]
                    p = _nerf(*ref, a["bond"], math.radians(a["angle"]), math.radians(a["torsion"]))
                local[f, a["name"]] = p
                t["frame"][k, i], t["local"][k, i] = at[f], p
        _table.got = t
    return _table.got


_table.got = None


class _Shape:
    """The packed batch: which chain, residue and frame everything is in."""

    def __init__(self, offsets, seq):
        dev = torch.device("cuda")
        self.offsets, self.seq = offsets, seq
        lengths = torch.from_numpy(np.diff(offsets)).to(dev)
        off = torch.from_numpy(offsets).to(dev)
        self.n_chains, self.R = len(offsets) - 1, int(offsets[-1])
        self.max_len = int(np.diff(offsets).max())
        self.chain = torch.repeat_interleave(torch.arange(self.n_chains, device=dev), lengths)
        self.first, self.end = off[:-1][self.chain], off[1:][self.chain]
        r = torch.arange(self.R, device=dev)
        if seq is None:
            self.type = None
            self.A = 3 * self.R
            self.aoff = 3 * torch.arange(self.R + 1, device=dev)
            self.res_of_atom = torch.repeat_interleave(r, 3)
            self.frame_of_atom = torch.arange(3, device=dev).repeat(self.R)
            self.local = torch.zeros((self.A, 3), device=dev, dtype=torch.float64)
        else:
            tab = _table()
            self.type = torch.from_numpy(seq.astype(np.int64)).to(dev)
            n = torch.from_numpy(tab["n_atoms"]).to(dev)[self.type]
            self.aoff = torch.cat([n.new_zeros(1), n.cumsum(0)])
            self.A = int(self.aoff[-1])
            self.res_of_atom = torch.repeat_interleave(r, n)
            slot = torch.arange(self.A, device=dev) - self.aoff[self.res_of_atom]
            t = self.type[self.res_of_atom]
            self.frame_of_atom = torch.from_numpy(tab["frame"]).to(dev)[t, slot]
            self.local = torch.from_numpy(tab["local"]).to(dev)[t, slot]
        self.chain_of_atom = self.chain[self.res_of_atom]


def _frames(shape, angles):
    """Frames [F][R, 3, 4] of every residue (N, CA, C and the side frames)."""
    steps = [_transform(angles[p], SPINE_THETA[s], SPINE_D[s]) for s, p in enumerate((2, 0, 1))]
    x = _compose(_compose(steps[0], steps[1]), steps[2])
    r = torch.arange(shape.R, device=x.device)
    d = 1
    while d < shape.max_len:  # products over the d residues before, within the chain
        at = torch.nonzero(r - d >= shape.first).squeeze(1)
        x[at] = _compose(x[at - d], x[at])
        d *= 2
    before = torch.roll(x, 1, 0)
    before[r == shape.first] = torch.eye(3, 4, device=x.device, dtype=torch.float64)
    n = _compose(before, steps[0])
    out = [n, _compose(n, steps[1]), x]
    if shape.type is not None:
        tab = {k: torch.from_numpy(v).to(x.device) for k, v in _table().items()}
        pre = tab["pre"][shape.type]
        f = _compose(out[1], _transform(pre, 0.0, 0.0))
        for k in range(4):
            f = _compose(f, _transform(angles[3 + k] * tab["chi"][shape.type, k],
                                       tab["theta"][shape.type, k], tab["d"][shape.type, k]))
            out.append(f)
    return out


def _coords(shape, angles):
    """([3][A], frames): every atom's position."""
    frames = _frames(shape, angles)
    xyz = torch.empty((shape.A, 3), device=angles.device, dtype=torch.float64)
    for k, f in enumerate(frames):
        at = torch.nonzero(shape.frame_of_atom == k).squeeze(1)
        xyz[at] = _point(f[shape.res_of_atom[at]], shape.local[at])
    return xyz.T.contiguous(), frames


def _adjoint(shape, frames, xyz, g):
    """dL/dangle = u . (M - o x G): u and o the axis of the frame that the
    angle turns, G and M the force and moment of every atom it moves."""
    n = len(frames)
    r, g = xyz.T, g.T
    w = torch.cat([g, torch.linalg.cross(r, g)], dim=1)
    group = torch.zeros((shape.R * n, 6), device=r.device, dtype=torch.float64)
    group.index_add_(0, shape.res_of_atom * n + shape.frame_of_atom, w)
    group = group.reshape(shape.R, n, 6)
    whole = group.sum(1)
    upto = whole.cumsum(0)
    after = upto[shape.end - 1] - upto   # every later residue of the chain
    side = group[:, 3:].sum(1)
    moved = [after + whole, after + group[:, 1] + group[:, 2] + side, after + group[:, 2]]
    moved += [group[:, 3 + k:].sum(1) for k in range(n - 3)]
    out = torch.zeros((n, shape.R), device=r.device, dtype=torch.float64)
    for k, plane in enumerate([2, 0, 1, 3, 4, 5, 6][:n]):
        o, u, m = frames[k][:, :, 3], frames[k][:, :, 0], moved[k]
        out[plane] = (u * (m[:, 3:] - torch.linalg.cross(o, m[:, :3]))).sum(1)
    if shape.type is not None:
        out[3:] *= torch.from_numpy(_table()["chi"]).to(r.device)[shape.type].T
    return out


def _torsion(a, b, c, d):
    b1, b2, b3 = b - a, c - b, d - c
    n1, n2 = torch.linalg.cross(b1, b2), torch.linalg.cross(b2, b3)
    return torch.atan2(b2.norm(dim=1) * (b1 * n2).sum(1), (n1 * n2).sum(1))


def _inverse(shape, xyz):
    p, a = xyz.T, shape.aoff
    r = torch.arange(shape.R, device=p.device)
    head, last = r == shape.first, r == shape.end - 1
    n, ca, c = p[a[:-1]], p[a[:-1] + 1], p[a[:-1] + 2]
    prev_ca, prev_c, next_n = torch.roll(ca, 1, 0), torch.roll(c, 1, 0), torch.roll(n, -1, 0)
    prev_ca[head] = torch.tensor([-1.0, 0.0, 0.0], device=p.device, dtype=torch.float64)
    prev_c[head] = 0.0
    psi = _torsion(n, ca, c, next_n)
    psi[last] = 0.0
    out = [_torsion(prev_c, n, ca, c), psi, _torsion(prev_ca, prev_c, n, ca)]
    if shape.type is not None:
        quad = torch.from_numpy(_table()["quad"]).to(p.device)[shape.type]
        for k in range(4):
            has = quad[:, k, 0] >= 0
            q = [p[a[:-1] + quad[:, k, i].clamp(min=0)] for i in range(4)]
            out.append(torch.where(has, _torsion(*q), torch.zeros_like(psi)))
    return torch.stack(out)


def _superposition(shape, xyz, target):
    """(LRMSD of every chain, its gradient by the coordinates [3][A])."""
    c, n = shape.chain_of_atom, shape.n_chains
    count = torch.bincount(c, minlength=n).double()
    total = lambda v: torch.zeros((n, *v.shape[1:]), device=v.device,  # noqa: E731
                                  dtype=torch.float64).index_add_(0, c, v)
    y, x = xyz.T, target.T
    y, x = y - (total(y) / count[:, None])[c], x - (total(x) / count[:, None])[c]
    h = torch.stack([total(y * x[:, j:j + 1]) for j in range(3)], dim=2)  # sum y x^T
    u, _, vt = torch.linalg.svd(h.cpu())
    det = torch.det(u) * torch.det(vt)
    u[:, :, 2] *= torch.sign(det)[:, None]
    rot = (u @ vt).to(h.device)   # carries the target onto the coordinates
    off = y - torch.stack([(rot[c, i] * x).sum(1) for i in range(3)], dim=1)
    val = (total(off.square().sum(1)) / count).sqrt()
    return val, (off / (count * val)[c][:, None]).T


def exact(case, seed):
    inp = _inputs(case, seed)
    shape, op = inp["shape"], case["op"]
    if op == "inverse":
        return {"angles": _inverse(shape, inp["coords"].double())}
    xyz, frames = _coords(shape, inp["angles"].double())
    if op == "forward":
        return {"coords": xyz}
    if op == "mse":
        diff = xyz - inp["target"].double()
        return {"coords": xyz, "loss": diff.square().sum(),
                "grad": _adjoint(shape, frames, xyz, 2.0 * diff)}
    if op == "lrmsd":
        val, g = _superposition(shape, xyz, inp["target"].double())
        return {"coords": xyz, "lrmsd": val, "grad": _adjoint(shape, frames, xyz, g)}
    return {"coords": xyz, "grad": _adjoint(shape, frames, xyz, inp["grad"].double())}
