"""The work that users of this package have it do, as measurable cases.

A case is a dict of plain values.  ``kind`` is the program:

* ``grid_train``   -- ``autograd.persistence_lowerstar`` on one FP32 volume, then the gradient of the
                      total persistence of one dimension (a topological loss on an image or a network
                      output); the loop keeps its filtration workspace from step to step.
* ``grid_reduce``  -- ``api.build_lowerstar`` + ``api.reduce_filtration`` of one volume (analysis: every
                      low, pair and essential simplex).
* ``cloud_train``  -- ``autograd.persistence_vr`` on a batch of FP32 clouds and the gradient of the
                      squared persistence of one dimension (a topological loss on embeddings).
* ``cloud_reduce`` -- ``api.build_vr`` + ``api.reduce_batched`` of integer clouds, each truncated at a
                      percentile of its squared distances.
* ``csc_reduce``   -- ``api.reduce`` of a boundary matrix the caller brings as CSC tensors, with the
                      input check that it has by default.

``workspace`` says whether the program keeps a ``Filtration`` whose buffers are reused (loops do) or
lets every call make a new one (one-off analysis).
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

from paper_1708_04710_amd import api, autograd, synth

_DEV = "cuda"


def listed():
    return [
        # the smallest training step on a volume: a patch of a network's output; launches and
        # host round trips count
        dict(name="grid16_train", kind="grid_train", nx=16, ny=16, nz=16, field="smooth", loss_dim=1, workspace=True),
        # the headline workload: build, reduce, pairs and backward of a 64^3 smooth field
        dict(name="grid64_train", kind="grid_train", nx=64, ny=64, nz=64, field="smooth", loss_dim=1, workspace=True),
        # an odd-sized volume analysed once
        dict(name="grid_ragged_reduce", kind="grid_reduce", nx=37, ny=50, nz=23, field="smooth", workspace=False),
        # unsmoothed data: far more critical simplices per vertex than a smooth field
        dict(name="grid32_noise_reduce", kind="grid_reduce", nx=32, ny=32, nz=32, field="noise", workspace=True),
        # a full volume, as scans come: the largest grid, analysed in a loop over volumes
        dict(name="grid128_reduce", kind="grid_reduce", nx=128, ny=128, nz=128, field="smooth", workspace=True),
        # the smallest cloud: 50 integer points, whole 2-skeleton, one call
        dict(name="cloud50_reduce", kind="cloud_reduce", source="cube", data=1, clouds=1, n_lo=50, n_hi=50, d_lo=3, d_hi=3,
             pct=1.0, maxdim=2, workspace=False),
        # hundreds of uneven truncated clouds as one batch (a data set's diagrams)
        dict(name="clouds512_reduce", kind="cloud_reduce", source="mixed", data=3, clouds=512, n_lo=32, n_hi=256,
             d_lo=2, d_hi=8, pct=0.3, maxdim=2, workspace=True),
        # one larger cloud to dimension 3 (H2 with its deaths)
        dict(name="torus400_dim3_reduce", kind="cloud_reduce", source="torus", data=2, clouds=1, n_lo=400,
             n_hi=400, d_lo=3, d_hi=3, pct=0.2, maxdim=3, workspace=True),
        # one embedding, whole 2-skeleton, with gradient: an ordinary single training step
        dict(name="cloud100_train", kind="cloud_train", clouds=1, n=100, D=3, maxdim=2, loss_dim=1, workspace=True),
        # a batch of noisy circles, whole 2-skeleton, with gradient: a training step on a mini-batch
        dict(name="circles64_train", kind="cloud_train", clouds=64, n=128, D=2, maxdim=2, loss_dim=1, workspace=True),
        # a small batch with H2 in the loss
        dict(name="clouds8_dim3_train", kind="cloud_train", clouds=8, n=31, D=3, maxdim=3, loss_dim=2,
             workspace=True),
        # a caller's own matrix: the 400-point torus to dimension 2 as CSC tensors
        dict(name="csc_torus_reduce", kind="csc_reduce", source="torus", data=2, n=400, D=3, pct=0.2),
    ]


# ------------------------------------------------------------------ draws
def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["grid_train", "grid_reduce", "cloud_train", "cloud_reduce", "csc_reduce"])
    if kind in ("grid_train", "grid_reduce"):
        # sides over 8..128 independently (odd ones and flat boxes among them)
        top = 64 if kind == "grid_train" else 128
        c = dict(kind=kind, nx=_log_int(rng, 8, top), ny=_log_int(rng, 8, top), nz=_log_int(rng, 8, top),
                 field=rng.choice(["smooth", "smooth", "noise"]), workspace=rng.random() < 0.7)
        if c["field"] == "noise":
            for k in ("nx", "ny", "nz"):
                c[k] = min(c[k], 40)
        if kind == "grid_train":
            c["loss_dim"] = rng.choice([0, 1, 1, 2])
        return c
    if kind == "cloud_train":
        maxdim = rng.choice([2, 2, 2, 3])
        n = _log_int(rng, 16, 160) if maxdim == 2 else _log_int(rng, 12, 40)
        clouds = _log_int(rng, 1, 64)
        while clouds > 1 and clouds * _full_simplices(n, maxdim) > 20_000_000:
            clouds //= 2
        return dict(kind=kind, clouds=clouds, n=n, D=rng.randint(2, 8), maxdim=maxdim,
                    loss_dim=rng.choice([0, 1, maxdim - 1]), workspace=rng.random() < 0.7)
    data = rng.randrange(1 << 20)
    if kind == "cloud_reduce":
        maxdim = rng.choice([1, 2, 2, 2, 3])
        workspace = rng.random() < 0.7
        if maxdim == 3:
            n = rng.randint(60, 400)
            return dict(kind=kind, source="torus", data=data, clouds=1, n_lo=n, n_hi=n, d_lo=3, d_hi=3,
                        pct=rng.uniform(0.05, 0.2), maxdim=3, workspace=workspace)
        lo = _log_int(rng, 16, 128)
        hi = _log_int(rng, lo, 256)
        d = rng.randint(2, 4)
        pct = rng.uniform(0.1, 0.35)
        clouds = _log_int(rng, 1, 512)
        while clouds > 1 and clouds * _cloud_simplices(0.5 * (lo + hi), pct, maxdim) > 20_000_000:
            clouds //= 2
        return dict(kind=kind, source=rng.choice(["mixed", "cube"]), data=data, clouds=clouds, n_lo=lo, n_hi=hi,
                    d_lo=d, d_hi=rng.randint(d, 8), pct=pct, maxdim=maxdim, workspace=workspace)
    if rng.random() < 0.5:
        return dict(kind=kind, source="grid", nx=_log_int(rng, 6, 40), ny=_log_int(rng, 6, 40),
                    nz=_log_int(rng, 6, 40))
    return dict(kind=kind, source="torus", data=data, n=_log_int(rng, 30, 400), D=3, pct=rng.uniform(0.1, 0.3))


# ------------------------------------------------------------------ inputs
def _volume(case, seed):
    """FP32 volume (nz, ny, nx): white noise, smoothed over about four cells for ``smooth``."""
    g = torch.Generator().manual_seed(seed)
    f = torch.randn(case["nz"], case["ny"], case["nx"], generator=g, dtype=torch.float64)
    if case["field"] == "smooth":
        t = torch.arange(-16, 17, dtype=torch.float64)
        w = torch.exp(-0.5 * (t / 4.0) ** 2)
        w /= w.sum()
        for ax in range(3):
            n = f.shape[ax]
            i = torch.arange(n)
            a = torch.zeros(n, n, dtype=torch.float64)
            for o, x in zip(range(-16, 17), w.tolist()):
                a[i, (i + o) % n] += x
            f = torch.movedim(torch.tensordot(a, f, dims=([1], [ax])), 0, ax)
        f = (f - f.mean()) / f.std()
    return f.to(torch.float32).contiguous()


def _cloud_batch(case, seed):
    """FP32 (clouds, n, D): noisy unit circles in the first two coordinates."""
    rng = np.random.default_rng(seed)
    a = rng.uniform(0.0, 2.0 * math.pi, (case["clouds"], case["n"]))
    x = np.zeros((case["clouds"], case["n"], case["D"]))
    x[..., 0], x[..., 1] = np.cos(a), np.sin(a)
    return (x + rng.normal(0.0, 0.1, x.shape)).astype(np.float32)


def _int_clouds(case, seed):
    """[(int32 points, squared-distance threshold or -1)].  ``data`` names the data set; a seed is one
    presentation of it, as augmentation makes them: every cloud's points in another order, its axes
    swapped and mirrored.  A truncated complex then keeps its size from seed to seed."""
    if case["source"] == "torus":
        inst = [synth.vr_torus(seed=case["data"], n=case["n_lo"], pct=case["pct"])]
    elif case["source"] == "mixed":
        inst = synth.vr_batch(seed=case["data"], count=case["clouds"], pct=case["pct"],
                              n_range=(case["n_lo"], case["n_hi"]), d_range=(case["d_lo"], case["d_hi"]))
    else:
        rng = np.random.default_rng(case["data"])
        inst = []
        for _ in range(case["clouds"]):
            n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
            D = int(rng.integers(case["d_lo"], case["d_hi"] + 1))
            p = rng.integers(0, 1024, (n, D)).astype(np.int32)
            inst.append((p, -1 if case["pct"] >= 1.0 else synth.percentile_threshold_sqd(p, case["pct"])))
    rng = np.random.default_rng(seed)
    out = []
    for p, thr in inst:
        p = p[rng.permutation(p.shape[0])][:, rng.permutation(p.shape[1])]
        mirror = rng.random(p.shape[1]) < 0.5
        out.append((np.ascontiguousarray(np.where(mirror, 65535 - p, p), dtype=np.int32), thr))
    return out


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, ws=None)
    if case.get("workspace"):
        st["ws"] = api.Filtration(torch.device(_DEV, torch.cuda.current_device()))
    if kind in ("grid_train", "grid_reduce"):
        st["x"] = _volume(case, seed).to(_DEV).requires_grad_(kind == "grid_train")
    elif kind == "cloud_train":
        st["x"] = torch.as_tensor(_cloud_batch(case, seed), device=_DEV).requires_grad_(True)
    elif kind == "cloud_reduce":
        inst = _int_clouds(case, seed)
        st["clouds"] = [torch.as_tensor(p, device=_DEV) for p, _ in inst]
        st["thr"] = [t for _, t in inst]
    else:
        if case["source"] == "grid":
            f = api.build_lowerstar(_volume(dict(case, field="smooth"), seed).to(_DEV))
        else:
            (p, t), = _int_clouds(dict(case, n_lo=case["n"]), seed)
            f, _ = api.build_vr([torch.as_tensor(p, device=_DEV)], [t], 2)
        d = f.to_torch()
        st["csc"] = (d["col_ptr"], d["rows"], d["dim"])
    return st


# ------------------------------------------------------------------ passes
def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "grid_train":
        b, d, dims = autograd.persistence_lowerstar(st["x"], workspace=st["ws"])
        loss = torch.where(dims == case["loss_dim"], d - b, torch.zeros_like(d)).sum()
        return {"birth": b.detach(), "death": d.detach(), "dims": dims, "grad": torch.autograd.grad(loss, st["x"])[0]}
    if kind == "cloud_train":
        b, d, dims, cloud = autograd.persistence_vr(st["x"], case["maxdim"], workspace=st["ws"])
        loss = torch.where(dims == case["loss_dim"], (d - b) ** 2, torch.zeros_like(d)).sum()
        return {"birth": b.detach(), "death": d.detach(), "dims": dims, "cloud": cloud,
                "grad": torch.autograd.grad(loss, st["x"])[0]}
    if kind == "grid_reduce":
        r = api.reduce_filtration(api.build_lowerstar(st["x"], out=st["ws"]))
    elif kind == "cloud_reduce":
        f, off = api.build_vr(st["clouds"], st["thr"], case["maxdim"], out=st["ws"])
        r = api.reduce_batched(f, off)
        return {"low_star": r.low_star, "birth": r.pair_birth, "death": r.pair_death, "essential": r.essential,
                "inst_pair_off": r.inst_pair_off, "inst_ess_off": r.inst_ess_off, "pair_inst": r.pair_inst}
    else:
        r = api.reduce(*st["csc"])
    return {"low_star": r.low_star, "birth": r.pair_birth, "death": r.pair_death, "essential": r.essential}


# ------------------------------------------------------------------ needed work
def _full_simplices(n, maxdim):
    return sum(math.comb(n, k + 1) for k in range(maxdim + 1))


def _grid_simplices(nx, ny, nz):
    """Simplices of the Freudenthal triangulation of an nx x ny x nz grid."""
    x, y, z = nx - 1, ny - 1, nz - 1
    e = x * ny * nz + nx * y * nz + nx * ny * z + x * y * nz + x * ny * z + nx * y * z + x * y * z
    f = 2 * (x * y * nz + x * ny * z + nx * y * z) + 6 * x * y * z
    return nx * ny * nz + e + f + 6 * x * y * z


def _cloud_simplices(n, pct, maxdim):
    """Expected simplices of a truncated cloud: an edge is kept with probability pct, a triangle or
    tetrahedron about as often as the edges of one that share a vertex."""
    return sum(math.comb(int(n), k + 1) * pct ** k for k in range(maxdim + 1))


def work(case):
    """Inputs read once and outputs written once (lows, pairs and essentials of m simplices: about 3
    int32 each; a training step's pair values and gradient).  The reduction has no arithmetic to price."""
    kind = case["kind"]
    if kind == "grid_train":
        v, m = case["nx"] * case["ny"] * case["nz"], _grid_simplices(case["nx"], case["ny"], case["nz"])
        return {"bytes": 8 * v + 8 * m, "flops": 0}
    if kind == "grid_reduce":
        v, m = case["nx"] * case["ny"] * case["nz"], _grid_simplices(case["nx"], case["ny"], case["nz"])
        return {"bytes": 4 * v + 8 * m, "flops": 0}
    if kind == "cloud_train":
        pairs = case["clouds"] * _full_simplices(case["n"], case["maxdim"] - 1)
        pts = 4 * case["clouds"] * case["n"] * case["D"]
        return {"bytes": 2 * pts + 24 * pairs, "flops": 3 * case["clouds"] * math.comb(case["n"], 2) * case["D"]}
    if kind == "cloud_reduce":
        n, D = (case["n_lo"] + case["n_hi"]) / 2, (case["d_lo"] + case["d_hi"]) / 2
        m = case["clouds"] * _cloud_simplices(n, case["pct"], case["maxdim"])
        return {"bytes": int(4 * case["clouds"] * n * D + 8 * m), "flops": 0}
    if case["source"] == "grid":
        m = _grid_simplices(case["nx"], case["ny"], case["nz"])
    else:
        m = _cloud_simplices(case["n"], case["pct"], 2)
    return {"bytes": int((8 + 1 + 3 * 4 + 8) * m), "flops": 0}


# ------------------------------------------------------------------ 64-bit reference
def _pairs(simplices, value):
    """Persistence pairs of a filtration by the twist reduction on Python sets.

    simplices: tuples sorted by (order value, dimension, vertices); value: their values.  Returns
    [(birth index, death index)] ascending in death."""
    pos = {s: i for i, s in enumerate(simplices)}
    top = max(len(s) for s in simplices)
    low, cols, dead = {}, {}, set()
    for size in range(top, 1, -1):
        for j, s in enumerate(simplices):
            if len(s) != size or j in dead:
                continue
            c = {pos[s[:k] + s[k + 1:]] for k in range(size)}
            while c:
                i = max(c)
                o = low.get(i)
                if o is None:
                    low[i] = j
                    cols[j] = c
                    dead.add(i)
                    break
                c ^= cols[o]
    return sorted(((i, j) for i, j in low.items()), key=lambda p: p[1])


def _exact_grid(case, seed):
    x = _volume(case, seed).numpy()
    nz, ny, nx = x.shape
    steps = [(dx, dy, dz) for dx in (0, 1) for dy in (0, 1) for dz in (0, 1) if dx + dy + dz]
    simp = []
    for z, y, xx in itertools.product(range(nz), range(ny), range(nx)):
        stack = [((xx, y, z), (xx + nx * (y + ny * z),), (0, 0, 0))]
        while stack:
            p, s, used = stack.pop()
            simp.append(s)
            for d in steps:
                if any(u and e for u, e in zip(used, d)):
                    continue
                q = tuple(a + e for a, e in zip(p, d))
                if q[0] < nx and q[1] < ny and q[2] < nz:
                    stack.append((q, s + (q[0] + nx * (q[1] + ny * q[2]),), tuple(u | e for u, e in zip(used, d))))
    flat = (x.reshape(-1) + np.float32(0.0)).tolist()
    simp = [tuple(sorted(s)) for s in simp]
    simp.sort(key=lambda s: (max(flat[v] for v in s), len(s), s))
    val = [max(flat[v] for v in s) for s in simp]
    pr = _pairs(simp, val)
    grad = np.zeros(x.size)
    for i, j in pr:
        if len(simp[i]) - 1 == case["loss_dim"]:
            for k, sign in ((i, -1.0), (j, 1.0)):
                grad[max(simp[k], key=lambda v: (flat[v], v))] += sign
    return {"birth": torch.tensor([val[i] for i, _ in pr], dtype=torch.float64),
            "death": torch.tensor([val[j] for _, j in pr], dtype=torch.float64),
            "dims": torch.tensor([len(simp[i]) - 1 for i, _ in pr]),
            "grad": torch.from_numpy(grad.reshape(x.shape))}


def _exact_clouds(case, seed):
    """The order is the FP32 squared distance's (rounded coordinate by coordinate, as the values that
    the filtration is sorted by are); values and gradients are in 64 bits."""
    xs = _cloud_batch(case, seed)
    birth, death, dims, cloud = [], [], [], []
    grad = np.zeros(xs.shape)
    for b, x in enumerate(xs):
        n = x.shape[0]
        key = np.zeros((n, n), np.float32)
        for k in range(x.shape[1]):
            d = x[:, None, k] - x[None, :, k]
            key = key + d * d
        x64 = x.astype(np.float64)
        sq = ((x64[:, None] - x64[None]) ** 2).sum(-1)
        key = key.tolist()
        simp = [(0.0, 0, (v,)) for v in range(n)]
        for k in range(1, case["maxdim"] + 1):
            simp += [(max(key[p][q] for p, q in itertools.combinations(s, 2)), k, s)
                     for s in itertools.combinations(range(n), k + 1)]
        simp.sort()
        simp = [s for _, _, s in simp]
        crit = [None if len(s) == 1 else max(itertools.combinations(s, 2), key=lambda e: (key[e[0]][e[1]], e))
                for s in simp]
        val = [0.0 if e is None else sq[e] for e in crit]
        for i, j in _pairs(simp, val):
            birth.append(val[i])
            death.append(val[j])
            dims.append(len(simp[i]) - 1)
            cloud.append(b)
            if dims[-1] == case["loss_dim"]:
                g = 2.0 * (val[j] - val[i])
                for e, w in ((crit[i], -g), (crit[j], g)):
                    if e is not None:
                        t = 2.0 * w * (x64[e[0]] - x64[e[1]])
                        grad[b, e[0]] += t
                        grad[b, e[1]] -= t
    return {"birth": torch.tensor(birth, dtype=torch.float64), "death": torch.tensor(death, dtype=torch.float64),
            "dims": torch.tensor(dims), "cloud": torch.tensor(cloud), "grad": torch.from_numpy(grad)}


def exact(case, seed):
    """The floating-point cases small enough for plain Python; the others are whole numbers or too large."""
    if case["kind"] == "grid_train" and _grid_simplices(case["nx"], case["ny"], case["nz"]) <= 120_000:
        return _exact_grid(case, seed)
    if case["kind"] == "cloud_train" and case["clouds"] * _full_simplices(case["n"], case["maxdim"]) <= 350_000:
        return _exact_clouds(case, seed)
    return None
