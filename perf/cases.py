"""Workloads of the gravity library as its users run them, from the smallest
force evaluation to the 2^20-body rubble pile: what is timed, the work each
cannot do without, and what plain 64-bit torch gives for it.

A case is a dict of plain values. ``prepare`` makes the bodies (drawn from the
seed) and the context a program keeps between calls, ``run`` is one pass
through the public entry points, ``exact`` is the same result in 64 bits
without the library.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1912_04197_amd as bhx
from paper_1912_04197_amd import ics


def listed():
    return [
        # One force evaluation of a small cloud with every default (the paper's
        # 1000-body scenes): launches and latency.
        {"name": "accel_1000", "kind": "accel", "shape": "cube", "n": 1000, "leaf": 16,
         "precision": "fp32c", "theta": 0.5, "phi": False, "quad": False},
        # A force and potential evaluation with quadrupole nodes in full FP64
        # (accuracy studies on a Plummer sphere).
        {"name": "accel_quad_20011", "kind": "accel", "shape": "plummer", "n": 20011, "leaf": 16,
         "precision": "fp64", "theta": 0.7, "phi": True, "quad": True},
        # The paper's pulsating cube: 1000 bodies, one-body leaves, FP64,
        # semi-implicit Euler substeps with gravity at every one.
        {"name": "euler_1000", "kind": "euler", "shape": "cube", "n": 1000, "leaf": 1,
         "precision": "fp64", "theta": 0.75, "steps": 20, "every": 1},
        # Plain FP64 leapfrog steps of a mid-size ball.
        {"name": "steps_fp64_50021", "kind": "steps", "shape": "ball", "n": 50021, "leaf": 8,
         "precision": "fp64", "theta": 0.5, "steps": 5},
        # Leapfrog steps of the 131072-body Plummer sphere (uneven density, deep tree).
        {"name": "steps_plummer_131072", "kind": "steps", "shape": "plummer", "n": 131072,
         "leaf": 16, "precision": "fp32c", "theta": 0.5, "steps": 4},
        # The benchmark: the 2^20-body rubble pile, softening length per body.
        {"name": "steps_rubble_1048576", "kind": "steps", "shape": "rubble", "n": 1 << 20,
         "leaf": 4, "precision": "fp32c", "theta": 0.5, "steps": 8},
        # Direct sum of a small cloud in FP64 (below the tree's crossover).
        {"name": "direct_fp64_2048", "kind": "direct", "shape": "cube", "n": 2048,
         "precision": "fp64", "phi": False},
        # Direct sum used as the reference force of a large rubble pile.
        {"name": "direct_fp32c_65536", "kind": "direct", "shape": "rubble", "n": 65536,
         "precision": "fp32c", "phi": False},
        # Many independent scenes a launch, steps captured in a graph.
        {"name": "batched_64", "kind": "batched", "scenes": 64, "lo": 1024, "hi": 16384,
         "leaf": 4, "precision": "fp32c", "theta": 0.5, "steps": 4},
        # Gradient through a tree rollout, recomputed from checkpoints.
        {"name": "rollout_tree_40009", "kind": "rollout", "shape": "ball", "n": 40009, "leaf": 2,
         "precision": "fp32c", "theta": 0.5, "steps": 6, "every": 3, "keep": False},
        # Gradient through a direct-sum rollout with every position kept, FP64.
        {"name": "rollout_direct_8192", "kind": "rollout", "shape": "ball", "n": 8192, "leaf": 16,
         "precision": "fp64", "theta": -1.0, "steps": 4, "every": 2, "keep": True},
        # Aggregate identification at the end of a run.
        {"name": "contacts_200003", "kind": "contacts", "shape": "rubble", "n": 200003},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["accel", "accel", "euler", "steps", "steps", "steps", "direct", "direct",
                       "batched", "rollout", "rollout", "contacts"])
    shape = rng.choice(["cube", "ball", "plummer", "rubble"])
    precision = rng.choice(["fp32c", "fp32c", "fp64"])
    theta = rng.choice([0.5, 0.6, 0.75])
    if kind == "accel":
        quad = rng.random() < 0.3
        return {"kind": kind, "shape": shape, "n": _size(rng, 200, 250000),
                "leaf": rng.choice([1, 4, 8, 16, 16, 24]), "precision": precision, "theta": theta,
                "phi": rng.random() < 0.4, "quad": quad}
    if kind == "euler":
        return {"kind": kind, "shape": shape, "n": _size(rng, 300, 8000),
                "leaf": rng.choice([1, 8, 16]), "precision": precision, "theta": theta,
                "steps": rng.randint(8, 20), "every": rng.choice([1, 2, 5])}
    if kind == "steps":
        top = 150000 if precision == "fp64" or shape == "plummer" else 600000
        return {"kind": kind, "shape": shape, "n": _size(rng, 500, top),
                "leaf": rng.choice([2, 4, 8, 16]), "precision": precision, "theta": theta,
                "steps": rng.randint(1, 5)}
    if kind == "direct":
        return {"kind": kind, "shape": shape, "n": _size(rng, 300, 90000), "precision": precision,
                "phi": rng.random() < 0.4}
    if kind == "batched":
        return {"kind": kind, "scenes": rng.randint(2, 80), "lo": rng.choice([256, 1024]),
                "hi": rng.choice([8192, 16384]), "leaf": rng.choice([4, 8, 16]),
                "precision": precision, "theta": theta, "steps": rng.randint(1, 4)}
    if kind == "rollout":
        direct = rng.random() < 0.4
        return {"kind": kind, "shape": shape, "n": _size(rng, 300, 10000 if direct else 40000),
                "leaf": rng.choice([2, 4, 16]), "precision": precision,
                "theta": -1.0 if direct else theta, "steps": rng.randint(2, 5),
                "every": rng.choice([2, 3, 20]), "keep": rng.random() < 0.5}
    return {"kind": "contacts", "shape": "rubble", "n": _size(rng, 1000, 300000)}


def _scene(shape, n, seed):
    if shape == "cube":
        return ics.uniform_cube(n, seed=seed)
    if shape == "ball":
        return ics.uniform_ball(n, seed=seed)
    if shape == "plummer":
        return ics.plummer(n, seed=seed)
    return ics.rubble_pile(n, seed=seed)


def _scene_sizes(case):
    """Log-spread scene sizes in [lo, hi], in an uneven order."""
    k = case["scenes"]
    f = [(0.6180339887498949 * (s + 1)) % 1.0 for s in range(k)]
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    return [int(round(math.exp(lo + (hi - lo) * x))) for x in f]


def _offsets(case):
    return np.concatenate([[0], np.cumsum(_scene_sizes(case))]).astype(np.int64)


def _inputs(case, seed):
    """The bodies of a case as FP64 GPU tensors: pos, vel, mass, eps or None, and
    the scalar softening."""
    seed = int(seed) % (1 << 40)
    if case["kind"] == "batched":
        parts = [ics.uniform_ball(k, seed=1000 * seed + s)
                 for s, k in enumerate(_scene_sizes(case))]
        pos, vel, mass = (np.concatenate([getattr(p, a) for p in parts])
                          for a in ("pos", "vel", "mass"))
        eps, soft = None, 1e-3
    else:
        sc = _scene(case["shape"], case["n"], seed)
        pos, vel, mass, eps = sc.pos, sc.vel, sc.mass, sc.eps
        soft = 2.0 if case["kind"] == "euler" else sc.softening
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    return up(pos), up(vel), up(mass), None if eps is None else up(eps), soft


def _target(pos, seed):
    g = np.random.Generator(np.random.PCG64(int(seed) % (1 << 40) + 1))
    return pos + torch.from_numpy(0.01 * g.standard_normal(tuple(pos.shape))).cuda()


_DT = {"steps": 5e-4, "euler": 5e-3, "batched": 1e-3, "rollout": 1e-3}


def prepare(case, seed):
    kind = case["kind"]
    pos, vel, mass, eps, soft = _inputs(case, seed)
    n = int(mass.shape[0])
    s = {"case": case, "pos": pos, "vel": vel, "mass": mass, "eps": eps, "soft": soft}
    if kind == "accel" and case["quad"]:
        s["ctx"] = bhx.Context(n, leaf_size=case["leaf"], precision=case["precision"], quad=True)
    elif kind in ("steps", "euler"):
        s["ctx"] = bhx.Context(n, leaf_size=case["leaf"], precision=case["precision"])
        s["acc"] = s["ctx"].compute_accel(pos, mass, case["theta"], softening=soft, eps=eps)
    elif kind == "batched":
        s["off"] = _offsets(case)
        s["ctx"] = bhx.Context(n, leaf_size=case["leaf"], precision=case["precision"],
                               max_scenes=case["scenes"], graph=True)
        s["acc"] = s["ctx"].batched_accel(s["off"], pos, mass, case["theta"], softening=soft)
        # the state that the captured steps advance
        s["now"] = [t.clone() for t in (pos, vel, s["acc"])]
    elif kind == "rollout":
        s["ctx"] = bhx.Context(n, leaf_size=case["leaf"], precision=case["precision"],
                               adjoint=True)
        s["target"] = _target(pos, seed)
    elif kind == "contacts":
        s["ctx"] = bhx.Context(n)
        s["radius"] = 4.0 * eps
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    pos, vel, mass, eps, soft = s["pos"], s["vel"], s["mass"], s["eps"], s["soft"]
    if kind == "accel":
        if case["quad"]:
            return s["ctx"].compute_accel(pos, mass, case["theta"], softening=soft, eps=eps,
                                          potential=case["phi"])
        return bhx.compute_accel(pos, mass, soft, case["theta"], eps=eps, leaf=case["leaf"],
                                 precision=case["precision"], potential=case["phi"])
    if kind == "direct":
        return bhx.compute_accel_direct(pos, mass, soft, eps=eps, precision=case["precision"],
                                        potential=case["phi"])
    if kind == "contacts":
        return s["ctx"].contact_components(pos, mass, s["radius"])
    if kind == "rollout":
        x0, v0, m = (t.clone().requires_grad_() for t in (pos, vel, mass))
        x, v = bhx.rollout(x0, v0, m, s["ctx"], _DT[kind], case["steps"], theta=case["theta"],
                           softening=soft, eps=eps, checkpoint_every=case["every"],
                           keep_positions=case["keep"])
        ((x - s["target"]) ** 2).sum().backward()
        return x.detach(), v.detach(), x0.grad, v0.grad, m.grad
    if kind == "batched":
        p, v, a = s["now"]
        for t, t0 in zip(s["now"], (pos, vel, s["acc"])):
            t.copy_(t0)
        s["ctx"].batched_step(s["off"], p, v, mass, a, _DT[kind], case["steps"],
                              theta=case["theta"], softening=soft)
        return p, v, a
    p, v, a = pos.clone(), vel.clone(), s["acc"].clone()
    if kind == "euler":
        s["ctx"].step_euler(p, v, mass, a, _DT[kind], case["steps"], case["every"],
                            theta=case["theta"], softening=soft, eps=eps)
    else:
        s["ctx"].step_leapfrog(p, v, mass, a, _DT[kind], case["steps"], theta=case["theta"],
                               softening=soft, eps=eps)
    return p, v, a


def _per_body(theta, leaf, n, shape):
    """About how many terms a body's walk sums (fitted, within a third, to counts
    of balls and Plummer spheres of 10^3 to 10^6 bodies)."""
    far = 80.0 * math.log(max(n, 100) / 60.0) * (2.0 if shape == "plummer" else 1.0)
    return min(0.6 * n, far * (1.0 + leaf / 7.0) * (0.5 / theta) ** 2.3)


def work(case):
    """Bytes: inputs read once, outputs written once. Flops: 20 a softened term
    (about twice that for its gradient's share), each term once."""
    kind = case["kind"]
    n = sum(_scene_sizes(case)) if kind == "batched" else case["n"]
    eps = 8 * n if case.get("shape") == "rubble" else 0
    if kind == "contacts":
        return {"bytes": 24 * n + 8 * n + 8 * n + 4 * n, "flops": 10.0 * 30 * n}
    if kind == "direct":
        return {"bytes": 32 * n + eps + 24 * n + (8 * n if case["phi"] else 0),
                "flops": 20.0 * n * (n - 1)}
    if kind == "batched":
        terms = sum(k * _per_body(case["theta"], case["leaf"], k, "ball")
                    for k in _scene_sizes(case))
        return {"bytes": 2 * 72 * n + 8 * n, "flops": 20.0 * terms * case["steps"]}
    per = n - 1 if case["theta"] < 0 else _per_body(case["theta"], case["leaf"], n, case["shape"])
    terms = float(n) * per
    if kind == "accel":
        return {"bytes": 32 * n + eps + 24 * n + (8 * n if case["phi"] else 0),
                "flops": (40.0 if case["quad"] else 20.0) * terms}
    if kind == "steps":
        return {"bytes": 2 * 72 * n + 8 * n + eps, "flops": 20.0 * terms * case["steps"]}
    if kind == "euler":
        return {"bytes": 2 * 72 * n + 8 * n + eps,
                "flops": 20.0 * terms * (case["steps"] // case["every"])}
    # rollout: the forward's steps + 1 evaluations and as many gradients
    return {"bytes": 56 * n + 24 * n + eps + 48 * n + 56 * n,
            "flops": (20.0 + 40.0) * terms * (case["steps"] + 1)}


# ---------------------------------------------------------------- 64 bits
# Barnes-Hut and the direct sum as plain torch in FP64: the octree on the 2^21
# grid of the bounding cube, level by level; each body's own walk, all bodies
# of a chunk at once.


def _spread(v):
    for sh, mask in ((32, 0x1F00000000FFFF), (16, 0x1F0000FF0000FF), (8, 0x100F00F00F00F00F),
                     (4, 0x10C30C30C30C30C3), (2, 0x1249249249249249)):
        v = (v | (v << sh)) & mask
    return v


def _tree_levels(pos, mass, eps2, leaf, scene):
    """Sorted order and, per level, the nodes: first, count, leaf flag, side^2,
    mass, centre of mass, mean eps^2, first child, children."""
    with torch.no_grad():
        ns = int(scene.max()) + 1
        at = scene[:, None].expand(-1, 3)
        lo = torch.full((ns, 3), math.inf, dtype=pos.dtype, device=pos.device)
        hi = -lo
        lo = lo.scatter_reduce(0, at, pos, "amin")
        hi = hi.scatter_reduce(0, at, pos, "amax")
        side = (hi - lo).amax(1)
        side = torch.where(side > 0, side, torch.ones_like(side))
        x0 = (lo + hi) * 0.5 - side[:, None] * 0.5
        q = torch.floor((pos - x0[scene]) * (2097152.0 / side)[scene][:, None])
        q = _spread(q.clamp(0, 2097151).to(torch.int64))
        key = (q[:, 0] << 2) | (q[:, 1] << 1) | q[:, 2]
        order = torch.argsort(key, stable=True)
        order = order[torch.argsort(scene[order], stable=True)]
        key, sc = key[order], scene[order]
    x, m = pos[order], mass[order]
    e2 = None if eps2 is None else eps2[order]
    n = int(m.shape[0])
    levels = []
    active = torch.ones(n, dtype=torch.bool, device=pos.device)
    nid_above = None
    for lvl in range(22):
        with torch.no_grad():
            cell = key >> (3 * (21 - lvl))
            flag = torch.ones_like(active)
            flag[1:] = (cell[1:] != cell[:-1]) | (sc[1:] != sc[:-1])
            flag &= active
            first = torch.nonzero(flag).squeeze(1)
            if first.numel() == 0:
                break
            nid = torch.cumsum(flag, 0) - 1
            body = torch.nonzero(active).squeeze(1)
            count = torch.bincount(nid[body], minlength=first.numel())
            is_leaf = (count <= leaf) | (lvl == 21)
            s2 = (side[sc[first]] * 2.0 ** -lvl) ** 2
            if nid_above is not None:
                up = levels[-1]
                up["nch"] = torch.bincount(nid_above[first], minlength=up["first"].numel())
                up["child0"] = torch.cumsum(up["nch"], 0) - up["nch"]
        k = nid[body]
        nm = torch.zeros(first.numel(), dtype=m.dtype, device=m.device).index_add(0, k, m[body])
        safe = torch.where(nm > 0, nm, torch.ones_like(nm))
        com = torch.zeros((first.numel(), 3), dtype=m.dtype, device=m.device).index_add(
            0, k, m[body, None] * x[body]) / safe[:, None]
        ne2 = None if e2 is None else torch.zeros_like(nm).index_add(
            0, k, m[body] * e2[body]) / safe
        levels.append({"first": first, "count": count, "leaf": is_leaf, "s2": s2, "m": nm,
                       "com": com, "e2": ne2, "scene": sc[first]})
        with torch.no_grad():
            levels[-1]["quad"] = None
            nid_above = nid
            active = active & ~is_leaf[nid.clamp(min=0)]
            levels[-1]["nid"], levels[-1]["body"] = nid, body
    last = levels[-1]
    last["nch"] = torch.zeros_like(last["count"])
    last["child0"] = torch.zeros_like(last["count"])
    return order, x, m, e2, levels


def _add_quads(x, m, levels):
    """Traceless quadrupoles of every node about its centre of mass."""
    for lv in levels:
        b, k = lv["body"], lv["nid"][lv["body"]]
        d = x[b] - lv["com"][k]
        t = 3.0 * d[:, :, None] * d[:, None, :] - (d * d).sum(1)[:, None, None] * torch.eye(
            3, dtype=x.dtype, device=x.device)
        lv["quad"] = torch.zeros((lv["first"].numel(), 3, 3), dtype=x.dtype,
                                 device=x.device).index_add(0, k, m[b, None, None] * t)


def _terms(d, e2, m):
    r2 = (d * d).sum(1) + e2
    live = r2 > 0
    r2 = torch.where(live, r2, torch.ones_like(r2))
    rinv = torch.where(live, 1.0 / torch.sqrt(r2), torch.zeros_like(r2))
    return (m * rinv ** 3)[:, None] * d, -m * rinv, rinv


def _tree_accel(pos, mass, eps, soft, theta, leaf, scene=None, quad=False, chunk=1 << 16):
    """(acc, phi) of every body by its own walk, G = 1."""
    if scene is None:
        scene = torch.zeros(mass.shape[0], dtype=torch.int64, device=pos.device)
    eps2 = None if eps is None else eps * eps
    order, x, m, e2, levels = _tree_levels(pos, mass, eps2, leaf, scene)
    if quad:
        _add_quads(x, m, levels)
    n = int(m.shape[0])
    root = scene[order]
    accs, phis = [], []
    for c0 in range(0, n, chunk):
        c1 = min(n, c0 + chunk)
        acc = torch.zeros((c1 - c0, 3), dtype=x.dtype, device=x.device)
        phi = torch.zeros(c1 - c0, dtype=x.dtype, device=x.device)
        b = torch.arange(c0, c1, device=x.device)
        k = root[b]
        for lv in levels:
            if b.numel() == 0:
                break
            with torch.no_grad():
                leafy = lv["leaf"][k]
                d = lv["com"][k] - x[b]
                ok = ~leafy & (lv["s2"][k] < theta * theta * (d * d).sum(1))
                take, open_ = torch.nonzero(ok).squeeze(1), torch.nonzero(~ok & ~leafy).squeeze(1)
                lf = torch.nonzero(leafy).squeeze(1)
            bb, kk = b[take], k[take]
            d = lv["com"][kk] - x[bb]
            s2 = soft * soft if e2 is None else 0.5 * (e2[bb] + lv["e2"][kk])
            t, p, rinv = _terms(d, s2, lv["m"][kk])
            if quad:
                qd = torch.einsum("pij,pj->pi", lv["quad"][kk], d)
                dqd = (d * qd).sum(1)
                t = t + (2.5 * dqd * rinv ** 7)[:, None] * d - qd * (rinv ** 5)[:, None]
                p = p - 0.5 * dqd * rinv ** 5
            acc = acc.index_add(0, bb - c0, t)
            phi = phi.index_add(0, bb - c0, p)
            with torch.no_grad():
                kl, cnt = k[lf], lv["count"][k[lf]]
                bl = torch.repeat_interleave(b[lf], cnt)
                start = torch.cumsum(cnt, 0) - cnt
                j = torch.repeat_interleave(lv["first"][kl] - start, cnt) + torch.arange(
                    bl.numel(), device=x.device)
                other = j != bl
                bl, j = bl[other], j[other]
            s2 = soft * soft if e2 is None else 0.5 * (e2[bl] + e2[j])
            t, p, _ = _terms(x[j] - x[bl], s2, m[j])
            acc = acc.index_add(0, bl - c0, t)
            phi = phi.index_add(0, bl - c0, p)
            with torch.no_grad():
                ko, cnt = k[open_], lv["nch"][k[open_]]
                b = torch.repeat_interleave(b[open_], cnt)
                start = torch.cumsum(cnt, 0) - cnt
                k = torch.repeat_interleave(lv["child0"][ko] - start, cnt) + torch.arange(
                    b.numel(), device=x.device)
        accs.append(acc)
        phis.append(phi)
    back = torch.empty_like(order)
    back[order] = torch.arange(n, device=order.device)
    return torch.cat(accs)[back], torch.cat(phis)[back]


def _direct_accel(pos, mass, eps, soft):
    n = int(mass.shape[0])
    step = max(1, (1 << 27) // max(n, 1))
    accs, phis = [], []
    for i in range(0, n, step):
        d = pos[None, :, :] - pos[i:i + step, None, :]
        r2 = (d * d).sum(2)
        r2 = r2 + (soft * soft if eps is None else
                   0.5 * ((eps * eps)[None, :] + (eps * eps)[i:i + step, None]))
        own = torch.arange(n, device=pos.device)[None, :] == torch.arange(
            i, min(n, i + step), device=pos.device)[:, None]
        live = ~own & (r2 > 0)
        rinv = torch.where(live, torch.where(live, r2, torch.ones_like(r2)) ** -0.5,
                           torch.zeros_like(r2))
        accs.append(((mass[None, :] * rinv ** 3)[:, :, None] * d).sum(1))
        phis.append(-(mass[None, :] * rinv).sum(1))
    return torch.cat(accs), torch.cat(phis)


def exact(case, seed):
    kind = case["kind"]
    if kind == "contacts":
        return None  # whole numbers
    if kind == "steps" and case["n"] * case["steps"] > 1_500_000:
        return None  # too long in plain torch
    if kind == "batched" and sum(_scene_sizes(case)) * case["steps"] > 1_500_000:
        return None
    if kind == "rollout" and case["n"] * (case["n"] / 20 if case["theta"] < 0 else 1000) \
            * (case["steps"] + 1) > 4e8:
        return None
    pos, vel, mass, eps, soft = _inputs(case, seed)
    if kind == "direct":
        acc, phi = _direct_accel(pos, mass, eps, soft)
        return (acc, phi) if case["phi"] else acc
    theta, leaf = case["theta"], case["leaf"]
    scene = None
    if kind == "batched":
        off = _offsets(case)
        scene = torch.repeat_interleave(torch.arange(case["scenes"]),
                                        torch.from_numpy(np.diff(off))).cuda()

    def force(p, m):
        if theta < 0:
            return _direct_accel(p, m, eps, soft)[0]
        return _tree_accel(p, m, eps, soft, theta, leaf, scene)[0]

    if kind == "accel":
        acc, phi = _tree_accel(pos, mass, eps, soft, theta, leaf, quad=case["quad"])
        return (acc, phi) if case["phi"] else acc
    dt = _DT[kind]
    if kind == "euler":
        a = force(pos, mass)
        for k in range(case["steps"]):
            vel = vel + dt * a
            pos = pos + dt * vel
            if (k + 1) % case["every"] == 0:
                a = force(pos, mass)
        return pos, vel, a
    if kind == "rollout":
        x0, v0, m = (t.requires_grad_() for t in (pos, vel, mass))
    else:
        x0, v0, m = pos, vel, mass
    x, v = x0, v0
    a = force(x, m)
    for _ in range(case["steps"]):
        v = v + 0.5 * dt * a
        x = x + dt * v
        a = force(x, m)
        v = v + 0.5 * dt * a
    if kind != "rollout":
        return x, v, a
    ((x - _target(pos.detach(), seed)) ** 2).sum().backward()
    return x.detach(), v.detach(), x0.grad, v0.grad, m.grad
