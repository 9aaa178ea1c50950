"""What a user of this library has it do, from one small mask to holograms of a thousand traps.

Each case is one pass through the public entry points of `paper_0907_4027_amd`.  The grids, trap
counts and iteration counts are those of the workloads, the benchmark and the tests of this
repository, or generic.  Optics: 15 um pitch, 1.064 um light, 5 mm focal length; traps in a box of
40 x 40 x 20 um or on a planar grid of 3 um pitch.

Solvers return what they compute about the traps: V of the final mask, the weights and trap phases
that produced it and the figures of merit.  The mask itself, an angle per pixel, is compared through
V (Eq. 1 over all of its pixels): where its sum S nearly vanishes, or at the cut between 0 and 2 pi,
the last bit of S decides an angle, and iterations carry that on.  One mask is returned whole, as
the field e^{i phase} that a beam simulation takes.  The passes alone return all that they write.
"""
import math

import numpy as np
import torch

import paper_0907_4027_amd as hot

PITCH, WAVELENGTH, FOCAL = 15e-6, 1.064e-6, 5e-3
UM = 1e-6
TWO_PI = 2.0 * math.pi


def listed():
    return [
        # a small mask of a few traps at random superposition, and its field for a beam simulation:
        # a call that is all latency
        {"name": "mask-128x96-10", "kind": "mask", "nx": 128, "ny": 96, "m": 10},
        # weighted Gerchberg-Saxton on a small planar grid of traps, convergence looked at
        {"name": "gsw-256sq-grid16", "kind": "solve", "algo": "gsw", "nx": 256, "ny": 256, "m": 16, "traps": "grid",
         "iters": 30, "variant": "onthefly", "stats": True},
        # two frames of an interactive session: traps that move, five warm-started iterations and the
        # 8-bit frame copied to the host
        {"name": "frames-1024x768-8", "kind": "frames", "nx": 1024, "ny": 768, "m": 8, "iters": 5},
        # a grid that divides by nothing, an odd trap count, few iterations
        {"name": "gsw-641x479-37", "kind": "solve", "algo": "gsw", "nx": 641, "ny": 479, "m": 37, "traps": "box",
         "iters": 10, "variant": "onthefly", "stats": True},
        # plain Gerchberg-Saxton on the paper's 768 x 768 grid
        {"name": "gs-768sq-81", "kind": "solve", "algo": "gs", "nx": 768, "ny": 768, "m": 81, "traps": "box",
         "iters": 20, "variant": "onthefly", "stats": True},
        # the benchmark's hologram: 100 traps in the box, 50 iterations
        {"name": "gsw-512sq-100", "kind": "solve", "algo": "gsw", "nx": 512, "ny": 512, "m": 100, "traps": "box",
         "iters": 50, "variant": "onthefly", "stats": False},
        # the same, shorter, through the separable variant, which a user may choose
        {"name": "sep-512sq-100", "kind": "solve", "algo": "gsw", "nx": 512, "ny": 512, "m": 100, "traps": "box",
         "iters": 10, "variant": "separable", "stats": False},
        # a large hologram of many traps
        {"name": "gsw-1024sq-256", "kind": "solve", "algo": "gsw", "nx": 1024, "ny": 1024, "m": 256, "traps": "box",
         "iters": 40, "variant": "onthefly", "stats": False},
        # the largest: a thousand traps on 2048 x 2048 pixels, a few iterations
        {"name": "gsw-2048sq-1000", "kind": "solve", "algo": "gsw", "nx": 2048, "ny": 2048, "m": 1000, "traps": "box",
         "iters": 3, "variant": "onthefly", "stats": False},
        # a batch of holograms with uneven trap counts
        {"name": "batch-64x512sq", "kind": "batch", "b": 64, "nx": 512, "ny": 512, "mlo": 4, "mhi": 256, "iters": 10},
        # Eq. 1 of given masks: what traps a set of masks really makes
        {"name": "forward-8x512sq-64", "kind": "forward", "b": 8, "nx": 512, "ny": 512, "m": 64},
        # a differentiable hologram's step: V of the masks and the gradient of a loss of V
        {"name": "grad-8x512sq-64", "kind": "grad", "b": 8, "nx": 512, "ny": 512, "m": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mask", "frames", "solve", "solve", "solve", "batch", "forward", "grad"])
    if kind == "mask":
        return {"kind": kind, "nx": rng.randint(48, 144), "ny": rng.randint(48, 112), "m": _log(rng, 3, 40)}
    if kind == "frames":
        return {"kind": kind, "nx": rng.randint(400, 1280), "ny": rng.randint(300, 1024), "m": _log(rng, 4, 40),
                "iters": rng.randint(2, 8)}
    if kind == "solve":
        nx, ny = _log(rng, 200, 1400), _log(rng, 200, 1400)
        m = _log(rng, 6, min(400, nx * ny // 1500))  # (more traps than a mask has room for never settle)
        variant = rng.choice(["onthefly"] * 4 + ["separable"])
        iters = _log(rng, 3, 30 if variant == "onthefly" else 10)
        most = int(5.5e9 / (nx * ny * m))  # no more than the listed ones cost
        return {"kind": kind, "algo": rng.choice(["gsw", "gsw", "gs"]), "nx": nx, "ny": ny, "m": m, "traps": "box",
                "iters": max(1, min(iters, most)), "variant": variant, "stats": rng.random() < 0.5}
    nx, ny = _log(rng, 150, 700), _log(rng, 150, 700)
    if kind == "batch":
        mlo = _log(rng, 3, max(4, nx * ny // 8000))
        return {"kind": kind, "b": _log(rng, 2, 32), "nx": nx, "ny": ny, "mlo": mlo,
                "mhi": mlo + _log(rng, 8, max(9, min(200, nx * ny // 2000))), "iters": _log(rng, 3, 20)}
    return {"kind": kind, "b": _log(rng, 1, 16), "nx": nx, "ny": ny, "m": _log(rng, 4, 200)}


# ---------------------------------------------------------------- inputs

def _rng(case, seed):
    return np.random.default_rng([int(seed) & 0x7FFFFFFF, case["nx"], case["ny"]])


def _box(rng, m):
    return rng.uniform([-20 * UM, -20 * UM, -10 * UM], [20 * UM, 20 * UM, 10 * UM], size=(m, 3))


def _grid(m):
    n = math.isqrt(m - 1) + 1
    xyz = np.zeros((n * n, 3))
    for k in range(n * n):
        xyz[k, :2] = [(k % n - (n - 1) / 2) * 3 * UM, (k // n - (n - 1) / 2) * 3 * UM]
    return xyz[:m]


def _inputs(case, seed):
    """Host inputs of a case, the same for the library and for the 64-bit evaluation."""
    rng = _rng(case, seed)
    k = case["kind"]
    if k == "batch":
        # the trap counts belong to the case, not to the seed
        sizes = np.random.default_rng([case["b"], case["mlo"], case["mhi"]])
        counts = sizes.integers(case["mlo"], case["mhi"] + 1, case["b"]).astype(np.int32)
    elif k in ("forward", "grad"):
        counts = np.full(case["b"], case["m"], dtype=np.int32)
    else:
        counts = np.array([case["m"]], dtype=np.int32)
    total = int(counts.sum())
    xyz = _grid(total) if case.get("traps") == "grid" else _box(rng, total)
    theta = rng.uniform(0.0, TWO_PI, total)
    return rng, counts, xyz, theta


def _poses(rng, xyz):
    """The traps of two consecutive frames: each trap moves by up to 0.2 um."""
    return [xyz, xyz + rng.uniform(-0.2 * UM, 0.2 * UM, xyz.shape)]


def _context(case):
    ctx = hot.Context(0)
    ctx.set_variant(case.get("variant", "onthefly"))
    return ctx


def prepare(case, seed):
    rng, counts, xyz, theta = _inputs(case, seed)
    nx, ny, k = case["nx"], case["ny"], case["kind"]
    ctx = _context(case)
    dev = ctx.device
    s = {"case": case, "ctx": ctx, "slm": hot.hot_slm(nx=nx, ny=ny, pitch=PITCH, wavelength=WAVELENGTH, focal=FOCAL),
         "counts": counts, "xyz": xyz, "theta": theta}
    f32 = {"dtype": torch.float32, "device": dev}
    m, b = int(counts.sum()), len(counts)
    if k in ("mask", "solve", "frames", "batch"):
        s["phase"] = torch.empty((ny, nx) if k != "batch" else (b, ny, nx), **f32)
        s["V"] = torch.empty(m, 2, **f32)
    if k == "mask":
        s["one"] = torch.ones(ny, nx, **f32)
    if k in ("solve", "frames"):
        s["w"], s["th"] = torch.empty(m, **f32), torch.empty(m, **f32)
    if k == "frames":
        s["poses"] = _poses(rng, xyz)
        s["w0"] = torch.tensor(_weights(rng, m), **f32)
        s["out"] = [(torch.empty(m, 2, **f32), torch.empty(m, **f32), torch.empty(m, **f32)) for _ in range(2)]
        s["frame"] = torch.empty(ny, nx, dtype=torch.uint8, device=dev)
        s["host"] = torch.empty(ny, nx, dtype=torch.uint8, pin_memory=True)
    if k in ("forward", "grad"):
        s["phase"] = _masks(case, counts, xyz, theta, dev)
        s["phase"].requires_grad_(k == "grad")
    if k == "grad":
        s["G"] = torch.tensor(rng.standard_normal((m, 2)), **f32)
    torch.cuda.synchronize()
    return s


def _weights(rng, m):
    return rng.uniform(0.8, 1.2, m).astype(np.float32).astype(np.float64)


def run(s):
    case, ctx, k = s["case"], s["ctx"], s["case"]["kind"]
    if k == "mask":
        r = ctx.hot_rs(s["slm"], s["xyz"], s["theta"], phase=s["phase"], V=s["V"], stats=False)
        return [torch.polar(s["one"], r.phase), r.V]
    if k == "solve":
        if case["algo"] == "gs":
            r = ctx.hot_gs(s["slm"], s["xyz"], s["theta"], case["iters"], phase=s["phase"], V=s["V"],
                           stats=case["stats"])
            return _result(r, False)
        r = ctx.hot_gsw(s["slm"], s["xyz"], s["theta"], case["iters"], phase=s["phase"], V=s["V"],
                        stats=case["stats"], state=True, w_out=s["w"], theta_out=s["th"])
        return _result(r, True)
    if k == "frames":
        outs = []
        for xyz, (V, w, th) in zip(s["poses"], s["out"]):
            r = ctx.hot_gsw(s["slm"], xyz, s["theta"], case["iters"], w0=s["w0"], phase=s["phase"], V=V, stats=False,
                            state=True, w_out=w, theta_out=th)
            ctx.hot_encode_u8(r.phase, s["frame"])
            s["host"].copy_(s["frame"], non_blocking=True)
            torch.cuda.current_stream().synchronize()  # the display takes the frame
            outs.append(_result(r, True))
        return outs
    if k == "batch":
        r = ctx.hot_gsw_batched(s["slm"], s["counts"], s["xyz"], s["theta"], case["iters"], phase=s["phase"], V=s["V"],
                                stats=True)
        return _result(r, False)
    if k == "forward":
        return ctx.hot_forward_V(s["slm"], s["counts"], s["xyz"], s["phase"])
    V = hot.TrapField.apply(s["phase"], ctx, s["slm"], s["counts"], s["xyz"])
    (grad,) = torch.autograd.grad(V, s["phase"], s["G"])
    return [V.detach(), grad]


def _result(r, state):
    """V and what else a solver returns about the traps (the figures of merit are 32-bit values)."""
    out = {"V": r.V}
    if state:
        out["w"], out["theta"] = r.w, r.theta
    if r.stats is not None:
        out["stats"] = r.stats.astype(np.float32)
    return out


# ---------------------------------------------------------------- work

def work(case):
    n = case["nx"] * case["ny"]
    k = case["kind"]
    # a term, one (pixel, trap) pair of one pass, is a complex multiply-add: 8 operations
    if k == "mask":
        return {"bytes": 4.0 * n + 40.0 * case["m"], "flops": 8.0 * 2 * n * case["m"]}
    if k == "solve":
        return {"bytes": 4.0 * n + 48.0 * case["m"], "flops": 8.0 * 2 * (case["iters"] + 1) * n * case["m"]}
    if k == "frames":
        return {"bytes": 2 * (4.0 * n + 5.0 * n + 56.0 * case["m"]), "flops": 2 * 8.0 * 2 * (case["iters"] + 1) * n * case["m"]}
    if k == "batch":
        m = case["b"] * (case["mlo"] + case["mhi"]) / 2.0
        return {"bytes": 4.0 * n * case["b"] + 48.0 * m, "flops": 8.0 * 2 * (case["iters"] + 1) * n * m}
    bm = case["b"] * case["m"]
    if k == "forward":
        return {"bytes": 4.0 * n * case["b"] + 32.0 * bm, "flops": 8.0 * n * bm}
    return {"bytes": 12.0 * n * case["b"] + 48.0 * bm, "flops": 8.0 * 2 * n * bm}


# ---------------------------------------------------------------- the same in 64 bits

def _factors(case, xyz, dev):
    """X [nx, M] and Y [ny, M] with e^{i Delta} = X Y (Eq. 2 is a sum of a term in x and one in y)."""
    p = torch.tensor(xyz, dtype=torch.float64, device=dev)

    def factor(n, lateral):
        q = (torch.arange(n, dtype=torch.float64, device=dev) - (n - 1) / 2) * PITCH
        d = p[:, 2] / (2 * WAVELENGTH * FOCAL ** 2) * (q * q)[:, None] + lateral / (WAVELENGTH * FOCAL) * q[:, None]
        return torch.polar(torch.ones_like(d), TWO_PI * (d - torch.floor(d)))

    return factor(case["nx"], p[:, 0]), factor(case["ny"], p[:, 1])


def _sum_over_traps(X, Y, c):
    return (Y * c) @ X.t().contiguous()  # S [ny, nx]


def _sum_over_pixels(X, Y, E):
    return (Y.conj().resolve_conj() * (E @ X.conj().resolve_conj())).sum(0)  # [M]


def _unit(S):
    return torch.where(S == 0, torch.ones_like(S), S / S.abs())


def _split(Z):
    return torch.view_as_real(Z.contiguous())


def _merit(V):
    I = V.abs() ** 2
    return [float(I.sum()), float(1 - (I.max() - I.min()) / (I.max() + I.min())),
            float(torch.sqrt(((I - I.mean()) ** 2).mean()) / I.mean())]


def _solve64(case, algo, xyz, theta, w, iters, dev):
    X, Y = _factors(case, xyz, dev)
    n = case["nx"] * case["ny"]
    th = torch.tensor(theta, dtype=torch.float64, device=dev)
    w = torch.ones_like(th) if w is None else torch.tensor(w, dtype=torch.float64, device=dev)
    stats = []
    for k in range(iters + 1):
        E = _unit(_sum_over_traps(X, Y, torch.polar(w, th)))
        V = _sum_over_pixels(X, Y, E) / n
        stats.append(_merit(V))
        if k < iters:
            if algo == "gsw":
                w = w * V.abs().mean() / V.abs()
            th = V.angle()
    return V, w, th, np.array(stats), E


def _masks(case, counts, xyz, theta, dev):
    """Masks of given traps at random superposition, radians in [0, 2 pi)."""
    out = torch.empty(len(counts), case["ny"], case["nx"], dtype=torch.float32, device=dev)
    o = 0
    for b, m in enumerate(counts):
        X, Y = _factors(case, xyz[o:o + m], dev)
        th = torch.tensor(theta[o:o + m], dtype=torch.float64, device=dev)
        S = _sum_over_traps(X, Y, torch.polar(torch.ones_like(th), th))
        out[b] = torch.remainder(S.angle(), TWO_PI).to(torch.float32)
        o += m
    return out


def exact(case, seed):
    dev = torch.device("cuda", 0)
    rng, counts, xyz, theta = _inputs(case, seed)
    k = case["kind"]
    if k == "mask":
        V, _, _, _, E = _solve64(case, "rs", xyz, theta, None, 0, dev)
        return [E, _split(V)]
    if k == "solve":
        V, w, th, stats, _ = _solve64(case, case["algo"], xyz, theta, None, case["iters"], dev)
        out = {"V": _split(V)}
        if case["algo"] == "gsw":
            out["w"], out["theta"] = w, th
        if case["stats"]:
            out["stats"] = stats
        return out
    if k == "frames":
        poses = _poses(rng, xyz)
        w0 = _weights(rng, int(counts[0]))
        outs = []
        for p in poses:
            V, w, th, _, _ = _solve64(case, "gsw", p, theta, w0, case["iters"], dev)
            outs.append({"V": _split(V), "w": w, "theta": th})
        return outs
    off = np.concatenate([[0], np.cumsum(counts)])
    if k == "batch":
        sol = [_solve64(case, "gsw", xyz[a:b], theta[a:b], None, case["iters"], dev) for a, b in zip(off[:-1], off[1:])]
        return {"V": torch.cat([_split(x[0]) for x in sol]), "stats": np.stack([x[3] for x in sol])}
    phase = _masks(case, counts, xyz, theta, dev).to(torch.float64)
    G = rng.standard_normal((int(counts.sum()), 2)).astype(np.float32).astype(np.float64) if k == "grad" else None
    n = case["nx"] * case["ny"]
    V, grads = [], []
    for b, (lo, hi) in enumerate(zip(off[:-1], off[1:])):
        X, Y = _factors(case, xyz[lo:hi], dev)
        E = torch.polar(torch.ones_like(phase[b]), phase[b])
        V.append(_split(_sum_over_pixels(X, Y, E) / n))
        if G is not None:
            g = torch.view_as_complex(torch.tensor(G[lo:hi], device=dev))
            grads.append((_sum_over_traps(X, Y, g) * E.conj()).imag / n)
    return torch.cat(V) if k == "forward" else [torch.cat(V), torch.stack(grads)]
