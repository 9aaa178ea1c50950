"""The kernels that launch-shape knobs select, each against the FP64 oracle (needs an MI355X): the direct
sums (k_iter, k_forward, k_backward) of the on-the-fly variant and the FP32 matrix kernels (k_sep) of the
separable one.  Without a knob both variants run on the tile kernels.

Bars as for the same calls without a knob: fields within 2e-6 on the scale of their terms, gradients within
1e-4 relative L2, masks within 1e-3 rad on 99.9 % of pixels and |V| within 1e-4."""
import ctypes as C
import math
import sys

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_0907_4027_amd.solver import _dp, _vp, as_slm
from tests.parity import as_complex, assert_phase, assert_stats, assert_V, to_np, wrapped_diff

pytestmark = pytest.mark.gpu

KNOBS = [("onthefly", {"rows": 1}), ("onthefly", {"rows": 2}), ("onthefly", {"fract": 1}),
         ("onthefly", {"segment": 256, "traps_per_lane": 3}), ("separable", {"sep_waves": 4}),
         ("separable", {"sep_waves": 1, "sep_split": 2}), ("separable", {"sep_chunk": 32})]


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu case] {request.node.nodeid}", file=sys.stderr, flush=True)
    yield


@pytest.fixture(params=KNOBS, ids=lambda k: k[0] + "-" + "-".join(f"{a}{b}" for a, b in k[1].items()))
def ctx(hot, request):
    variant, knobs = request.param
    with hot.Context(0) as c:
        c.set_variant(variant)
        c.set_tuning(**knobs)
        yield c


@pytest.mark.parametrize("nx,ny,counts", [(64, 64, [4]), (200, 120, [5, 64, 131]), (545, 70, [100])])
def test_fields_and_gradients(ctx, nx, ny, counts):
    rng = np.random.default_rng(11 * nx + ny)
    slm, T = W.Slm(nx, ny), sum(counts)
    xyz = W.box_uniform(rng, T)
    phi = rng.uniform(0.0, 2.0 * math.pi, (len(counts), ny, nx)).astype(np.float32)
    G = rng.standard_normal((T, 2)).astype(np.float32)
    dphi, dG = torch.tensor(phi, device="cuda"), torch.tensor(G, device="cuda")
    V = to_np(ctx.hot_forward_V(slm, counts, xyz, dphi))
    g = to_np(ctx.hot_adjoint(slm, counts, xyz, dphi, dG))
    o = 0
    for b, m in enumerate(counts):
        flat = phi[b].ravel().astype(np.float64)
        assert np.abs(as_complex(V[o:o + m]) - oracle.forward(slm, xyz[o:o + m], flat)).max() <= 2e-6
        ref = np.ravel(oracle.adjoint(slm, xyz[o:o + m], flat, G[o:o + m, 0].astype(np.float64) + 1j * G[o:o + m, 1]))
        assert np.linalg.norm(g[b].ravel() - ref) <= 1e-4 * np.linalg.norm(ref)
        o += m


@pytest.mark.parametrize("nx,ny,m", [(96, 80, 12), (300, 77, 100)])
def test_solves_and_single_passes(ctx, nx, ny, m):
    """A solve, and the mask that the pixel pass alone leaves behind when the passes are timed."""
    p = W.random_problem(960 + m, nx, ny, m, 3)
    r = ctx.hot_gsw(p.slm, p.xyz, p.theta0, p.iters)
    o = oracle.solve("gsw", p.slm, p.xyz, p.theta0, p.iters)
    assert_phase(to_np(r.phase), o["phi"])
    assert_V(to_np(r.V), o["V"])
    assert_stats(r.stats, o["stats"])
    s, xyz, th = as_slm(p.slm), np.ascontiguousarray(p.xyz), np.ascontiguousarray(p.theta0)
    phase, V, ms = torch.empty(ny, nx, device="cuda"), torch.empty(m, 2, device="cuda"), (C.c_float * 4)()
    assert ctx._lib.hot_time_passes(ctx._ctx, C.byref(s), m, _dp(xyz), _dp(th), 2, _vp(phase), _vp(V), ms) == 0
    assert all(t > 0 for t in ms[:])
    assert_phase(to_np(phase), oracle.backward(p.slm, p.xyz, None, p.theta0))


def test_strong_defocus_reduces_explicitly_by_itself(hot):
    """Traps 3 mm out of focus on the direct sums: lens terms of up to 200 revolutions per block, past the
    margin of the hardware sine's domain, so every argument is reduced without the knob that asks for it
    (the same bits as with it).  An argument of up to 256 revolutions carries 1.5e-5 of rounding (1e-4 rad):
    the mask's error is at most 1e-4 sum(w) / |S_j| rad, the bar 1e-3 where |S_j| >= sum(w) / 10."""
    rng = np.random.default_rng(373)
    xyz = np.column_stack([rng.uniform(-2e-5, 2e-5, 6), rng.uniform(-2e-5, 2e-5, 6), rng.uniform(2.5e-3, 3e-3, 6)])
    slm, theta0 = W.Slm(256, 256), rng.uniform(0, 2 * math.pi, 6)
    with hot.Context(0) as c, hot.Context(0) as k:
        c.set_tuning(rows=1)
        k.set_tuning(rows=1, fract=1)
        r, f = c.hot_rs(slm, xyz, theta0), k.hot_rs(slm, xyz, theta0)
        assert torch.equal(r.phase, f.phase) and torch.equal(r.V, f.V)
    ref, S = oracle.backward(slm, xyz, None, theta0, return_field=True)
    ok = np.abs(S) >= len(xyz) / 10
    assert ok.mean() > 0.8
    assert wrapped_diff(to_np(r.phase).ravel()[ok], ref[ok]).max() <= 1e-3
    assert_V(to_np(r.V), oracle.forward(slm, xyz, to_np(r.phase).ravel()))
