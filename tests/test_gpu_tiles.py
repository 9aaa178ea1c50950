"""The tile kernels (the default of the on-the-fly and separable variants) at the edges of their
blocks, trap tiles and super-chunks, against the FP64 oracle (needs an MI355X).

Bars: the solver's (phase within 1e-3 rad on 99.9 % of pixels, |V| within 1e-4); gradients and trap
fields of given masks within 2e-6 relative L2: a table entry's FP32 argument is at most 5 revolutions,
so its rounding is at most 2^-22 revolutions (1.5e-6 rad, far less on average), the hardware sin/cos
add 1.2e-7 each and the split products 2^-24 each.
"""
import sys

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from tests.parity import as_complex, assert_phase, assert_stats, assert_V, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu case] {request.node.nodeid}", file=sys.stderr, flush=True)
    yield


# (nx, ny, traps): 32 x 32 blocks with 4 or 8 waves, 64 x 64 blocks (grids of half as many as the
# compute units; of more than the compute units, two to a unit), one and several trap tiles and
# super-chunks, grids off every multiple
EDGES = [(16, 16, 1), (17, 33, 15), (31, 65, 16), (64, 32, 17), (33, 100, 48), (96, 65, 49), (127, 129, 65),
         (700, 840, 5), (705, 769, 40), (769, 705, 97), (700, 840, 257), (1030, 1100, 17), (1030, 1100, 120)]


@pytest.mark.parametrize("nx,ny,m", EDGES)
def test_gsw_at_block_edges(hot, nx, ny, m):
    p = W.random_problem(900 + m, nx, ny, m, 2)
    with hot.Context(0) as c:
        r = c.hot_gsw(p.slm, p.xyz, p.theta0, p.iters, state=True)
        q = c.hot_gsw(p.slm, p.xyz, p.theta0, p.iters, stats=False)
        torch.cuda.synchronize()
    o = oracle.solve("gsw", p.slm, p.xyz, p.theta0, p.iters)
    if m * 64 <= nx * ny:  # (more traps than that on so small a mask: the iterations amplify rounding)
        assert_phase(to_np(r.phase), o["phi"])
        assert_V(to_np(r.V), o["V"])
        assert_stats(r.stats, o["stats"])
    assert torch.equal(r.phase, q.phase) and torch.equal(r.V, q.V)


def relative(x, ref):
    return np.linalg.norm(x - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("nx,ny,counts", [(16, 16, [1, 16]), (33, 31, [17, 3, 33]), (130, 65, [300, 2]),
                                          (512, 257, [64, 5, 100, 31, 48, 16]), (200, 72, [2048]),
                                          (641, 833, [273]), (545, 577, [7, 130, 64, 1])])
def test_fields_and_gradients_at_edges(hot, nx, ny, counts):
    rng = np.random.default_rng(7 * nx + ny)
    slm, T = W.Slm(nx, ny), int(sum(counts))
    xyz = W.box_uniform(rng, T)
    phi = rng.uniform(-40.0, 40.0, (len(counts), ny, nx)).astype(np.float32)
    G = rng.standard_normal((T, 2)).astype(np.float32)
    dphi, dG = torch.tensor(phi, device="cuda"), torch.tensor(G, device="cuda")
    with hot.Context(0) as c:
        V = c.hot_forward_V(slm, counts, xyz, dphi)
        g = c.hot_adjoint(slm, counts, xyz, dphi, dG)
        up = c.hot_adjoint(slm, counts, xyz, dphi, dG * 2.0 ** 60)
        zero = c.hot_adjoint(slm, counts, xyz, dphi, dG * 0.0)
        torch.cuda.synchronize()
    o = 0
    for b, m in enumerate(counts):
        flat = phi[b].ravel().astype(np.float64)
        # V of a mask of random phases is of size 1/sqrt(N): the bar is on the scale of its terms
        ref = oracle.forward(slm, xyz[o:o + m], flat)
        assert np.abs(as_complex(to_np(V[o:o + m])) - ref).max() <= 2e-6
        gr = oracle.adjoint(slm, xyz[o:o + m], flat, G[o:o + m, 0].astype(np.float64) + 1j * G[o:o + m, 1])
        assert relative(to_np(g[b]).ravel(), np.ravel(gr)) <= 2e-6
        o += m
    assert torch.equal(up, g * 2.0 ** 60)  # a power of two in G passes through exactly
    assert not zero.any()


def test_nan_phase_stays_in_its_hologram(hot):
    slm = W.Slm(70, 40)
    xyz = W.box_uniform(np.random.default_rng(5), 9)
    phi = torch.rand(3, 40, 70, device="cuda")
    phi[1, 13, 21] = float("nan")
    with hot.Context(0) as c:
        V = to_np(c.hot_forward_V(slm, [3, 3, 3], xyz, phi))
    assert np.isnan(V[3:6]).all() and np.isfinite(V[:3]).all() and np.isfinite(V[6:]).all()


def test_wide_range_of_weights(hot):
    """Weights over twelve decades: the largest decide the mask; the split of c_m Y_m is scaled by the
    largest weight, so none of them overflows the halves."""
    p = W.random_problem(941, 96, 80, 20)
    w = np.logspace(-6, 6, 20)
    w0 = torch.tensor(w, dtype=torch.float32, device="cuda")
    with hot.Context(0) as c:
        r = c.hot_gsw(p.slm, p.xyz, p.theta0, 0, w0=w0)
        torch.cuda.synchronize()
    ref = oracle.backward(p.slm, p.xyz, to_np(w0), p.theta0)
    assert_phase(to_np(r.phase), ref)


def test_statistics_over_more_masks_than_are_kept(hot):
    """The figures of merit are taken from V of up to 64 masks at a time; 130 iterations take three
    turns, and give what the direct-sum kernels (a launch-shape knob set) give mask by mask."""
    p = W.random_problem(942, 96, 64, 6)
    with hot.Context(0) as c:
        a = c.hot_gsw(p.slm, p.xyz, p.theta0, 130)
        b = c.hot_gsw_noalloc(p.slm, p.xyz, p.theta0, 130)
        c.set_tuning(rows=1)
        d = c.hot_gsw(p.slm, p.xyz, p.theta0, 130)
        torch.cuda.synchronize()
    np.testing.assert_array_equal(a.stats, b.stats)
    assert_stats(a.stats, d.stats)


def test_changing_kernels_on_one_context(hot):
    """Launch-shape knobs select the direct-sum kernels; the tables of one choice are not reused for
    the other, and the first result comes back."""
    p = W.random_problem(943, 150, 90, 24, 3)
    with hot.Context(0) as c:
        a = c.hot_gsw(p.slm, p.xyz, p.theta0, 3)
        c.set_tuning(rows=1)
        b = c.hot_gsw(p.slm, p.xyz, p.theta0, 3)
        c.set_tuning()
        d = c.hot_gsw(p.slm, p.xyz, p.theta0, 3)
        torch.cuda.synchronize()
    assert torch.equal(a.phase, d.phase) and torch.equal(a.V, d.V)
    o = oracle.solve("gsw", p.slm, p.xyz, p.theta0, 3)
    for r in (a, b):
        assert_phase(to_np(r.phase), o["phi"])
        assert_V(to_np(r.V), o["V"])


@pytest.mark.parametrize("nx,ny,m", [(150, 90, 24), (700, 840, 20)])
def test_replays_of_long_solves_match_eager(hot, nx, ny, m):
    """Long solves replay a captured graph: every replay, with other work and synchronisations between
    them, gives the bits of the eager launches."""
    p = W.random_problem(944, nx, ny, m)
    q = W.random_problem(945, 96, 64, 7)
    with hot.Context(0) as eager, hot.Context(0) as c:
        eager.set_graphs(False)
        ref = eager.hot_gsw(p.slm, p.xyz, p.theta0, 30, state=True)
        torch.cuda.synchronize()
        bufs = dict(phase=torch.empty(ny, nx, device="cuda"), V=torch.empty(m, 2, device="cuda"),
                    w_out=torch.empty(m, device="cuda"), theta_out=torch.empty(m, device="cuda"))
        for rep in range(4):
            for b in bufs.values():
                b.zero_()
            r = c.hot_gsw(p.slm, p.xyz, p.theta0, 30, state=True, **bufs)
            assert torch.equal(r.phase, ref.phase) and torch.equal(r.V, ref.V), rep
            assert torch.equal(r.w, ref.w) and torch.equal(r.theta, ref.theta), rep
            np.testing.assert_array_equal(r.stats, ref.stats)
            if rep % 2:
                c.hot_gsw(q.slm, q.xyz, q.theta0, 2)  # another problem on the same buffers of the context
                torch.cuda.synchronize()


@pytest.mark.parametrize("nx,ny,m", [(70, 40, 9), (96, 64, 60), (700, 840, 20)])
@pytest.mark.parametrize("algo_iters", [0, 3])
def test_non_finite_weights(hot, nx, ny, m, algo_iters):
    """A NaN weight makes every sum of Eq. 3 NaN, whose phase is 0: the mask is flat, V is the flat mask's
    field, and neither is an error.  An infinite weight leaves no phase to return: the mask is NaN, its V 0
    (the rounding of the trap sums), and the update meets <|V|> = 0.  Both as the direct sums have it."""
    p = W.random_problem(946, nx, ny, m)
    nan, inf = torch.ones(m, device="cuda"), torch.ones(m, device="cuda")
    nan[m // 2] = float("nan")
    inf[m // 2] = float("inf")
    flat = oracle.forward(p.slm, p.xyz, np.zeros(nx * ny))
    for knobs in ({}, {"rows": 1}):
        with hot.Context(0) as c:
            c.set_tuning(**knobs)
            r = c.hot_gsw(p.slm, p.xyz, p.theta0, algo_iters, w0=nan, state=True)
            assert not r.phase.any()
            # the trap sums are rounded to 2^-30 per block (at most a thousand), the terms are FP32
            assert np.abs(as_complex(to_np(r.V)) - flat).max() <= 5e-6
            assert np.isfinite(r.stats).all()
            w = to_np(r.w)
            assert np.isnan(w[m // 2]) and np.isfinite(np.delete(w, m // 2)).all()
            if algo_iters:
                with pytest.raises(hot.HotError) as e:
                    c.hot_gsw(p.slm, p.xyz, p.theta0, algo_iters, w0=inf)
                assert e.value.code == hot.HOT_EDEGENERATE
            r = c.hot_gsw(p.slm, p.xyz, p.theta0, algo_iters, w0=inf, stats=False)
            assert torch.isnan(r.phase).all() and not r.V.any()


def test_non_finite_gradients_stay_in_their_hologram(hot):
    slm = W.Slm(70, 40)
    rng = np.random.default_rng(6)
    xyz = W.box_uniform(rng, 9)
    phi = torch.tensor(rng.uniform(0, 6, (3, 40, 70)), dtype=torch.float32, device="cuda")
    G = torch.tensor(rng.standard_normal((9, 2)), dtype=torch.float32, device="cuda")
    with hot.Context(0) as c:
        ref = c.hot_adjoint(slm, [3, 3, 3], xyz, phi, G)
        for bad in (float("nan"), float("inf"), -float("inf")):
            H = G.clone()
            H[4, 1] = bad
            g = c.hot_adjoint(slm, [3, 3, 3], xyz, phi, H)
            assert not torch.isfinite(g[1]).any()
            assert torch.equal(g[0], ref[0]) and torch.equal(g[2], ref[2])


@pytest.mark.parametrize("nx,ny,m", [(16, 16, 512), (51, 40, 512), (52, 40, 512), (128, 120, 1280), (96, 257, 1000)])
def test_many_traps_on_small_masks(hot, nx, ny, m):
    """The direct sums take over for many traps on small masks (same bits as with a knob that selects them
    and is their default); either side of the line matches the oracle."""
    p = W.random_problem(947, nx, ny, m)
    direct = m >= 10 * nx and ny <= 256
    with hot.Context(0) as c, hot.Context(0) as k:
        k.set_tuning(rows=1)
        a, b, n = (f(p.slm, p.xyz, p.theta0, 2) for f in (c.hot_gsw, k.hot_gsw, c.hot_gsw_noalloc))
        r = c.hot_rs(p.slm, p.xyz, p.theta0)
        torch.cuda.synchronize()
    assert torch.equal(a.phase, b.phase) == direct
    assert torch.equal(a.phase, n.phase) and torch.equal(a.V, n.V)
    o = oracle.solve("rs", p.slm, p.xyz, p.theta0, 0)
    assert_phase(to_np(r.phase), o["phi"])
    # |V| is of size sqrt(1 / M) here: the bar is on the scale of its terms
    assert np.abs(as_complex(to_np(r.V)) - o["V"]).max() <= 5e-6


@pytest.mark.parametrize("nx,ny,counts", [(64, 40, [896]), (64, 40, [897]), (300, 96, [1000]), (300, 97, [1000]),
                                          (33, 20, [1000, 900])])
def test_fields_of_many_traps_beside_their_adjoint(hot, nx, ny, counts):
    """Eq. 1 of one small mask of very many traps runs on the direct sums, its adjoint on the tile kernels:
    in turn on one context, with the tables of either, they match the oracle and themselves."""
    rng = np.random.default_rng(nx + ny)
    slm, T, B = W.Slm(nx, ny), int(sum(counts)), len(counts)
    xyz = W.box_uniform(rng, T)
    phi = rng.uniform(0.0, 6.0, (B, ny, nx)).astype(np.float32)
    G = rng.standard_normal((T, 2)).astype(np.float32)
    dphi, dG = torch.tensor(phi, device="cuda"), torch.tensor(G, device="cuda")
    direct = B == 1 and T > 896 and -(-nx // 256) * ny <= 192
    with hot.Context(0) as c, hot.Context(0) as k:
        k.set_tuning(rows=1)
        V = [c.hot_forward_V(slm, counts, xyz, dphi)]
        g = [c.hot_adjoint(slm, counts, xyz, dphi, dG)]
        V.append(c.hot_forward_V(slm, counts, xyz, dphi))
        g.append(c.hot_adjoint(slm, counts, xyz, dphi, dG))
        assert torch.equal(V[0], k.hot_forward_V(slm, counts, xyz, dphi)) == direct
        torch.cuda.synchronize()
    assert torch.equal(V[0], V[1]) and torch.equal(g[0], g[1])
    o = 0
    for b, m in enumerate(counts):
        flat = phi[b].ravel().astype(np.float64)
        assert np.abs(as_complex(to_np(V[0][o:o + m])) - oracle.forward(slm, xyz[o:o + m], flat)).max() <= 2e-6
        gr = oracle.adjoint(slm, xyz[o:o + m], flat, G[o:o + m, 0].astype(np.float64) + 1j * G[o:o + m, 1])
        assert relative(to_np(g[0][b]).ravel(), np.ravel(gr)) <= 2e-6
        o += m


@pytest.mark.parametrize("decades", [2, 6, 12])
def test_fields_and_gradients_of_widely_spread_weights(hot, decades):
    """Weights and G over many decades are split relative to the largest: V of the mask and the gradient
    stay within the bars of equal ones (their errors are those of the largest terms)."""
    p = W.random_problem(948, 200, 150, 50)
    rng = np.random.default_rng(decades)
    w = rng.permutation(np.logspace(-decades / 2, decades / 2, p.m))
    w0 = torch.tensor(w, dtype=torch.float32, device="cuda")
    phi = rng.uniform(0.0, 6.0, (1, 150, 200)).astype(np.float32)
    G = (rng.standard_normal((p.m, 2)) * w[:, None]).astype(np.float32)
    with hot.Context(0) as c:
        r = c.hot_gsw(p.slm, p.xyz, p.theta0, 0, w0=w0)
        g = to_np(c.hot_adjoint(p.slm, [p.m], p.xyz, torch.tensor(phi, device="cuda"), torch.tensor(G, device="cuda")))
    mask = oracle.backward(p.slm, p.xyz, to_np(w0), p.theta0)
    assert np.abs(as_complex(to_np(r.V)) - oracle.forward(p.slm, p.xyz, mask)).max() <= 2e-6
    ref = oracle.adjoint(p.slm, p.xyz, phi.ravel().astype(np.float64), G[:, 0].astype(np.float64) + 1j * G[:, 1])
    assert relative(g.ravel(), np.ravel(ref)) <= 2e-6


@pytest.mark.parametrize("nx,ny,m", [(70, 40, 20), (96, 64, 60), (512, 300, 100), (700, 840, 20)])
@pytest.mark.parametrize("variant,knobs", [("onthefly", {}), ("onthefly", {"rows": 1}), ("separable", {"sep_waves": 1})])
def test_adjoint_in_place(hot, nx, ny, m, variant, knobs):
    """The gradient may be written over the phase it is taken at: every pixel's phase is read once, by the
    wave that writes its gradient (two waves share the traps of a tile in the second and third case)."""
    slm, rng = W.Slm(nx, ny), np.random.default_rng(m)
    xyz = W.box_uniform(rng, m)
    phi = torch.tensor(rng.uniform(0.0, 6.0, (1, ny, nx)), dtype=torch.float32, device="cuda")
    G = torch.tensor(rng.standard_normal((m, 2)), dtype=torch.float32, device="cuda")
    with hot.Context(0) as c:
        c.set_variant(variant)
        c.set_tuning(**knobs)
        ref = c.hot_adjoint(slm, [m], xyz, phi, G)
        for _ in range(3):
            x = phi.clone()
            assert torch.equal(c.hot_adjoint(slm, [m], xyz, x, G, grad=x), ref)


@pytest.mark.parametrize("nx,ny,counts,iters,direct", [(1500, 2, [100] * 12, 40, True), (4096, 1, [8, 20, 3] * 3, 30, True),
                                                       (4096, 1, [8, 20, 3], 30, False), (640, 3, [260] * 20, 9, True),
                                                       (1500, 2, [100] * 12, 0, False), (1024, 40, [30] * 16, 30, False)])
def test_batches_of_thin_masks(hot, nx, ny, counts, iters, direct):
    """Batches of masks of a few rows run on the direct sums (same bits as with a knob that selects them and
    is their default); either side of the line matches the oracle."""
    rng = np.random.default_rng(nx + ny)
    slm, T = W.Slm(nx, ny), sum(counts)
    xyz, theta0 = W.box_uniform(rng, T), rng.uniform(0.0, 2.0 * np.pi, T)
    with hot.Context(0) as c, hot.Context(0) as k:
        k.set_tuning(rows=1)
        a, b = (x.hot_gsw_batched(slm, counts, xyz, theta0, iters) for x in (c, k))
        r = c.hot_gsw_batched(slm, counts, xyz, theta0, 0)
        torch.cuda.synchronize()
    assert torch.equal(a.phase, b.phase) == direct
    o = 0
    for i, m in enumerate(counts[:3]):
        ref = oracle.backward(slm, xyz[o:o + m], None, theta0[o:o + m])
        assert_phase(to_np(r.phase[i]), ref)
        assert np.abs(as_complex(to_np(r.V[o:o + m])) - oracle.forward(slm, xyz[o:o + m], ref)).max() <= 5e-6
        o += m


@pytest.mark.parametrize("b,nx,ny,m", [(2, 4096, 16, 50), (4, 32, 2048, 20), (2, 4096, 33, 20)])
def test_half_empty_grids(hot, b, nx, ny, m):
    """As many 64 x 64 blocks as half of the units: masks of up to 32 rows or columns take 32 x 32 ones."""
    rng = np.random.default_rng(ny)
    slm, T = W.Slm(nx, ny), b * m
    xyz, theta0 = W.box_uniform(rng, T), rng.uniform(0.0, 2.0 * np.pi, T)
    with hot.Context(0) as c:
        r = c.hot_gsw_batched(slm, [m] * b, xyz, theta0, 2)
    for i in range(b):
        s = slice(i * m, i * m + m)
        o = oracle.solve("gsw", slm, xyz[s], theta0[s], 2)
        assert_phase(to_np(r.phase[i]), o["phi"])
        assert_V(to_np(r.V[s]), o["V"])
