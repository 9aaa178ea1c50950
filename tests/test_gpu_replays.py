"""Solves long enough to replay a captured launch sequence, against the same launches given out one by
one (needs an MI355X).  Both run the same kernels on the same tables, so results agree bit for bit."""
import sys

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

ITERS = 30  # solves of at most 24 iterations on the tile kernels are launched eagerly


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu case] {request.node.nodeid}", file=sys.stderr, flush=True)
    yield


def batch(seed, counts):
    rng = np.random.default_rng(seed)
    T = int(sum(counts))
    return W.box_uniform(rng, T), rng.uniform(0.0, 2.0 * np.pi, T)


def spread(b, total, largest):
    rest = total - largest
    return [largest] + [rest // (b - 1) + (i < rest % (b - 1)) for i in range(b - 1)]


# (variant, knobs, grid, trap counts of one batch, of the next): as many holograms and traps in all and
# the same launch shape, but more traps in the largest hologram, for which a block takes more LDS
PAIRS = [("onthefly", {}, 512, [260, 140], [275, 125]),
         ("separable", {}, 512, [260, 140], [275, 125]),
         ("onthefly", {}, 1024, [300, 20], [310, 10]),
         ("onthefly", {}, 512, spread(8, 880, 144), spread(8, 880, 240)),
         ("separable", {"sep_split": 1}, 512, [260, 140], [275, 125]),
         ("onthefly", {"rows": 1, "traps_per_lane": 3}, 256, [60, 40], [90, 10])]


@pytest.mark.parametrize("variant,knobs,n,first,second", PAIRS)
def test_batches_of_other_counts_do_not_share_a_replay(hot, variant, knobs, n, first, second):
    assert sum(first) == sum(second) and len(first) == len(second) and max(first) < max(second)
    slm, B, T = W.Slm(n, n), len(first), sum(first)
    with hot.Context(0) as eager, hot.Context(0) as c:
        for x in (eager, c):
            x.set_variant(variant)
            x.set_tuning(**knobs)
        eager.set_graphs(False)
        phase, V = torch.empty(B, n, n, device="cuda"), torch.empty(T, 2, device="cuda")
        for counts in (first, second, first):
            xyz, theta0 = batch(3, counts)
            ref = eager.hot_gsw_batched(slm, counts, xyz, theta0, ITERS)
            phase.zero_()
            V.zero_()
            r = c.hot_gsw_batched(slm, counts, xyz, theta0, ITERS, phase=phase, V=V)
            assert torch.equal(r.phase, ref.phase) and torch.equal(r.V, ref.V), counts
            np.testing.assert_array_equal(r.stats, ref.stats)


# every kernel family behind a solve: (variant, knobs, grid, trap counts)
FAMILIES = [("stored", {}, (130, 70), [17]),
            ("onthefly", {"rows": 1}, (300, 77), [37]),
            ("onthefly", {"rows": 2}, (120, 90), [5, 64, 20]),
            ("separable", {"sep_split": 1}, (150, 90), [40]),
            ("separable", {"sep_split": 2}, (96, 64), [33, 7]),
            ("separable", {}, (130, 70), [60]),
            ("onthefly", {}, (64, 60), [700]),
            ("onthefly", {}, (96, 64), [5, 64, 20]),
            ("onthefly", {}, (520, 500), [60, 3, 100, 40])]


@pytest.mark.parametrize("variant,knobs,grid,counts", FAMILIES)
@pytest.mark.parametrize("stats", [False, True])
def test_replays_match_eager(hot, variant, knobs, grid, counts, stats):
    """Several replays, with other work and synchronisations between them."""
    (nx, ny), B, T = grid, len(counts), sum(counts)
    slm = W.Slm(nx, ny)
    xyz, theta0 = batch(4, counts)
    q = W.random_problem(950, 80, 60, 7, 2)
    with hot.Context(0) as eager, hot.Context(0) as c:
        for x in (eager, c):
            x.set_variant(variant)
            x.set_tuning(**knobs)
        eager.set_graphs(False)
        phase = torch.empty(*((B,) if B > 1 else ()), ny, nx, device="cuda")
        V = torch.empty(T, 2, device="cuda")
        if B > 1:
            run = lambda x, **out: x.hot_gsw_batched(slm, counts, xyz, theta0, ITERS, stats=stats, **out)
        else:
            run = lambda x, **out: x.hot_gsw(slm, xyz, theta0, ITERS, stats=stats, **out)
        ref = run(eager)
        for rep in range(4):
            phase.zero_()
            V.zero_()
            r = run(c, phase=phase, V=V)
            torch.cuda.synchronize()
            assert torch.equal(r.phase, ref.phase) and torch.equal(r.V, ref.V), rep
            if stats:
                np.testing.assert_array_equal(r.stats, ref.stats)
            if rep % 2:
                c.hot_gsw(q.slm, q.xyz, q.theta0, 2)  # another problem on the same buffers of the context
                torch.randn(1 << 20, device="cuda").sum()
                torch.cuda.synchronize()
