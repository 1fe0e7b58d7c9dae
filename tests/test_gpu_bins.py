"""The binned form of the type-sorted sums, at the sizes where it can go wrong.

Profiles are held to 1e-6 of the FP64 oracle at every q and gradients to 1e-5
in norm and at the worst atom, the bounds stated for these paths.  A call whose
sums were binned reports variant() == (0, 0)."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import oracle
import workloads as W
from tests.gradcheck import GTOL, assert_grad_close

pytestmark = pytest.mark.gpu

TOL = 1e-6


@pytest.fixture(scope="module")
def sd():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1306_2258_amd as mod

    return mod


def say(msg):
    print(f"[case] {msg}", flush=True)
    sys.stdout.flush()


def dev(m):
    import torch

    return (torch.from_numpy(m.coords).cuda(), torch.from_numpy(m.types).cuda(), torch.from_numpy(m.table).cuda())


def close(got, ref):
    assert np.all(np.isfinite(got))
    err = np.abs(got - ref) / np.abs(ref)
    assert err.max() <= TOL, f"max rel err {err.max():.3e} at q[{err.argmax()}]"


def check(sd, m, binned=True):
    ctx = sd.Context(0)
    got = sd.debye_profile(*dev(m), m.q, ctx=ctx).cpu().numpy()
    assert (ctx.variant() == (0, 0)) == binned
    close(got, oracle.profile(m.coords, m.types, m.table, m.q))
    return got


# first sizes binned on a uniform and on any grid; tiles of 64 and items of 16,
# 32 and 64 swept atoms; the last size of the one-kernel pack and the next
@pytest.mark.parametrize("n", [128, 129, 191, 193, 301, 302, 1023, 1025, 2047, 2048, 2049, 4097])
@pytest.mark.parametrize("grid", ["uniform", "log"])
def test_sizes(sd, n, grid):
    say(f"binned N={n} {grid}")
    q = W.log_grid(1e-3, 0.9, 41) if grid == "log" else None
    m = W.random_molecule(7000 + n, n, 41, q1=0.9, extent=3.0 * n ** (1 / 3) + 2.0, q=q)
    check(sd, m, n >= (302 if grid == "log" else 129))


@pytest.mark.parametrize("nq", [7, 8, 63, 64, 65, 129, 300])
def test_q_counts(sd, nq):
    say(f"binned Nq={nq}")
    check(sd, W.random_molecule(7100 + nq, 700, nq, q1=1.0, extent=25.0), nq >= 8)


# types: one; those of the small pack (T <= 16) and beyond; the largest; empty
# segments and segments of one atom
@pytest.mark.parametrize("t", [1, 2, 16, 17, 63, 64, 65])
def test_types(sd, t):
    say(f"binned T={t}")
    m = W.random_molecule(7200 + t, 1900, 24, t=t, q1=0.8, extent=22.0, widths=np.linspace(0.2, 1.4, t))
    if t > 4:
        m.types[m.types == 1] = 0
        m.types[m.types == 3] = 0
        m.types[-1] = 3
    ctx = sd.Context(0)
    got = sd.debye_profile(*dev(m), m.q, ctx=ctx).cpu().numpy()
    assert t > 64 or ctx.variant() == (0, 0)
    close(got, oracle.profile(m.coords, m.types, m.table, m.q))


# 0.52 / q per bin, 6,592 bins a window: just inside one, in two, in four, and
# too many for any
@pytest.mark.parametrize("span", [3390.0, 3440.0, 6800.0, 13500.0, 20000.0])
def test_windows(sd, span):
    say(f"binned, {span:g} A long")
    m = W.random_molecule(7300, 5000, 32, t=2, q1=1.0, extent=30.0)
    m.coords[:, 0] *= np.float32(span / 30.0)
    check(sd, m)


def test_full_bins(sd):
    """Millions of pairs of one distance: bins are emptied between rounds."""
    say("binned, atoms on two sites")
    m = W.random_molecule(7400, 3000, 20, t=2, q1=0.9, extent=20.0)
    m.coords[:1700] = m.coords[0]
    m.coords[1700:2990] = m.coords[2999]
    check(sd, m)


def test_far_from_the_origin(sd):
    say("binned, off centre")
    m = W.random_molecule(7500, 900, 30, q1=0.9, extent=24.0)
    m.coords += np.float32(4096.0)
    check(sd, m)


@pytest.mark.parametrize("n", [800, 3000])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_non_finite_coordinate_takes_the_other_form(sd, value, n):
    say(f"a coordinate of {value}, N={n}")
    m = W.random_molecule(7600, n, 16, q1=0.9, extent=20.0)
    m.coords[17, 1] = value
    ctx, old = sd.Context(0), sd.Context(0)
    old.set_form("direct")
    got = sd.debye_profile(*dev(m), m.q, ctx=ctx).cpu().numpy()
    ref = sd.debye_profile(*dev(m), m.q, ctx=old).cpu().numpy()
    assert np.array_equal(np.isfinite(got), np.isfinite(ref))


def test_batch_of_all_kinds(sd):
    """Compact, sparse, tiny and empty structures of one batch, each as alone."""
    import torch

    say("binned batch")
    q = W.q_grid(0.0, 1.0, 40)
    parts = [W.random_molecule(7700 + k, n, 40, q1=1.0, extent=e) for k, (n, e) in
             enumerate([(900, 24.0), (0, 1.0), (300, 9000.0), (1, 5.0), (2500, 34.0), (64, 9.0), (3000, 40000.0), (129, 12.0)])]
    off = np.concatenate([[0], np.cumsum([p.n for p in parts])]).astype(np.int64)
    c = torch.from_numpy(np.concatenate([p.coords.reshape(-1, 3) for p in parts])).cuda()
    t = torch.from_numpy(np.concatenate([p.types for p in parts])).cuda()
    tab = torch.from_numpy(parts[0].table).cuda()
    ctx = sd.Context(0)
    got = sd.debye_profile_batched(c, t, off, tab, q, ctx=ctx)
    assert ctx.variant() == (0, 0)
    plan = sd.BatchedPlan(c, t, off, tab, q, ctx=ctx)
    for _ in range(3):
        assert torch.equal(plan.execute(), got)
    for s, p in enumerate(parts):
        if p.n == 0:
            assert torch.all(got[s] == 0.0)
            continue
        close(got[s].cpu().numpy(), oracle.profile(p.coords, p.types, p.table, q))
        alone = sd.debye_profile(c[off[s]:off[s + 1]].contiguous(), t[off[s]:off[s + 1]].contiguous(), tab, q, ctx=ctx)
        if ctx.variant() == (0, 0) and s in (0, 4):
            assert torch.equal(alone, got[s])


@pytest.mark.parametrize("n,t", [(129, 5), (255, 1), (1000, 17), (2049, 5), (3500, 2), (1500, 64)])
def test_coordinate_gradient(sd, n, t):
    import torch

    say(f"binned gradient N={n} T={t}")
    m = W.random_molecule(7800 + n, n, 30, t=t, q1=0.8, extent=3.0 * n ** (1 / 3) + 2.0, widths=np.linspace(0.2, 1.4, t))
    m.coords[7] = m.coords[3]
    w = np.random.default_rng(n).normal(size=30)
    ctx = sd.Context(0)
    g, prof = sd.debye_grad(*dev(m), m.q, torch.from_numpy(w).cuda(), ctx=ctx, with_profile=True)
    close(prof.cpu().numpy(), oracle.profile(m.coords, m.types, m.table, m.q))
    assert_grad_close(g.cpu().numpy(), oracle.grad(m.coords, m.types, m.table, m.q, w), GTOL, f"N={n} T={t}")


@pytest.mark.parametrize("span", [3390.0, 3440.0, 20000.0])
def test_coordinate_gradient_of_long_molecules(sd, span):
    """One window of bins has a gradient of its own; more take the adjoint."""
    import torch

    say(f"binned gradient, {span:g} A long")
    m = W.random_molecule(7900, 2500, 20, t=2, q1=1.0, extent=30.0)
    m.coords[:, 0] *= np.float32(span / 30.0)
    w = np.random.default_rng(3).normal(size=20)
    g = sd.debye_grad(*dev(m), m.q, torch.from_numpy(w).cuda())
    assert_grad_close(g.cpu().numpy(), oracle.grad(m.coords, m.types, m.table, m.q, w), GTOL, f"{span:g} A")


@pytest.mark.parametrize("n,t,nq", [(129, 2, 8), (700, 5, 65), (1999, 16, 33), (2500, 3, 130)])
def test_table_gradient(sd, n, t, nq):
    import torch

    say(f"binned table gradient N={n} T={t} Nq={nq}")
    m = W.random_molecule(8000 + n, n, nq, t=t, q1=0.8, extent=3.0 * n ** (1 / 3) + 2.0, widths=np.linspace(0.2, 1.4, t))
    w = np.random.default_rng(n).normal(size=nq)
    g, prof = sd.debye_grad_table(*dev(m), m.q, torch.from_numpy(w).cuda(), with_profile=True)
    ref = oracle.grad_table(m.coords, m.types, m.table, m.q, w)
    assert np.linalg.norm(g.cpu().numpy() - ref) <= GTOL * np.linalg.norm(ref)
    close(prof.cpu().numpy(), oracle.profile(m.coords, m.types, m.table, m.q))


@pytest.mark.parametrize("n", [300, 1500, 6000])
def test_noalloc_agrees(sd, n):
    import torch

    say(f"binned noalloc N={n}")
    m = W.random_molecule(8100 + n, n, 50, q1=0.9, extent=3.0 * n ** (1 / 3) + 2.0)
    ctx = sd.Context(0)
    a = sd.debye_profile_noalloc(*dev(m), m.q, ctx=ctx)
    b = sd.debye_profile(*dev(m), m.q, ctx=ctx)
    assert torch.equal(a, b)
    close(a.cpu().numpy(), oracle.profile(m.coords, m.types, m.table, m.q))


# half the sphere: rules with an odd and with an even number of nodes
@pytest.mark.parametrize("q1", [0.05, 0.11, 0.17, 0.23, 0.31])
def test_orientation_average_of_half_the_sphere(sd, q1):
    say(f"orientation average to q={q1}")
    m = W.random_molecule(8200, 400, 16, q1=q1, extent=26.0)
    r = float(np.linalg.norm(m.coords - m.coords.mean(axis=0, dtype=np.float64), axis=1).max())
    print("degree", sd.orient_degree(q1, r, 1e-9))
    I, averaged = sd.debye_profile_hybrid(*dev(m), m.q, tol=1e-9, mode="orient")
    assert averaged == 16
    close(I.cpu().numpy(), oracle.profile(m.coords, m.types, m.table, m.q))
