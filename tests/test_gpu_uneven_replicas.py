"""Fixed-point steps from states in which a few positions tower over the rest.

A row that does not contain the large positions (their own row; in real
couplings also one uncoupled to them) sums small positions only.  FP32 sums n
such products to n 2^-24 of their magnitudes, in any order; held relative to
the replica's largest position, 2^-31 of that is more than they are.
"""
import numpy as np
import pytest

import oracle
from paper_2305_07187_amd import instances

from gpu_common import QMAX, announce, ensure_built, oracle_schedules, to_dev

pytestmark = pytest.mark.gpu
WIDE, FEW, REAL = "step_i8x4_256x32", "step_i8x4_32x16", "step_i8x10"


def _state(n, r):
    """Replicas 0, 3, ..: even; the others: one or five positions of about 1.4
    among ones below 1e-9.  Returns x and the large positions' spins."""
    x = instances.random_state(n, r, 1, scale=1.4)
    big = [[(7 * c) % n] if c % 3 == 1 else [(11 * c + 3 * k) % n for k in range(5)] for c in range(r)]
    for c in range(r):
        if c % 3:
            keep = x[c, big[c]].copy()
            x[c] *= np.float32(1e-9)
            x[c, big[c]] = np.where(keep < 0, -1, 1) * np.float32(1.4)
    return x, big


def _couplings(n, kind):
    if kind == "pm1":
        return instances.make_pm1(n, n)
    J = instances.make_gauss(n, n).astype(np.float32)
    rng = np.random.default_rng(n)  # 3 % zeros
    hole = np.triu(rng.uniform(size=(n, n)) < 0.03, 1)
    J[hole | hole.T] = 0.0
    return J


def _err_bounds(J64, Q, P, dt, zeta, k):
    u, n = 2.0 ** -24, J64.shape[0]
    F = J64 @ Q
    f_err = (n + 4) * u * (np.abs(J64) @ np.abs(Q))
    p_err = dt * zeta * f_err + 4 * u * (np.abs(P) + dt * (zeta * np.abs(F) + k * np.abs(Q)))
    return 3 * u * (np.abs(Q) + dt * np.abs(P)) + 1e-45, p_err + 1e-45


# n at and off the row tiles, with and without an incomplete last slab; every column tile's last columns
@pytest.mark.parametrize("kind,n,r,k,name", [
    ("pm1", 513, 1409, 0.0, WIDE), ("pm1", 768, 961, 0.5, WIDE), ("pm1", 600, 257, 0.0, FEW),
    ("pm1", 1100, 97, 0.0, FEW), ("real", 1000, 641, 0.5, REAL), ("real", 640, 1001, 0.0, REAL)])
@pytest.mark.parametrize("wall", ["clamp", "inelastic"])
def test_one_step(kind, n, r, k, name, wall):
    import torch
    si = ensure_built()
    announce(f"uneven replicas N={n} R={r} {kind} k={k} {wall}")
    J = _couplings(n, kind)
    x, _ = _state(n, r)
    h = to_dev(instances.make_x0(n, 1, 5, scale=1e-9)[0])
    S, t = 50, 7
    m = si.SpringIsing(to_dev(J), to_dev(x), None, total_steps=S, wall=wall, k=k)
    assert m.info()["kernel_name"].startswith(name)
    m.set_field(h)
    m.set_state(to_dev(x), None, t)
    m.step()
    xg, pg, _ = m.state()
    torch.cuda.synchronize()
    m.close()
    cols = sorted({0, 1, 2, 3, 15, 16, 17, 31, 32, 33, 64, r // 2, r - 3, r - 2, r - 1} & set(range(r)))
    dts, zetas = oracle_schedules(S)
    dt, zeta = float(dts[t]), float(zetas[t])
    J64, Q0 = J.astype(np.float64), x[cols].T.astype(np.float64)
    P0, h64 = np.zeros_like(Q0), h.cpu().numpy().astype(np.float64)
    Q1, P1 = oracle.step(J64, Q0, P0, dt, zeta, k=k, qmax=QMAX, wall=wall, h=h64)
    qb, pb = _err_bounds(J64, Q0, P0, dt, zeta, k)
    pb = pb + 4 * 2.0 ** -24 * dt * zeta * np.abs(h64)[:, None]
    dq, dp = np.abs(xg.cpu().numpy()[cols].T - Q1), np.abs(pg.cpu().numpy()[cols].T - P1)
    assert np.all(dq <= qb), (dq / qb).max()
    assert np.all(dp <= pb), (dp / pb).max()


@pytest.mark.parametrize("kind,n,r,name,resident", [
    ("pm1", 520, 1408, WIDE, False), ("pm1", 2000, 1024, WIDE, True), ("pm1", 1100, 97, FEW, False),
    ("real", 1000, 1000, REAL, True)])
def test_neighbours_and_resident(kind, n, r, name, resident):
    # an even replica's steps do not depend on uneven ones beside it; the
    # resident form repeats the steps bit for bit; and where the positions
    # even out on the way (the oracle's do), the trajectory follows
    import torch
    si = ensure_built()
    announce(f"uneven replicas beside even ones N={n} R={r} {kind}")
    J = _couplings(n, kind)
    x, _ = _state(n, r)
    even = instances.random_state(n, r, 1, scale=1.4)
    S, steps = 50, 12
    m = si.SpringIsing(to_dev(J), to_dev(x), None, total_steps=S)
    assert m.info()["kernel_name"].startswith(name)
    out = []
    for start, res in ((x, 0), (even, 0)) + (((x, 2),) if resident else ()):
        m.set_resident(res)
        assert not res or m.info()["resident_groups"] > 0
        m.set_state(to_dev(start), None, 0)
        m.run(steps)
        xo, po, _ = m.state()
        torch.cuda.synchronize()
        out.append((xo.cpu().numpy(), po.cpu().numpy()))
    m.close()
    for a, b in zip(out[0], out[1]):
        assert np.array_equal(a[::3], b[::3])
    for other in out[2:]:
        assert np.array_equal(out[0][0], other[0]) and np.array_equal(out[0][1], other[1])
    cols = [0, 1, 2, r - 1]
    dt, zeta = oracle_schedules(S)
    ref = oracle.run(J.astype(np.float64), x[cols].T.astype(np.float64), None, dt, zeta, qmax=QMAX, n_steps=steps)
    for got, want in zip(out[0], (ref["Q"], ref["P"])):
        for c in range(len(cols)):  # each replica by its own largest
            err = np.abs(got[cols[c]] - want[:, c]).max() / np.abs(want[:, c]).max()
            assert err <= 1e-5, (cols[c], err)


@pytest.mark.parametrize("kind,n,r,name", [("pm1", 530, 1345, WIDE), ("pm1", 530, 260, FEW), ("real", 700, 961, REAL)])
def test_non_finite_and_zero(kind, n, r, name):
    # infinite, NaN and zero replicas step as on the FP32 matrix cores, and the
    # replicas beside them are not touched
    import torch
    si = ensure_built()
    announce(f"infinite, NaN and zero replicas N={n} R={r} {kind}")
    J = to_dev(instances.make_J(n, "pm1" if kind == "pm1" else "gauss", 6))
    x = instances.random_state(n, r, 7, scale=1.4)
    clean = x.copy()
    x[1, 5], x[2, 6], x[2, 7], x[3, 8] = np.inf, np.inf, -np.inf, np.nan
    x[4, :] = 0.0
    x[5, :] = 0.0
    x[5, 9] = -1.25
    x[r - 1, n - 1] = -np.inf
    odd = [1, 2, 3, 4, 5, r - 1]
    out = []
    for start, tile in ((x, 0), (x, 14), (clean, 0)):
        m = si.SpringIsing(J, to_dev(start), total_steps=6, tile=tile)
        assert m.info()["kernel_name"].startswith(name) == (tile == 0)
        m.run(1)
        xs, ps, _ = m.state()
        m.run(4)
        xe, pe, _ = m.state()
        torch.cuda.synchronize()
        assert torch.isfinite(xe).all() and torch.isfinite(pe).all()
        out.append([v.cpu().numpy() for v in (xs, ps, xe, pe)])
        m.close()
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1][odd], out[1][1][odd])
    rest = np.setdiff1d(np.arange(r), odd)
    for a, b in zip(out[0], out[2]):
        np.testing.assert_array_equal(a[rest], b[rest])
