"""The 256 x 32 tiles of the fixed-point step by themselves (few replicas take
32 x 16 tiles): one step at the edges of its slabs and tiles, the calls that
move a context on or off it, graphs, and the exact-split form."""
import numpy as np
import pytest

import oracle
from paper_2305_07187_amd import instances

from gpu_common import QMAX, announce, ensure_built, oracle_schedules, rel_err, to_dev
from test_gpu_fixed_point import _bounds, _signed

pytestmark = pytest.mark.gpu
WIDE = "step_i8x4_256x32"


# n: three slabs and more, whole and with a remainder, whole and padded row tiles, N |J| at
# its limit; r: the last column tile with one, some and all of its columns
@pytest.mark.parametrize("n,r,jmax,scale", [
    (513, 1409, 1, 1.0), (514, 1377, 127, 1.0), (768, 961, 85, 1.0), (769, 961, 1, 1e-3), (1000, 1025, 65, 1.0),
    (2305, 321, 1, 1.0), (4097, 193, 2, 1e-30), (600, 1216, 1, 1e20)])
@pytest.mark.parametrize("wall", ["clamp", "inelastic"])
def test_one_step(n, r, jmax, scale, wall):
    import torch
    si = ensure_built()
    announce(f"fixed-point step, wide tiles N={n} R={r} |J|={jmax} scale {scale} {wall}")
    J = instances.make_pm1(n, n) * np.float32(jmax)
    x, p = _signed(n, r, 1, scale), _signed(n, r, 2, min(scale, 1.0))
    S, t = 50, 7
    m = si.SpringIsing(to_dev(J), to_dev(x), to_dev(p), total_steps=S, wall=wall)
    assert m.info()["kernel_name"].startswith(WIDE)
    m.set_state(to_dev(x), to_dev(p), t)
    m.step()
    xg, pg, _ = m.state()
    torch.cuda.synchronize()
    m.close()
    tail = list(range((r - 1) // 32 * 32 - 1, r))  # the last column tile and the column before it
    cols = sorted({0, 1, 31, 32, 33, r // 2, *tail})
    dts, zetas = oracle_schedules(S)
    J64, Q0, P0 = J.astype(np.float64), x[cols].T.astype(np.float64), p[cols].T.astype(np.float64)
    Q1, P1 = oracle.step(J64, Q0, P0, float(dts[t]), float(zetas[t]), qmax=QMAX, wall=wall)
    qb, pb = _bounds(J64, Q0, P0, J64 @ Q0, float(dts[t]), float(zetas[t]))
    dq, dp = np.abs(xg.cpu().numpy()[cols].T - Q1), np.abs(pg.cpu().numpy()[cols].T - P1)
    assert np.all(dq <= qb), (dq / qb).max()
    assert np.all(dp <= pb), (dp / pb).max()


def test_field_and_state_calls():
    # 30 steps with a field; a schedule replaced on the way, a state written
    # back, a split set and taken back: the digits follow the FP32 state
    import torch
    si = ensure_built()
    n, r, S = 700, 1001, 60
    announce(f"fixed-point trajectory, wide tiles N={n} R={r}")
    J, x0 = instances.make_pm1(n, 3), instances.make_x0(n, r, 3)
    h = instances.make_x0(1, n, 4)[:, 0].copy() * np.float32(5)
    dt, zeta = oracle_schedules(S)
    dt2 = (dt * np.linspace(1.0, 0.5, S)).astype(np.float32)
    m = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S)
    m.set_field(to_dev(h))
    m.run(10)
    m.set_schedule(to_dev(dt2), to_dev(zeta))
    m.run(5)
    x, p, t = m.state()
    m.set_state(x * 0, None, 0)
    m.set_state(x, p, t)
    m.run(5)
    assert m.info()["kernel_name"].startswith(WIDE)
    m.set_ksplit(1)
    assert m.info()["kernel_name"].startswith("step_f32")
    m.run(5)
    m.set_ksplit(0)
    assert m.info()["kernel_name"].startswith(WIDE)
    m.run(5)
    xg, pg, t = m.state()
    torch.cuda.synchronize()
    m.close()
    cols = [0, 31, 32, 500, 991, 992, 1000]
    ref = oracle.run(J.astype(np.float64), x0[cols].T.astype(np.float64), None,
                     np.concatenate([dt[:10], dt2[10:]]), zeta, qmax=QMAX, h=h.astype(np.float64), n_steps=30)
    assert t == 30
    assert rel_err(xg.cpu().numpy()[cols], ref["Q"]) <= 1e-5
    assert rel_err(pg.cpu().numpy()[cols], ref["P"]) <= 1e-5


@pytest.mark.parametrize("precision", ["fp32", "bf16x3_exactj"])
def test_graph_and_autotune(precision):
    # replays of a captured run equal direct launches bit for bit, also with
    # in-run energy checks; autotune leaves the state and the kernel in place
    import torch
    si = ensure_built()
    n, r, S = 1000, 705, 24
    announce(f"fixed-point graph and autotune, wide tiles N={n} R={r} {precision}")
    si.spring_ising_tile_cache_clear()
    J, x0 = to_dev(instances.make_pm1(n, 5)), to_dev(instances.make_x0(n, r, 5))
    a, b = (si.SpringIsing(J, x0, total_steps=S, precision=precision, energy_every=4) for _ in range(2))
    a.run(10)
    xa, pa, _ = a.state()
    ea = a.energy_trace()
    b.set_graph(5)
    for _ in range(3):
        b.set_state(x0, None, 0)
        b.run(10)
        b.energy()  # eager work between replays
        xb, pb, _ = b.state()
        torch.cuda.synchronize()
        assert torch.equal(xa, xb) and torch.equal(pa, pb) and torch.equal(ea, b.energy_trace())
    b.set_graph(0)
    tile, _ = b.autotune(12)
    si.spring_ising_tile_cache_clear()
    # (FP32 takes twice as long on every tile, the exact split a fifth longer)
    assert precision != "fp32" or tile == si.SI_TILE_FIXED_POINT
    assert a.info()["kernel_name"].startswith(WIDE)
    assert b.info()["kernel_name"].startswith(WIDE) == (tile == si.SI_TILE_FIXED_POINT)
    a.run(4)
    b.run(4)
    for u, v in zip(a.state()[:2], b.state()[:2]):
        if tile == si.SI_TILE_FIXED_POINT:
            assert torch.equal(u, v)
        else:
            assert float((u - v).abs().max()) <= 1e-5 * float(v.abs().max())
    a.close()
    b.close()


@pytest.mark.parametrize("n,r,jmax", [(1000, 705, 65), (1025, 650, 1), (2000, 385, 32)])
def test_exact_split_form(n, r, jmax):
    # one step to the same bound on the fixed point, and to that of the BF16
    # planes' FP32 sums when a call takes the context off it and back
    import torch
    si = ensure_built()
    announce(f"fixed-point step of bf16x3_exactj, wide tiles N={n} R={r} |J|={jmax}")
    J = instances.make_pm1(n, n) * np.float32(jmax)
    x, p = _signed(n, r, 1, 1.0), _signed(n, r, 2, 1.0)
    S = 20
    m = si.SpringIsing(to_dev(J), to_dev(x), to_dev(p), total_steps=S, precision="bf16x3_exactj")
    m.set_state(to_dev(x), to_dev(p), 3)
    dts, zetas = oracle_schedules(S)
    J64 = J.astype(np.float64)
    cols = [0, 1, 31, 32, r // 2, r - 2, r - 1]
    for ksplit in (0, 1, 0):
        m.set_ksplit(ksplit)
        assert m.info()["kernel_name"].startswith("step_bf16" if ksplit else WIDE)
        x0, p0, t = m.state()
        m.step()
        xg, pg, _ = m.state()
        torch.cuda.synchronize()
        Q0, P0 = (v.cpu().numpy()[cols].T.astype(np.float64) for v in (x0, p0))
        dt, zeta = float(dts[t]), float(zetas[t])
        Q1, P1 = oracle.step(J64, Q0, P0, dt, zeta, qmax=QMAX)
        qb, pb = _bounds(J64, Q0, P0, J64 @ Q0, dt, zeta)
        if ksplit:  # 3 n products added in FP32, in any order
            pb = pb + dt * zeta * 3 * n * 2.0 ** -24 * (np.abs(J64) @ np.abs(Q0))
        assert np.all(np.abs(xg.cpu().numpy()[cols].T - Q1) <= qb)
        assert np.all(np.abs(pg.cpu().numpy()[cols].T - P1) <= pb)
    m.close()
