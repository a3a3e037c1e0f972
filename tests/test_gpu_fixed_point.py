"""FP32 steps whose coupling product runs in fixed point on the int8 matrix
cores (integer couplings of complete graphs): at the edges of its tiles and
ranges, against the oracle, and the calls that move a context on or off it.

Tolerance of one step, from the arithmetic: the positions enter the product
with at most 2^-31 of the replica's largest |q| each (half a unit of the
lowest of four base-256 digits, top digit not full), F is rounded to FP32
twice (two 32-bit halves, one fused multiply-add), and the update itself is
three FP32 operations of results up to |P| + D z |F| + D k |q|.
"""
import numpy as np
import pytest

import oracle
from paper_2305_07187_amd import instances

from gpu_common import QMAX, announce, ensure_built, oracle_schedules, rel_err, to_dev

pytestmark = pytest.mark.gpu
NAME = "step_i8x4"


def _bounds(J64, Q, P, F, dt, zeta):
    u = 2.0 ** -24
    f_err = 2.0 ** -31 * np.abs(Q).max(axis=0) * np.abs(J64).sum(axis=1)[:, None] + 3 * u * np.abs(F)
    p_err = dt * zeta * f_err + 4 * u * (np.abs(P) + dt * (zeta * np.abs(F) + 0.5 * np.abs(Q)))
    q_err = 3 * u * (np.abs(Q) + dt * np.abs(P))
    return q_err + 1e-45, p_err + 1e-45


def _signed(n, r, seed, scale):
    return instances.random_state(n, r, seed, scale=1.4) * np.float32(scale)


# n around the 256-deep slabs and 256-row tiles, r around the 32-replica tiles,
# N |J| up to its limit of 65281 (514 x 127, 768 x 85); positions of every magnitude
@pytest.mark.parametrize("n,r,jmax,scale", [
    (513, 256, 1, 1.0), (514, 257, 127, 1.0), (768, 256, 85, 1.0), (769, 300, 1, 1e-3), (1000, 1025, 1, 1.0),
    (2000, 1024, 1, 1.0), (2305, 65, 1, 1.0), (4097, 3, 2, 1e-30), (600, 288, 1, 1e20)])
@pytest.mark.parametrize("wall", ["clamp", "inelastic"])
def test_one_step_at_tile_edges(n, r, jmax, scale, wall):
    import torch
    si = ensure_built()
    announce(f"fixed-point step N={n} R={r} |J|={jmax} scale {scale} {wall}")
    J = instances.make_pm1(n, n) * np.float32(jmax)
    x, p = _signed(n, r, 1, scale), _signed(n, r, 2, min(scale, 1.0))
    S, t = 50, 7
    m = si.SpringIsing(to_dev(J), to_dev(x), to_dev(p), total_steps=S, wall=wall)
    assert m.info()["kernel_name"].startswith(NAME)
    m.set_state(to_dev(x), to_dev(p), t)
    m.step()
    xg, pg, _ = m.state()
    torch.cuda.synchronize()
    m.close()
    cols = sorted({0, 1, 2, 31, 32, r // 2, r - 2, r - 1} & set(range(r)))
    dts, zetas = oracle_schedules(S)
    dt, zeta = float(dts[t]), float(zetas[t])
    J64 = J.astype(np.float64)
    Q0, P0 = x[cols].T.astype(np.float64), p[cols].T.astype(np.float64)
    Q1, P1 = oracle.step(J64, Q0, P0, dt, zeta, qmax=QMAX, wall=wall)
    qb, pb = _bounds(J64, Q0, P0, J64 @ Q0, dt, zeta)
    dq = np.abs(xg.cpu().numpy()[cols].T - Q1)
    dp = np.abs(pg.cpu().numpy()[cols].T - P1)
    assert np.all(dq <= qb), (dq / qb).max()
    assert np.all(dp <= pb), (dp / pb).max()


def test_trajectory_field_and_state_calls():
    # 30 steps with a field; a schedule replaced on the way, a state written
    # back, a split set and taken back: the digits follow the FP32 state.
    import torch
    si = ensure_built()
    n, r, S = 700, 320, 60
    announce(f"fixed-point trajectory N={n} R={r}")
    J = instances.make_pm1(n, 3)
    x0 = instances.make_x0(n, r, 3)
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
    assert m.info()["kernel_name"].startswith(NAME)
    m.set_ksplit(1)
    assert not m.info()["kernel_name"].startswith(NAME)
    m.run(5)
    m.set_ksplit(0)
    assert m.info()["kernel_name"].startswith(NAME)
    m.run(5)
    xg, pg, t = m.state()
    torch.cuda.synchronize()
    m.close()
    cols = [0, 31, 32, 200, 319]
    ref = oracle.run(J.astype(np.float64), x0[cols].T.astype(np.float64), None,
                     np.concatenate([dt[:10], dt2[10:]]), zeta, qmax=QMAX,
                     h=h.astype(np.float64), n_steps=30)
    assert t == 30
    assert rel_err(xg.cpu().numpy()[cols], ref["Q"]) <= 1e-5
    assert rel_err(pg.cpu().numpy()[cols], ref["P"]) <= 1e-5


def test_graph_adjoint_and_autotune():
    # replays of a captured run equal direct launches bit for bit; the state
    # an adjoint or an autotune call leaves behind is stepped from correctly
    import torch
    si = ensure_built()
    n, r, S = 520, 300, 24
    announce(f"fixed-point graph, adjoint, autotune N={n} R={r}")
    J, x0 = to_dev(instances.make_pm1(n, 5)), to_dev(instances.make_x0(n, r, 5))

    def fresh():
        m = si.SpringIsing(J, x0, total_steps=S)
        assert m.info()["kernel_name"].startswith(NAME)
        return m
    a, b = fresh(), fresh()
    a.run(10)
    xa, pa, _ = a.state()
    b.set_graph(5)
    for _ in range(3):
        b.set_state(x0, None, 0)
        b.run(10)
        b.energy()  # eager work between replays
        xb, pb, _ = b.state()
        torch.cuda.synchronize()
        assert torch.equal(xa, xb) and torch.equal(pa, pb)
    a.run(4)
    xa, pa, _ = a.state()
    b.set_graph(0)
    b.autotune(3)
    b.set_ksplit(0)
    b.run(4)
    xb, pb, _ = b.state()
    torch.cuda.synchronize()
    if b.info()["kernel_name"].startswith(NAME):
        assert torch.equal(xa, xb) and torch.equal(pa, pb)
    si.spring_ising_tile_cache_clear()
    # the adjoint's forward half ends where a run on the same kernels ends,
    # and a rewound run after it equals one before it
    c = fresh()
    c.relaxed_energy_forward(8)
    c.set_state(x0, None, 0)
    c.run(14)
    xc, pc, _ = c.state()
    torch.cuda.synchronize()
    assert torch.equal(xa, xc) and torch.equal(pa, pc)
    for m in (a, b, c):
        m.close()


def test_non_finite_and_zero_replicas():
    # positions given by the caller may be infinite, NaN or all zero: one step
    # gives what the FP32 matrix cores' tile gives
    import torch
    si = ensure_built()
    n, r = 530, 260
    announce("fixed-point step with infinite, NaN and zero replicas")
    J = to_dev(instances.make_pm1(n, 6))
    x = instances.random_state(n, r, 7, scale=1.4)
    x[1, 5] = np.inf
    x[2, 6], x[2, 7] = np.inf, -np.inf
    x[3, 8] = np.nan
    x[4, :] = 0.0
    x[5, :] = 0.0
    x[5, 9] = -1.25
    x[259, 529] = -np.inf
    out = []
    for tile in (0, 14):
        m = si.SpringIsing(J, to_dev(x), total_steps=4, tile=tile)
        assert m.info()["kernel_name"].startswith(NAME) == (tile == 0)
        m.run(1)
        xs, ps, _ = m.state()
        m.run(3)
        xe, pe, _ = m.state()
        torch.cuda.synchronize()
        assert torch.isfinite(xe).all() and torch.isfinite(pe).all()
        out.append((xs.cpu().numpy(), ps.cpu().numpy()))
        m.close()
    rows = [1, 2, 3, 4, 5, 259]
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1][rows], out[1][1][rows])


def test_route():
    # taken for integer couplings of complete graphs in the paper order with an
    # automatic tile, and for nothing else
    si = ensure_built()
    n, r = 600, 256
    J = instances.make_pm1(n, 8)
    x = to_dev(instances.make_x0(n, r, 8))
    hole = J.copy()
    hole[3, 4] = hole[4, 3] = 0.0
    real = J.copy()
    real[3, 4] = real[4, 3] = 0.5
    cases = [(J, {}, True), (hole, {}, False), (real, {}, False), (J * 108, {}, True), (J * 109, {}, False),
             (J * 128, {}, False), (J, {"order": "symplectic"}, False), (J, {"tile": 14}, False),
             (J[:383, :383].copy(), {}, False)]
    for Jc, kw, want in cases:
        m = si.SpringIsing(to_dev(Jc), x[:, :Jc.shape[0]].contiguous(), total_steps=2, **kw)
        assert m.info()["kernel_name"].startswith(NAME) == want, (kw, Jc.shape)
        m.run(2)
        m.close()


@pytest.mark.parametrize("n,r,jmax", [(1000, 1, 1), (1000, 33, 65), (1025, 256, 1), (2000, 64, 32)])
def test_exact_split_form(n, r, jmax):
    # the BF16 matrix cores' exact form takes the same products: one step to
    # the same bound, and the BF16 planes follow when a call takes it off them
    import torch
    si = ensure_built()
    announce(f"fixed-point step of bf16x3_exactj N={n} R={r} |J|={jmax}")
    J = instances.make_pm1(n, n) * np.float32(jmax)
    x, p = _signed(n, r, 1, 1.0), _signed(n, r, 2, 1.0)
    S = 20
    m = si.SpringIsing(to_dev(J), to_dev(x), to_dev(p), total_steps=S, precision="bf16x3_exactj")
    assert m.info()["kernel_name"].startswith(NAME)
    m.set_state(to_dev(x), to_dev(p), 3)
    dts, zetas = oracle_schedules(S)
    J64 = J.astype(np.float64)

    def check_step(fp32_sum):
        x0, p0, t = m.state()
        torch.cuda.synchronize()
        m.step()
        xg, pg, _ = m.state()
        torch.cuda.synchronize()
        Q0, P0 = x0.cpu().numpy().T.astype(np.float64), p0.cpu().numpy().T.astype(np.float64)
        dt, zeta = float(dts[t]), float(zetas[t])
        Q1, P1 = oracle.step(J64, Q0, P0, dt, zeta, qmax=QMAX)
        qb, pb = _bounds(J64, Q0, P0, J64 @ Q0, dt, zeta)
        if fp32_sum:  # 3 n products added in FP32, in any order
            pb = pb + dt * zeta * 3 * n * 2.0 ** -24 * (np.abs(J64) @ np.abs(Q0))
        assert np.all(np.abs(xg.cpu().numpy().T - Q1) <= qb)
        assert np.all(np.abs(pg.cpu().numpy().T - P1) <= pb)

    check_step(False)
    m.set_ksplit(1)  # off the fixed point, and back, also through autotune
    assert not m.info()["kernel_name"].startswith(NAME)
    check_step(True)
    m.set_ksplit(0)
    assert m.info()["kernel_name"].startswith(NAME)
    check_step(False)
    m.autotune(2)
    check_step(not m.info()["kernel_name"].startswith(NAME))
    m.close()
    si.spring_ising_tile_cache_clear()
    f = si.SpringIsing(to_dev(instances.make_pm1(383, 1)), to_dev(instances.make_x0(383, r, 1)),
                       total_steps=2, precision="bf16x3_exactj")
    assert not f.info()["kernel_name"].startswith(NAME)
    f.close()


# Real couplings: four digits each, scaled per row (half a unit: 2^-31 of the
# row's largest); of the sixteen digit products the six lowest are left out,
# together below 3.2 x 2^16 x 2^14 units, a unit being at most 2^-60 of the
# product of the row's and the replica's largest.
REAL = "step_i8x10"


def _real_bounds(J64, Q, P, F, dt, zeta):
    u = 2.0 ** -24
    jm, qm = np.abs(J64).max(axis=1)[:, None], np.abs(Q).max(axis=0)
    f_err = (2.0 ** -31 * (qm * np.abs(J64).sum(axis=1)[:, None] + jm * np.abs(Q).sum(axis=0)) +
             3.2 * 2.0 ** -30 * J64.shape[0] * jm * qm + 4 * u * np.abs(F))
    p_err = dt * zeta * f_err + 4 * u * (np.abs(P) + dt * (zeta * np.abs(F) + 0.5 * np.abs(Q)))
    return 3 * u * (np.abs(Q) + dt * np.abs(P)) + 1e-45, p_err + 1e-45


def _real(n, seed, kind="gauss"):
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((n, n)) if kind == "gauss" else rng.uniform(1, 3, (n, n)) * 0.01
    a = np.triu(a, 1).astype(np.float32)
    return a + a.T


# n around the 128-deep slabs and 128-row tiles, r around the 64-replica tiles,
# one and several tiles per workgroup, positions and couplings of any magnitude
@pytest.mark.parametrize("n,r,kind,scale,wall", [
    (513, 1280, "gauss", 1.0, "clamp"), (640, 1001, "gauss", 1e-3, "inelastic"),
    (1000, 641, "uniform", 1.0, "clamp"), (1025, 640, "gauss", 1e20, "clamp"),
    (2305, 300, "gauss", 1e-30, "clamp"), (2000, 1025, "gauss", 1.0, "inelastic"),
    (10001, 40, "gauss", 1.0, "clamp")])
def test_real_one_step_at_tile_edges(n, r, kind, scale, wall):
    import torch
    si = ensure_built()
    announce(f"fixed-point step, real couplings N={n} R={r} {kind} scale {scale} {wall}")
    J = _real(n, n, kind)
    x, p = _signed(n, r, 1, scale), _signed(n, r, 2, min(scale, 1.0))
    S, t = 50, 7
    m = si.SpringIsing(to_dev(J), to_dev(x), to_dev(p), total_steps=S, wall=wall)
    assert m.info()["kernel_name"].startswith(REAL)
    m.set_state(to_dev(x), to_dev(p), t)
    m.step()
    xg, pg, _ = m.state()
    torch.cuda.synchronize()
    m.close()
    cols = sorted({0, 1, 31, 32, 33, r // 2, r - 2, r - 1} & set(range(r)))
    dts, zetas = oracle_schedules(S)
    dt, zeta = float(dts[t]), float(zetas[t])
    J64 = J.astype(np.float64)
    Q0, P0 = x[cols].T.astype(np.float64), p[cols].T.astype(np.float64)
    Q1, P1 = oracle.step(J64, Q0, P0, dt, zeta, qmax=QMAX, wall=wall)
    qb, pb = _real_bounds(J64, Q0, P0, J64 @ Q0, dt, zeta)
    dq = np.abs(xg.cpu().numpy()[cols].T - Q1)
    dp = np.abs(pg.cpu().numpy()[cols].T - P1)
    assert np.all(dq <= qb), (dq / qb).max()
    assert np.all(dp <= pb), (dp / pb).max()


def test_real_trajectory_resident_and_infinite():
    # a run with a field against the oracle; the resident form bit for bit;
    # infinite and NaN positions step as on the FP32 matrix cores
    import torch
    si = ensure_built()
    n, r, S = 1000, 1000, 40
    announce(f"fixed-point, real couplings: trajectory, resident, infinite N={n} R={r}")
    J, x0 = _real(n, 3), instances.make_x0(n, r, 3)
    h = instances.make_x0(1, n, 4)[:, 0].copy() * np.float32(5)
    out = []
    for resident in (0, 2):
        m = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S)
        m.set_field(to_dev(h))
        m.set_resident(resident)
        m.run(20)
        assert m.info()["kernel_name"].startswith(REAL) and m.info()["resident_groups"] == 128
        out.append(m.state())
        torch.cuda.synchronize()
        m.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    cols = [0, 31, 32, 63, 64, 999]
    dt, zeta = oracle_schedules(S)
    ref = oracle.run(J.astype(np.float64), x0[cols].T.astype(np.float64), None, dt, zeta,
                     qmax=QMAX, h=h.astype(np.float64), n_steps=20)
    assert rel_err(out[0][0].cpu().numpy()[cols], ref["Q"]) <= 1e-5
    assert rel_err(out[0][1].cpu().numpy()[cols], ref["P"]) <= 1e-5
    x = instances.random_state(n, r, 7, scale=1.4)
    x[1, 5], x[2, 6], x[2, 7], x[40, 8] = np.inf, np.inf, -np.inf, np.nan
    x[4, :] = 0.0
    x[999, 999] = -np.inf
    res = []
    for tile in (0, 14):
        m = si.SpringIsing(to_dev(J), to_dev(x), total_steps=4, tile=tile)
        assert m.info()["kernel_name"].startswith(REAL) == (tile == 0)
        m.run(1)
        xs, ps, _ = m.state()
        torch.cuda.synchronize()
        res.append((xs.cpu().numpy(), ps.cpu().numpy()))
        m.close()
    rows = [1, 2, 4, 40, 999]
    np.testing.assert_array_equal(res[0][0], res[1][0])
    np.testing.assert_array_equal(res[0][1][rows], res[1][1][rows])


def test_real_route():
    # dense rows of like couplings only, in FP32, with enough work
    si = ensure_built()
    n, r = 640, 1000
    J = _real(n, 8)
    x = to_dev(instances.make_x0(n, r, 8))
    heavy, thin, few = J.copy(), J.copy(), J.copy()
    heavy[3, 4] = heavy[4, 3] = 900.0        # most of the row below 1/1024 of it
    thin[3, :41] = thin[:41, 3] = 0.0        # more than a sixteenth of row 3
    few[3, :20] = few[:20, 3] = 0.0
    cases = [(J, r, {}, True), (heavy, r, {}, False), (thin, r, {}, False), (few, r, {}, True),
             (instances.make_pm1(n, 8) * np.float32(127), r, {}, True),  # N |J| beyond the integer form
             (J, 960, {}, False), (J, r, {"precision": "bf16x_hiloj"}, False),
             (J, r, {"order": "symplectic"}, False), (J, r, {"tile": 14}, False)]
    for k, (Jc, rc, kw, want) in enumerate(cases):
        m = si.SpringIsing(to_dev(Jc), x[:rc].contiguous(), total_steps=2, **kw)
        assert m.info()["kernel_name"].startswith(REAL) == want, (k, kw)
        m.run(2)
        m.close()


# 32 x 16 tiles: 32-row blocks and 64-deep steps of n (a wave without any), 16
# columns of r, four and eight waves, one and several rounds of steps ahead
@pytest.mark.parametrize("n,r,jmax,wall", [(384, 257, 1, "clamp"), (513, 65, 127, "inelastic"), (545, 100, 1, "clamp"),
                                           (1025, 81, 1, "inelastic"), (1999, 97, 32, "clamp"), (2000, 300, 1, "clamp"),
                                           (4097, 3, 2, "clamp")])
def test_few_replica_tiles(n, r, jmax, wall):
    # one step to the same bound, and ten equal the wide tiles' bit for bit
    import torch
    si = ensure_built()
    announce(f"fixed-point step, few replicas N={n} R={r} |J|={jmax} {wall}")
    J = instances.make_pm1(n, n) * np.float32(jmax)
    wide = max(r, 700000 // n + 64)  # beyond the rule: 256 x 32 tiles
    x, p = _signed(n, wide, 1, 1.0), _signed(n, wide, 2, 1.0)
    h = to_dev(instances.make_x0(n, 1, 5, scale=2.0)[0])
    S, t = 50, 7
    out, names = [], []
    for rr in (r, wide):
        xr, pr = to_dev(x[:rr].copy()), to_dev(p[:rr].copy())
        m = si.SpringIsing(to_dev(J), xr, pr, total_steps=S, wall=wall)
        names.append(m.info()["kernel_name"])
        m.set_state(xr, pr, t)
        m.step()
        xg, pg, _ = m.state()
        m.set_field(h)
        m.run(9)
        xe, pe, _ = m.state()
        torch.cuda.synchronize()
        out.append([v.cpu().numpy()[:r] for v in (xg, pg, xe, pe)])
        m.close()
    assert names[0].startswith(NAME + "_32x16")
    if n > 512:
        assert names[1].startswith(NAME + "_256x32")
        for a, b in zip(*out):
            assert np.array_equal(a, b)
    dts, zetas = oracle_schedules(S)
    cols = sorted({0, 1, 15, 16, r - 1} & set(range(r)))
    J64, Q0, P0 = J.astype(np.float64), x[cols].T.astype(np.float64), p[cols].T.astype(np.float64)
    Q1, P1 = oracle.step(J64, Q0, P0, float(dts[t]), float(zetas[t]), qmax=QMAX, wall=wall)
    qb, pb = _bounds(J64, Q0, P0, J64 @ Q0, float(dts[t]), float(zetas[t]))
    assert np.all(np.abs(out[0][0][cols].T - Q1) <= qb) and np.all(np.abs(out[0][1][cols].T - P1) <= pb)
