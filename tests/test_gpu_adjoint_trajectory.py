"""The gradient's forward half takes the trajectory of run() at every size: it
ends in the same state bit for bit, however the schedule is cut into segments,
and the sweep's loss and gradient belong to that trajectory."""
import numpy as np
import pytest

import oracle
from paper_2305_07187_amd import instances

from gpu_common import QMAX, announce, ensure_built, oracle_schedules, to_dev

pytestmark = pytest.mark.gpu


def _couplings(n, kind):
    return instances.make_pm1(n, n) if kind == "pm1" else instances.make_gauss(n, n).astype(np.float32)


# FP32 steps (small, split, one launch), 32 x 16, 256 x 32 and real fixed-point tiles
@pytest.mark.parametrize("kind,n,r,name", [
    ("pm1", 200, 65, "step_f32"), ("gauss", 600, 70, "step_f32"), ("pm1", 2000, 96, "step_i8x4_32x16"),
    ("pm1", 520, 300, "step_i8x4_32x16"), ("pm1", 4100, 40, "step_i8x4_32x16"), ("pm1", 700, 1001, "step_i8x4_256x32"),
    ("pm1", 2305, 321, "step_i8x4_256x32"), ("gauss", 1000, 641, "step_i8x10")])
def test_ends_as_run(kind, n, r, name):
    import torch
    si = ensure_built()
    S = 18
    announce(f"adjoint trajectory N={n} R={r} {kind}")
    J, x0 = _couplings(n, kind), instances.make_x0(n, r, 9)
    Jd, xd = to_dev(J), to_dev(x0)
    m = si.SpringIsing(Jd, xd, total_steps=S)
    assert m.info()["kernel_name"].startswith(name)
    m.run(S)
    xr, pr, _ = m.state()
    out = []
    for every, t0 in ((7, 0), (18, 0), (5, 3)):  # a recorded last segment of 4, of all, of 5 after 3 steps
        m.set_state(xd, None, 0)
        m.run(t0)
        loss = m.relaxed_energy_forward(every)
        x, p, t = m.state()
        gd, gz = m.relaxed_energy_backward()
        torch.cuda.synchronize()
        assert t == S and torch.equal(x, xr) and torch.equal(p, pr), (every, t0)
        out.append([v.cpu().numpy() for v in (loss, gd, gz)])
    for a, b in zip(out[0], out[1]):
        assert np.array_equal(a, b)
    assert np.array_equal(out[0][0], out[2][0])
    assert np.array_equal(out[0][1][3:], out[2][1][3:]) and np.array_equal(out[0][2][3:], out[2][2][3:])
    # the rewound context runs on as before
    m.set_state(xd, None, 0)
    m.run(S)
    x, p, _ = m.state()
    torch.cuda.synchronize()
    assert torch.equal(x, xr) and torch.equal(p, pr)
    m.close()
    e = si.SpringIsing(Jd, xd, total_steps=S, energy_every=5)
    loss = e.relaxed_energy_forward(7)
    gd, gz = e.relaxed_energy_backward()
    torch.cuda.synchronize()
    for a, b in zip(out[0], (loss, gd, gz)):
        assert np.array_equal(a, b.cpu().numpy())
    e.close()
    # 1e-5 and 1e-4 of the largest entry: the FP32 multipliers' bounds of the
    # adjoint's other tests
    dt, zeta = oracle_schedules(S)
    Lo, gdo, gzo = oracle.relaxed_energy_grad(J.astype(np.float64), x0.T.astype(np.float64), None,
                                              dt.astype(np.float64), zeta.astype(np.float64), qmax=QMAX)
    rel = lambda a, b: float(np.abs(a - b).max() / np.abs(b).max())
    assert abs(float(out[0][0][0]) - Lo) <= 1e-5 * abs(Lo)
    assert rel(out[0][1], gdo) <= 1e-4 and rel(out[0][2], gzo) <= 1e-4


@pytest.mark.parametrize("kind,n,r", [("pm1", 600, 100), ("pm1", 520, 1408), ("gauss", 700, 961)])
def test_walls_and_uneven_replicas(kind, n, r):
    # a start with many positions and momenta at their walls, one replica in
    # three uneven: the same state as run(), and the gradient of the segments
    # recorded by either half
    import torch
    si = ensure_built()
    S = 6
    announce(f"adjoint trajectory from walls and uneven replicas N={n} R={r} {kind}")
    J = to_dev(_couplings(n, kind))
    x, p = instances.random_state(n, r, 1, scale=3.0), instances.random_state(n, r, 2, scale=4.0)
    x, p = np.clip(x, -QMAX, QMAX).astype(np.float32), np.clip(p, -2, 2).astype(np.float32)
    x[1::3] *= np.float32(1e-6)
    p[1::3] = 0.0
    x[1::3, 5] = 1.25
    m = si.SpringIsing(J, to_dev(x), to_dev(p), total_steps=S)
    m.run(S)
    xr, pr, _ = m.state()
    out = []
    for every in (1, 2, 6):
        m.set_state(to_dev(x), to_dev(p), 0)
        loss = m.relaxed_energy_forward(every)
        xo, po, _ = m.state()
        gd, gz = m.relaxed_energy_backward()
        torch.cuda.synchronize()
        assert torch.equal(xo, xr) and torch.equal(po, pr), every
        out.append([v.cpu().numpy() for v in (loss, gd, gz)])
    m.close()
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)
    loss, gd, gz = out[0]
    dt, zeta = oracle_schedules(S)
    Lo, gdo, gzo = oracle.relaxed_energy_grad(J.cpu().numpy().astype(np.float64), x.T.astype(np.float64),
                                              p.T.astype(np.float64), dt.astype(np.float64),
                                              zeta.astype(np.float64), qmax=QMAX)
    rel = lambda a, b: float(np.abs(a - b).max() / np.abs(b).max())
    assert abs(float(loss[0]) - Lo) <= 1e-5 * abs(Lo)
    assert rel(gd, gdo) <= 1e-4 and rel(gz, gzo) <= 1e-4
