"""Without free device memory the fixed-point form's buffers are given back
before a call fails: the call succeeds and the context goes on with the tile
that stands by."""
import numpy as np
import pytest

import oracle
from paper_2305_07187_amd import instances

from gpu_common import QMAX, announce, ensure_built, oracle_schedules, rel_err, to_dev

pytestmark = pytest.mark.gpu
# reserve() and the first buffer's own allocation fail, then there is room
ADJOINT_FAILS = 2


def _check_state(m, J, x0, S, steps):
    import torch
    x, p, t = m.state()
    torch.cuda.synchronize()
    assert t == steps
    dt, zeta = oracle_schedules(S)
    cols = [0, 1, x0.shape[0] - 1]
    ref = oracle.run(J.astype(np.float64), x0[cols].T.astype(np.float64), None, dt, zeta, qmax=QMAX, n_steps=steps)
    assert rel_err(x.cpu().numpy()[cols], ref["Q"]) <= 1e-5
    assert rel_err(p.cpu().numpy()[cols], ref["P"]) <= 1e-5


@pytest.mark.parametrize("n,r,precision", [(600, 300, "fp32"), (1000, 705, "fp32"), (1000, 33, "bf16x3_exactj"),
                                           (1000, 705, "bf16x3_exactj")])
def test_best_state(n, r, precision):
    si = ensure_built()
    announce(f"memory released for the best state N={n} R={r} {precision}")
    S = 40
    J, x0 = instances.make_pm1(n, 5), instances.make_x0(n, r, 5)
    m = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S, precision=precision)
    assert m.info()["kernel_name"].startswith("step_i8")
    before = m.info()["device_bytes"]
    m.set_graph(4)
    m.run(5)
    si.spring_ising_debug_fail_allocs(m.ctx, 1)
    m.update_best()
    assert not m.info()["kernel_name"].startswith("step_i8") and m.info()["tile"] < 64
    assert m.info()["device_bytes"] < before
    m.run(5)
    _check_state(m, J, x0, S, 10)
    m.set_state(to_dev(x0), None, 0)
    m.run(5)  # captured anew
    m.run(7)
    _check_state(m, J, x0, S, 12)
    # nothing left to give back
    si.spring_ising_debug_fail_allocs(m.ctx, 1)
    with pytest.raises(si.SpringIsingError) as e:
        m.set_field(to_dev(x0[0]))
    assert e.value.status == si.SI_ERR_OOM
    m.close()


@pytest.mark.parametrize("n,r", [(600, 300), (1000, 705)])
def test_gradient_and_resident(n, r):
    import torch
    si = ensure_built()
    announce(f"memory released for the gradient, a resident run and autotune N={n} R={r}")
    S = 12
    J, x0 = instances.make_pm1(n, 5), instances.make_x0(n, r, 5)
    m = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S)
    si.spring_ising_debug_fail_allocs(m.ctx, ADJOINT_FAILS)
    loss, gd, gz = m.relaxed_energy_grad(5)
    torch.cuda.synchronize()
    assert not m.info()["kernel_name"].startswith("step_i8")
    _check_state(m, J, x0, S, S)
    dt, zeta = oracle_schedules(S)
    Lo, gdo, gzo = oracle.relaxed_energy_grad(J.astype(np.float64), x0.T.astype(np.float64), None,
                                              dt.astype(np.float64), zeta.astype(np.float64), qmax=QMAX)
    rel = lambda a, b: float(np.abs(a - b).max() / np.abs(b).max())
    assert abs(float(loss.cpu()[0]) - Lo) <= 1e-5 * abs(Lo)
    assert rel(gd.cpu().numpy(), gdo) <= 1e-4 and rel(gz.cpu().numpy(), gzo) <= 1e-4
    m.close()
    # between the halves: the recomputation would take other kernels
    m = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S)
    m.relaxed_energy_forward(5)
    si.spring_ising_debug_fail_allocs(m.ctx, 1)
    m.update_best()
    with pytest.raises(si.SpringIsingError) as e:
        m.relaxed_energy_backward()
    assert e.value.status == si.SI_ERR_STATE
    m.set_state(to_dev(x0), None, 0)
    m.relaxed_energy_grad(5)
    m.close()
    for call in ("resident", "autotune"):
        m = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S)
        m.set_resident(2)
        has_resident = m.info()["resident_groups"] > 0
        si.spring_ising_debug_fail_allocs(m.ctx, 1)
        if call == "autotune":
            m.autotune(3)
            si.spring_ising_tile_cache_clear()
        m.run(6)
        _check_state(m, J, x0, S, 6)
        assert m.info()["kernel_name"].startswith("step_i8") == (call == "resident" and not has_resident)
        m.close()
    with pytest.raises(si.SpringIsingError) as e:
        m2 = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S)
        si.spring_ising_debug_fail_allocs(m2.ctx, -1)
    assert e.value.status == si.SI_ERR_INVALID
