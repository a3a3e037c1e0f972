"""Many steps of a small problem in one launch: bit for bit the resident form
of the same tile (a kernel of its own), at the edges of its row blocks, for
odd and even numbers of steps (which buffer holds the result), with energy
checks on the way, and against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2305_07187_amd import instances

from gpu_common import QMAX, announce, ensure_built, oracle_schedules, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r", [(1, 1), (16, 3), (33, 70), (64, 16), (65, 17), (100, 8), (113, 5), (128, 300),
                                 (129, 64), (161, 9), (193, 33), (224, 65)])
@pytest.mark.parametrize("order,wall", [("paper", "inelastic"), ("symplectic", "clamp")])
def test_equals_resident_form(n, r, order, wall):
    import torch
    si = ensure_built()
    announce(f"small problem N={n} R={r} {order} {wall}")
    J = to_dev(np.zeros((1, 1), np.float32) if n == 1 else instances.make_gauss(n, 3))
    x, p = instances.random_state(n, r, 1, scale=1.4), instances.random_state(n, r, 2, scale=1.4)
    h = to_dev(instances.make_x0(n, 1, 5, scale=2.0)[0])
    out = []
    for resident in (0, 1):
        m = si.SpringIsing(J, to_dev(x), to_dev(p), total_steps=40, tile=3, order=order, wall=wall)
        m.set_ksplit(1)
        m.set_field(h)
        m.set_resident(resident)
        got = []
        for steps in (3, 4, 1, 2):
            m.run(steps)
            xo, po, t = m.state()
            H = m.hamiltonian()
            torch.cuda.synchronize()
            got += [t, xo.cpu().numpy(), po.cpu().numpy(), H.cpu().numpy()]
        out.append(got)
        m.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_checks_graph_and_oracle():
    import torch
    si = ensure_built()
    n, r, S = 100, 40, 60
    announce(f"small problem with energy checks and graphs N={n} R={r}")
    J, x0 = instances.make_pm1(n, 4), instances.make_x0(n, r, 4)
    a = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S, energy_every=7)
    a.run(33)
    xa, pa, _ = a.state()
    b = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S, energy_every=7)
    for _ in range(33):
        b.step()
    xb, pb, _ = b.state()
    torch.cuda.synchronize()
    assert torch.equal(xa, xb) and torch.equal(pa, pb)
    assert torch.equal(a.energy_trace(), b.energy_trace()) and a.energy_trace().shape[0] == 4
    c = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S)
    c.set_graph(5)
    for _ in range(3):
        c.set_state(to_dev(x0), None, 0)
        c.run(33)
        c.energy()
        xc, pc, _ = c.state()
        torch.cuda.synchronize()
        assert torch.equal(xa, xc) and torch.equal(pa, pc)
    dt, zeta = oracle_schedules(S)
    ref = oracle.run(J.astype(np.float64), x0.T.astype(np.float64), None, dt, zeta, qmax=QMAX, n_steps=33)
    assert rel_err(xa.cpu().numpy(), ref["Q"]) <= 1e-5 and rel_err(pa.cpu().numpy(), ref["P"]) <= 1e-5
    for m in (a, b, c):
        m.close()


@pytest.mark.parametrize("n", [128, 129])
def test_short_runs_take_the_tile(n):
    # below the least number of steps a run is launched step by step: any way
    # of cutting a run gives the same states
    import torch
    si = ensure_built()
    r, S = 20, 40
    announce(f"small problem, short runs N={n}")
    J, x0 = to_dev(instances.make_gauss(n, 4)), to_dev(instances.make_x0(n, r, 4))
    out = []
    for cuts in ([14], [1] * 14, [2, 5, 1, 6], [7, 7], [3, 11]):
        m = si.SpringIsing(J, x0, total_steps=S, energy_every=4 if len(cuts) == 2 else 0)
        for k in cuts:
            m.run(k)
        x, p, t = m.state()
        torch.cuda.synchronize()
        assert t == 14
        out.append((x.cpu().numpy(), p.cpu().numpy()))
        m.close()
    for x, p in out[1:]:
        assert np.array_equal(x, out[0][0]) and np.array_equal(p, out[0][1])
