"""The one-launch form of the split contraction at the edges of its ranges,
slabs and tiles: bit for bit the two-launch form (whose arithmetic it
repeats), which the same tile runs where the output has more tiles."""
import numpy as np
import pytest

import oracle
from paper_2305_07187_amd import instances

from gpu_common import QMAX, announce, ensure_built, oracle_schedules, to_dev

pytestmark = pytest.mark.gpu


# n: one range empty, ranges of one slab, a last range shorter than the others;
# tiles of 16 and of 32 rows; up to four and up to eight waves
@pytest.mark.parametrize("n,r,tile,ksplit", [
    (40, 1, 3, 2), (65, 3, 3, 8), (130, 33, 3, 4), (300, 64, 12, 7), (1999, 50, 3, 4),
    (33, 2, 14, 3), (257, 40, 9, 4), (300, 64, 26, 8), (1000, 128, 14, 4), (2000, 70, 14, 5)])
@pytest.mark.parametrize("order,wall", [("paper", "clamp"), ("symplectic", "inelastic")])
def test_one_launch_equals_two(n, r, tile, ksplit, order, wall):
    # the replicas of a wider context (two launches) are those of this one
    import torch
    si = ensure_built()
    announce(f"few replicas N={n} R={r} tile {tile} ksplit {ksplit} {order} {wall}")
    wide = 512 * 32 * 32 // max(n // 32 * 32, 32) + 64  # more than 512 tiles
    J = to_dev(instances.make_gauss(n, 3))
    x, p = instances.random_state(n, wide, 1, scale=1.4), instances.random_state(n, wide, 2, scale=1.4)
    h = to_dev(instances.make_x0(n, 1, 5, scale=2.0)[0])
    out = []
    for rr in (r, wide):
        m = si.SpringIsing(J, to_dev(x[:rr].copy()), to_dev(p[:rr].copy()), total_steps=20, tile=tile,
                           order=order, wall=wall)
        m.set_ksplit(ksplit)
        m.set_field(h)
        assert m.info()["kernel_name"].endswith(f"_ks{ksplit}")
        m.run(7)
        xo, po, _ = m.state()
        torch.cuda.synchronize()
        out.append((xo.cpu().numpy()[:r], po.cpu().numpy()[:r]))
        m.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("n,r,ksplit", [(65, 3, 2), (300, 50, 4), (700, 64, 8), (513, 40, 5)])
def test_adjoint_one_launch(n, r, ksplit):
    # short schedules, before trajectories part; the FP32 multipliers' bound is
    # the one of the adjoint's other tests (1e-4 of the largest entry)
    import torch
    si = ensure_built()
    S = 24
    announce(f"few replicas adjoint N={n} R={r} ksplit {ksplit}")
    J, x0 = instances.make_pm1(n, 9), instances.make_x0(n, r, 9)
    m = si.SpringIsing(to_dev(J), to_dev(x0), total_steps=S)
    m.set_ksplit(ksplit)
    loss, gd, gz = m.relaxed_energy_grad(7)
    torch.cuda.synchronize()
    dt, zeta = oracle_schedules(S)
    Lo, gdo, gzo = oracle.relaxed_energy_grad(J.astype(np.float64), x0.T.astype(np.float64), None,
                                              dt.astype(np.float64), zeta.astype(np.float64), qmax=QMAX)
    rel = lambda a, b: float(np.abs(a - b).max() / np.abs(b).max())
    assert abs(float(loss.cpu()[0]) - Lo) <= 1e-5 * abs(Lo)
    assert rel(gd.cpu().numpy(), gdo) <= 1e-4 and rel(gz.cpu().numpy(), gzo) <= 1e-4
    m.close()


@pytest.mark.parametrize("S,every", [(5, 1), (5, 5), (6, 4), (9, 100), (1, 3)])
def test_recorded_last_segment(S, every):
    # any split into segments gives the same loss, gradient and end state, with
    # the halves called one by one too
    import torch
    si = ensure_built()
    n, r = 300, 20
    announce(f"adjoint S={S} segments of {every}")
    J, x0 = to_dev(instances.make_pm1(n, 9)), to_dev(instances.make_x0(n, r, 9))
    out = []
    for every_k, energy_every in ((every, 0), (2, 0), (every, 3)):
        m = si.SpringIsing(J, x0, total_steps=S, energy_every=energy_every)
        loss = m.relaxed_energy_forward(every_k)
        x, p, t = m.state()
        gd, gz = m.relaxed_energy_backward()
        torch.cuda.synchronize()
        assert t == S
        out.append([v.cpu().numpy() for v in (loss, gd, gz, x, p)])
        m.close()
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)
