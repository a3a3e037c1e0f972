"""Tile id SI_TILE_FLOATING: the automatic choice without the fixed-point form,
which the autograd function steps with."""
import numpy as np
import pytest

from paper_2305_07187_amd import instances

from gpu_common import announce, ensure_built, oracle_schedules, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,kind,precision", [(100, 8, "pm1", "fp32"), (600, 64, "pm1", "fp32"), (700, 1001, "pm1", "fp32"),
                                                (700, 961, "gauss", "fp32"), (1000, 33, "pm1", "bf16x3_exactj"),
                                                (300, 64, "pm1", "bf16x_fp8j")])
def test_automatic_choice_without_the_form(n, r, kind, precision):
    import torch
    si = ensure_built()
    announce(f"floating tile N={n} R={r} {kind} {precision}")
    si.spring_ising_tile_cache_clear()
    J, x0 = to_dev(instances.make_J(n, kind, 2).astype(np.float32)), to_dev(instances.make_x0(n, r, 2))
    m = si.SpringIsing(J, x0, total_steps=20, precision=precision, tile=si.SI_TILE_FLOATING)
    info = m.info()
    assert not info["kernel_name"].startswith("step_i8") and info["tile"] < 64
    assert si.TILE_SOURCES[info["tile_source"]] == "table"
    m.run(8)
    x, p, _ = m.state()
    # the context that tile 0 makes, once off the form, steps the same way
    a = si.SpringIsing(J, x0, total_steps=20, precision=precision)
    if a.info()["kernel_name"].startswith("step_i8"):
        assert m.info()["device_bytes"] < a.info()["device_bytes"]
        si.spring_ising_debug_fail_allocs(a.ctx, 1)
        a.update_best()
    a.run(8)
    xa, pa, _ = a.state()
    torch.cuda.synchronize()
    assert a.info()["kernel_name"] == info["kernel_name"]
    assert torch.equal(x, xa) and torch.equal(p, pa)
    tile, _ = m.autotune(2)
    assert tile < 64 and m.info()["tile"] == tile
    b = si.SpringIsing(J, x0, total_steps=20, precision=precision, tile=si.SI_TILE_FLOATING)
    assert b.info()["tile"] == tile and si.TILE_SOURCES[b.info()["tile_source"]] == "cache"
    si.spring_ising_tile_cache_clear()
    for c in (m, a, b):
        c.close()


def test_autograd_steps_with_it():
    import torch
    from paper_2305_07187_amd.autograd import relaxed_energy
    si = ensure_built()
    n, r, S = 600, 70, 12
    announce(f"autograd on the floating tiles N={n} R={r}")
    J, x0 = to_dev(instances.make_pm1(n, 2)), to_dev(instances.make_x0(n, r, 2))
    dt, zeta = (to_dev(v.astype(np.float32)).requires_grad_() for v in oracle_schedules(S))
    loss = relaxed_energy(J, x0, None, dt, zeta, 5)
    loss.backward()
    m = si.SpringIsing(J, x0, total_steps=S, tile=si.SI_TILE_FLOATING)
    l, gd, gz = m.relaxed_energy_grad(5)
    m.set_state(x0, None, 0)
    m.run(S)
    torch.cuda.synchronize()
    m.close()
    assert float(loss.detach()) == float(l[0])
    assert torch.equal(dt.grad, gd.float()) and torch.equal(zeta.grad, gz.float())
    with pytest.raises(si.SpringIsingError) as e:
        si.SpringIsingBatch([J], [x0], total_steps=2, tile=si.SI_TILE_FLOATING)
    assert e.value.status == si.SI_ERR_INVALID
