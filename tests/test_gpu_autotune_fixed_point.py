"""The autotuner where the context has the fixed-point form: the id, the time,
the kernel in use and the cached choice name the same kernel."""
import numpy as np
import pytest

from paper_2305_07187_amd import instances

from gpu_common import announce, ensure_built, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def clean_cache():
    si = ensure_built()
    si.spring_ising_tile_cache_clear()
    yield
    si.spring_ising_tile_cache_clear()


def _run(m, steps):
    import torch
    m.run(steps)
    x, p, _ = m.state()
    torch.cuda.synchronize()
    return x, p


@pytest.mark.parametrize("n,r,precision", [(1000, 1024, "fp32"), (1500, 64, "fp32"), (1200, 300, "bf16x3_exactj")])
def test_choice_names_one_kernel(n, r, precision):
    import torch
    si = ensure_built()
    announce(f"autotune with the fixed-point form N={n} R={r} {precision}")
    S = 60
    J, x0 = instances.make_pm1(n, 3), to_dev(instances.make_x0(n, r, 3))
    Jd = to_dev(J)
    a = si.SpringIsing(Jd, x0, total_steps=S, precision=precision)
    assert a.info()["tile"] == si.SI_TILE_FIXED_POINT
    a.run(3)
    before = a.state()
    tile, us = a.autotune(20)
    after = a.state()
    torch.cuda.synchronize()
    assert before[2] == after[2] == 3
    assert torch.equal(before[0], after[0]) and torch.equal(before[1], after[1])
    info = a.info()
    fixed = info["kernel_name"].startswith("step_i8")
    assert info["tile"] == tile and (tile == si.SI_TILE_FIXED_POINT) == fixed and us > 0
    assert fixed or precision != "fp32"  # (FP32 takes twice as long on every tile at these sizes)
    a.set_state(x0, None, 0)
    want = _run(a, 12)
    # a later context of the key, and the id handed back, run the same kernel
    for tile_arg, source in ((0, "cache"), (tile, "caller")):
        b = si.SpringIsing(Jd, x0, total_steps=S, precision=precision, tile=tile_arg)
        i = b.info()
        assert i["tile"] == tile and i["kernel_name"] == info["kernel_name"]
        assert si.TILE_SOURCES[i["tile_source"]] == source
        got = _run(b, 12)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        b.close()
    # a context of the same sizes without the form has a key of its own
    J[3, 4] = J[4, 3] = 0.0
    c = si.SpringIsing(to_dev(J), x0, total_steps=S, precision=precision)
    assert si.TILE_SOURCES[c.info()["tile_source"]] == "table" and c.info()["tile"] < 64
    tile_c, _ = c.autotune(3)
    assert c.info()["tile"] == tile_c < 64
    c.close()
    d = si.SpringIsing(Jd, x0, total_steps=S, precision=precision)
    assert d.info()["tile"] == tile
    d.close()
    a.close()


def test_cached_tile_is_honoured(tmp_path):
    # an entry that says a tile beat the fixed point: later contexts start on it
    import torch
    si = ensure_built()
    n, r, S = 1000, 1024, 30
    announce("cached tile in place of the fixed-point form")
    Jd, x0 = to_dev(instances.make_pm1(n, 3)), to_dev(instances.make_x0(n, r, 3))

    def load(entry):
        si.spring_ising_tile_cache_clear()
        path = tmp_path / "cache.txt"
        path.write_text(f"# spring_ising tile cache 1\nbuild {si.spring_ising_build_id()}\n{entry}\n")
        assert si.spring_ising_tile_cache_load(str(path)) == 1

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    load(f"0 0 10 1 1024 {cus} 14 1.0")
    a = si.SpringIsing(Jd, x0, total_steps=S)
    b = si.SpringIsing(Jd, x0, total_steps=S, tile=14)
    assert a.info()["tile"] == 14 and si.TILE_SOURCES[a.info()["tile_source"]] == "cache"
    assert a.info()["kernel_name"].startswith("step_f32")
    got, want = _run(a, 10), _run(b, 10)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    # tuning again: among the tiles, kept under the same key
    tile, _ = a.autotune(3)
    assert a.info()["tile"] == tile < 64
    c = si.SpringIsing(Jd, x0, total_steps=S)
    assert c.info()["tile"] == tile and si.TILE_SOURCES[c.info()["tile_source"]] == "cache"
    for m in (a, b, c):
        m.close()
    load(f"0 0 10 0 1024 {cus} 14 1.0")  # of contexts without the form
    a = si.SpringIsing(Jd, x0, total_steps=S)
    assert a.info()["tile"] == si.SI_TILE_FIXED_POINT
    a.close()


def test_asked_for_where_it_does_not_apply():
    si = ensure_built()
    n, r = 600, 300
    J = instances.make_pm1(n, 8)
    hole = J.copy()
    hole[3, 4] = hole[4, 3] = 0.0
    x = to_dev(instances.make_x0(n, r, 8))
    T = si.SI_TILE_FIXED_POINT
    m = si.SpringIsing(to_dev(J), x, total_steps=2, tile=T)
    assert m.info()["kernel_name"].startswith("step_i8")
    m.set_ksplit(1)
    assert m.info()["tile"] < 64
    m.close()
    for Jc, kw in ((hole, {}), (J, {"order": "symplectic"}), (J, {"precision": "bf16x_fp8j"}),
                   (J[:100, :100].copy(), {}), (hole, {"precision": "bf16x3_exactj"})):
        with pytest.raises(si.SpringIsingError) as e:
            si.SpringIsing(to_dev(Jc), x[:, :Jc.shape[0]].contiguous(), total_steps=2, tile=T, **kw)
        assert e.value.status == si.SI_ERR_INVALID
    with pytest.raises(si.SpringIsingError) as e:
        si.SpringIsingBatch([to_dev(J)], [x], total_steps=2, tile=T)
    assert e.value.status == si.SI_ERR_INVALID
