"""autotune with a single step, at the schedule's last one: no step past its end."""
import pytest

from paper_2305_07187_amd import instances

from gpu_common import announce, ensure_built, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,precision", [(100, 8, "fp32"), (600, 300, "fp32"), (300, 64, "bf16x_fp8j"), (0, 16, "fp32")])
def test_single_step(n, r, precision):
    import torch
    si = ensure_built()
    announce(f"autotune(1) at the last step N={n} R={r} {precision}")
    S = 1024  # (the schedule's buffer ends with it)
    si.spring_ising_tile_cache_clear()
    if n:
        m = si.SpringIsing(to_dev(instances.make_pm1(n, 1)), to_dev(instances.make_x0(n, r, 1)), total_steps=S,
                           precision=precision)
    else:
        m = si.SpringIsingBatch([to_dev(instances.make_pm1(k, 1)) for k in (64, 200)],
                                [to_dev(instances.make_x0(k, r, 1)) for k in (64, 200)], total_steps=S)
    flat = lambda st: [v for a in st[:2] for v in (a if isinstance(a, list) else [a])]
    m.run(S - 1)
    before = m.state()
    tile, us = m.autotune(1)
    after = m.state()
    torch.cuda.synchronize()
    assert tile >= 1 and us > 0 and before[2] == after[2] == S - 1
    for a, b in zip(flat(before), flat(after)):
        assert torch.equal(a, b)
    m.run(1)
    with pytest.raises(si.SpringIsingError) as e:
        m.autotune(1)
    assert e.value.status == si.SI_ERR_RANGE
    si.spring_ising_tile_cache_clear()
    m.close()
