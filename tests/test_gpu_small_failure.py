"""An injected HIP failure in a launch of many steps of a small problem: the
launch that users' runs take, failing at any of its steps."""
import pytest

from paper_2305_07187_amd import instances

from gpu_common import announce, ensure_built, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 200])
@pytest.mark.parametrize("after,ok_runs", [(1, 0), (9, 0), (10, 0), (11, 1), (25, 2)])
def test_failure_in_many_steps(n, after, ok_runs):
    import torch
    from torch.profiler import ProfilerActivity, profile
    si = ensure_built()
    announce(f"injected failure after {after} steps' calls N={n}")
    J, x0 = to_dev(instances.make_pm1(n, 1)), to_dev(instances.make_x0(n, 8, 1))
    m = si.SpringIsing(J, x0, total_steps=100)
    clean = si.SpringIsing(J, x0, total_steps=100)
    m.run(5)
    clean.run(5)
    si.spring_ising_debug_inject_hip_error(m.ctx, after)
    for _ in range(ok_runs):
        m.run(10)
        clean.run(10)
    assert m.info()["t"] == clean.info()["t"]
    with pytest.raises(si.SpringIsingError) as e:
        m.run(10)
    assert e.value.status == si.SI_ERR_HIP
    with pytest.raises(si.SpringIsingError) as e:
        m.run(1)
    assert e.value.status == si.SI_ERR_STATE
    m.close()
    # armed and never reached: the same states
    a = si.SpringIsing(J, x0, total_steps=100)
    si.spring_ising_debug_inject_hip_error(a.ctx, 1000)
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        a.run(5 + 10 * ok_runs)
        torch.cuda.synchronize()
    if n <= 128 or ok_runs:  # (N = 200: from six steps on)
        assert any("small_steps_kernel" in ev.name for ev in prof.events())
    for u, v in zip(a.state()[:2], clean.state()[:2]):
        assert torch.equal(u, v)
    a.close()
    clean.close()
