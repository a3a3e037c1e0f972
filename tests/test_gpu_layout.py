"""Copies between the caller's rows and the device layout, and the checks of J,
at the edges of their vectors, slices and tiles: copies are exact."""
import numpy as np
import pytest

from paper_2305_07187_amd import instances

from gpu_common import announce, ensure_built, to_dev

pytestmark = pytest.mark.gpu


def _shifted(a, shift):
    """Device copy of a whose first entry lies `shift` entries into a buffer."""
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a)).reshape(-1).to("cuda:0")
    buf = torch.zeros(t.numel() + 4, dtype=t.dtype, device="cuda:0")
    buf[shift:shift + t.numel()] = t
    return buf[shift:shift + t.numel()].view(a.shape)


@pytest.mark.parametrize("n,r,shift", [(1, 1, 0), (3, 5, 1), (64, 4, 0), (100, 65, 2), (255, 3, 0),
                                       (256, 64, 1), (257, 66, 3), (1028, 130, 0), (2001, 9, 0)])
@pytest.mark.parametrize("precision", ["fp32", "bf16x_fp8j"])
def test_state_round_trip(n, r, shift, precision):
    import torch
    si = ensure_built()
    announce(f"state copies N={n} R={r} shift {shift} {precision}")
    J = np.zeros((1, 1), np.float32) if n == 1 else instances.make_pm1(n, 1)
    x, p = instances.random_state(n, r, 1, scale=1.4), instances.random_state(n, r, 2, scale=1.4)
    x[0, 0] = -0.0
    m = si.SpringIsing(to_dev(J), to_dev(x), total_steps=4, precision=precision)
    s = np.where(x < 0, -1, 1).astype(np.int8)
    for pp in (p, None):
        m.set_state(_shifted(x, shift), None if pp is None else _shifted(pp, shift), 0)
        xo, po = _shifted(np.full((r, n), 7, np.float32), shift), _shifted(np.full((r, n), 7, np.float32), 3 - shift)
        so = _shifted(np.zeros((r, n), np.int8), shift)
        si.spring_ising_get_state(m.ctx, xo, po)
        si.spring_ising_spins(m.ctx, so)
        torch.cuda.synchronize()
        assert np.array_equal(xo.cpu().numpy(), x)
        assert np.array_equal(po.cpu().numpy(), 0 * p if pp is None else p)
        assert np.array_equal(so.cpu().numpy(), s)
    m.update_best()
    _, best = m.best()
    torch.cuda.synchronize()
    assert np.array_equal(best.cpu().numpy(), s)
    m.close()


@pytest.mark.parametrize("precision", ["fp32", "bf16x_mixedj"])
def test_batch_round_trip(precision):
    # a batch's copies equal single contexts' after steps, too (the BF16 planes
    # are written with the state)
    import torch
    si = ensure_built()
    ns, r = [65, 300, 128, 1001, 64, 259], 37
    announce(f"batch state copies {ns} R={r} {precision}")
    Js = [to_dev(instances.make_pm1(n, n)) for n in ns]
    xs = [instances.random_state(n, r, n, scale=1.4) for n in ns]
    ps = [instances.random_state(n, r, n + 1, scale=1.4) for n in ns]
    b = si.SpringIsingBatch(Js, [to_dev(0 * x) for x in xs], total_steps=8, precision=precision)
    flat = lambda v: np.concatenate([a.reshape(-1) for a in v])
    si.spring_ising_set_state(b.ctx, _shifted(flat(xs), 1), _shifted(flat(ps), 1), 2)
    xo, po = _shifted(flat(xs) * 0, 1), _shifted(flat(ps) * 0, 1)
    so = _shifted(flat(xs).astype(np.int8) * 0, 1)
    si.spring_ising_get_state(b.ctx, xo, po)
    si.spring_ising_spins(b.ctx, so)
    torch.cuda.synchronize()
    assert np.array_equal(xo.cpu().numpy(), flat(xs)) and np.array_equal(po.cpu().numpy(), flat(ps))
    assert np.array_equal(so.cpu().numpy(), np.where(flat(xs) < 0, -1, 1))
    b.run(3)
    c = si.SpringIsingBatch(Js, [to_dev(x) for x in xs], total_steps=8, precision=precision,
                            p0s=[to_dev(p) for p in ps])
    si.spring_ising_set_state(c.ctx, to_dev(flat(xs)), to_dev(flat(ps)), 2)
    c.run(3)
    si.spring_ising_get_state(b.ctx, xo, po)
    xc, pc = torch.empty_like(xo), torch.empty_like(po)
    si.spring_ising_get_state(c.ctx, xc, pc)
    torch.cuda.synchronize()
    assert torch.equal(xo, xc) and torch.equal(po, pc)
    b.close()
    c.close()


@pytest.mark.parametrize("n", [2, 63, 64, 65, 130, 257])
def test_checks_of_couplings_find_every_entry(n):
    # one entry changed at corners and edges of the tiles is found, on either
    # side of the diagonal; the largest coupling and the formats are reported
    si = ensure_built()
    announce(f"checks of J N={n}")
    x = to_dev(instances.make_x0(n, 3, 1))
    J = np.where(np.add.outer(np.arange(n), np.arange(n)) % 3 == 0, 1.0, -1.0).astype(np.float32)
    np.fill_diagonal(J, 0.0)
    spots = sorted({(i, j) for i in (0, 1, 62, 63, 64, 65, 128, n - 2, n - 1) for j in (0, 63, 64, n - 1)
                    if 0 <= i < n and 0 <= j < n and i != j})

    def init(M):
        m = si.SpringIsing(to_dev(M), x, total_steps=2)
        info = m.info()
        m.close()
        return info["j_integer"], info["j_fp8_exact"], info["j_bf16_exact"]
    assert init(J) == (1, 1, 1)
    for i, j in spots:
        for value in (5.0, np.nan, np.inf):
            M = J.copy()
            M[i, j] = value  # asymmetric or not finite
            with pytest.raises(si.SpringIsingError):
                init(M)
        for value, want in ((127.0, (1, 0, 1)), (128.0, (0, 1, 1)), (0.1, (0, 0, 0)), (0.0, (1, 1, 1))):
            M = J.copy()
            M[i, j] = M[j, i] = value
            assert init(M) == want, (i, j, value)
    M = J.copy()
    M[n - 1, n - 1] = 1.0
    with pytest.raises(si.SpringIsingError):
        init(M)


@pytest.mark.parametrize("n,r,shift", [(2, 1, 0), (63, 127, 1), (128, 128, 0), (130, 129, 3),
                                       (257, 20, 2), (1001, 300, 1), (1536, 640, 0)])
def test_energy_noalloc_tile_edges(n, r, shift):
    # tiles of 128, slabs of 64, one and several parts of the contraction, rows
    # that start on any float; integers, so equal
    import torch
    si = ensure_built()
    announce(f"energy_noalloc N={n} R={r} shift {shift}")
    rng = np.random.default_rng(n)
    A = np.triu(rng.integers(-127, 128, (n, n)), 1)
    A = A + A.T
    x = rng.uniform(-1, 1, (r, n)).astype(np.float32)
    x[0, 0], x[-1, -1] = -0.0, 0.0
    e = torch.zeros(r, dtype=torch.int32, device="cuda:0")
    si.spring_ising_energy_noalloc(_shifted(A.astype(np.float32), shift), _shifted(x, shift), e)
    torch.cuda.synchronize()
    s = np.where(x < 0, -1.0, 1.0)
    ref = -0.5 * np.einsum("ri,ri->r", s @ A.astype(np.float64), s)
    assert np.array_equal(e.cpu().numpy(), ref.astype(np.int64))
