"""GPU parity of the axis passes as y and x passes of their own, on grids that the
one-launch plane kernel refuses (an axis above 64 points, or more bands than its
workgroups hold at once): every length above 64 on every axis, plane groups that
cross spheres on one stream, buffers at any value, repeated executions, and graph
replays whose buffers change. The bars are those of the other parity tests."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import TOL, make_plan, rel, to_device

pytestmark = pytest.mark.gpu

# every length compiled above the plane kernel's
LENGTHS = [72, 75, 80, 81, 90, 96, 100, 108, 120, 125, 128, 135, 144, 150, 160, 162, 180, 192, 200, 216, 225, 240,
           243, 250, 256, 270, 288, 300, 320, 324, 360, 375, 384, 400, 405, 432, 450, 480, 486, 500, 512]


def _tensor(shape, dtype):
    import torch
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    return torch.full((shape,), complex(float("nan"), 0.0), dtype=tdt, device="cuda")


# complex128, complex64 one band per lane (an odd count) and two
@pytest.mark.parametrize("dtype,nb", [("c128", 3), ("c64", 3), ("c64", 4)])
@pytest.mark.parametrize("n", LENGTHS)
def test_pass_lengths(n, dtype, nb, capfd, monkeypatch):
    """Both directions against the oracle and the potential step against them,
    with the length along x, y and z; some columns and slabs hold nothing."""
    import torch
    from paper_2406_05577_amd import Plan
    monkeypatch.setenv("FFTB_LOG", "1")
    rng = np.random.default_rng(n)
    for axis in range(3):
        dims = tuple(np.roll([n, 2, 3], axis))
        lin = rng.permutation(np.flatnonzero(rng.random(6 * n) < 0.4)).astype(np.int32)
        p = Plan(dims, [lin], nb, dtype=dtype)
        log = capfd.readouterr().err
        assert log.count("axis passes") == 2 and ("planes in one launch" in log) == (axis == 2)
        c = rng.standard_normal((lin.size, nb)) + 1j * rng.standard_normal((lin.size, nb))
        sph = to_device(c, dtype)
        c = sph.cpu().numpy().reshape(c.shape).astype(np.complex128)
        g, back = _tensor(p.info["grid_elems"], dtype), _tensor(sph.numel(), dtype)
        p.sphere_to_grid(sph, g)
        p.grid_to_sphere(g, back)
        assert rel(g.cpu().numpy(), oracle.sphere_to_grid(dims, lin, c).ravel()) <= TOL[dtype], dims
        assert rel(back.cpu().numpy(), c.ravel()) <= TOL[dtype], dims
        v = rng.random(dims[::-1]) - 0.25
        vt = torch.from_numpy(v.ravel()).to(g.real.dtype).cuda()
        v = vt.cpu().numpy().astype("f8").reshape(dims[::-1])
        pg, out = _tensor(g.numel(), dtype), _tensor(sph.numel(), dtype)
        p.apply_potential(sph, vt, pg, out)
        assert rel(pg.cpu().numpy(), (g * vt.repeat_interleave(nb)).cpu().numpy()) <= TOL[dtype], dims
        assert rel(out.cpu().numpy(), oracle.apply_potential(dims, lin, c, v).ravel()) <= TOL[dtype], dims
        p.close()


# (even counts: two complex64 bands per lane)
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("nbs", [[3, 11, 8], [4, 12, 8]])
def test_pass_groups_on_one_stream(nbs, dtype, capfd, monkeypatch):
    """Two groups of planes on the caller's stream, cut inside a sphere, over
    spheres of other maps and band counts."""
    import torch
    from paper_2406_05577_amd import Plan
    dims = (72, 27, 20)
    ws = [synth.small_workload(dims, (18, 6.75, 5), [(0.1, -0.2, 0.3)], nb, seed=60 + s, dtype=dtype, shuffle=True)
          for s, nb in enumerate(nbs)]
    maps, coeffs = [w.spheres[0].lin for w in ws], [w.coeffs[0] for w in ws]
    maps[0] = maps[0][: maps[0].size // 2]
    coeffs[0] = coeffs[0][: maps[0].size]
    monkeypatch.setenv("FFTB_LOG", "1")
    monkeypatch.setenv("FFTB_MAX_DEVICE_BYTES", str(1 << 30))   # (small groups)
    p = Plan(dims, maps, nbs, dtype=dtype)
    log = capfd.readouterr().err
    assert log.count("axis passes, 2 groups of") == 2 and "two streams" not in log and "one launch" not in log
    sph = to_device(np.concatenate([c.reshape(-1) for c in coeffs]), dtype)
    g, back = _tensor(p.info["grid_elems"], dtype), _tensor(sph.numel(), dtype)
    pg, out = _tensor(g.numel(), dtype), _tensor(sph.numel(), dtype)
    v = np.random.default_rng(6).standard_normal(dims[::-1]).astype("f8" if dtype == "c128" else "f4")
    for _ in range(2):
        p.sphere_to_grid(sph, g)
        p.grid_to_sphere(g, back)
        p.apply_potential(sph, torch.from_numpy(v.ravel()).cuda(), pg, out)
    g, pg, back, out = (t.cpu().numpy() for t in (g, pg, back, out))
    n, ga, sa = 72 * 27 * 20, 0, 0
    for m, c, nb in zip(maps, coeffs, nbs):
        c = c.astype(np.complex128)
        want = oracle.sphere_to_grid(dims, m, c)
        assert rel(g[ga:ga + n * nb], want.ravel()) <= TOL[dtype]
        assert rel(pg[ga:ga + n * nb], (want * v[..., None].astype("f8")).ravel()) <= TOL[dtype]
        assert rel(back[sa:sa + c.size], c.ravel()) <= TOL[dtype]
        assert rel(out[sa:sa + c.size], oracle.apply_potential(dims, m, c, v.astype("f8")).ravel()) <= TOL[dtype]
        ga, sa = ga + n * nb, sa + c.size
    p.close()


@pytest.mark.parametrize("dtype,nb", [("c64", 8), ("c64", 9), ("c64", 3), ("c128", 3)])
def test_separate_passes_with_buffers_at_any_value(dtype, nb, capfd, monkeypatch):
    """Buffers that start at an odd complex value: the same bits, and the bytes
    around the buffers stay as they were."""
    import torch
    monkeypatch.setenv("FFTB_LOG", "1")
    w = synth.small_workload((72, 30, 25), (18, 7, 6), [(0.2, -0.3, 0.1), (0, 0, 0)], nb, seed=78, dtype=dtype)
    p = make_plan(w, dtype=dtype)
    assert "one launch" not in capfd.readouterr().err
    sph = to_device(np.concatenate([c.reshape(-1) for c in w.coeffs]), dtype)
    v = torch.rand(72 * 30 * 25, dtype=sph.real.dtype, device="cuda")
    mark = complex(7.0, -7.0)

    def odd(n):
        t = torch.full((n + 2,), mark, dtype=sph.dtype, device="cuda")
        return t, t[1:-1]

    ns, ng = sph.numel(), p.info["grid_elems"]
    g, pg = _tensor(ng, dtype), _tensor(ng, dtype)
    back, out = _tensor(ns, dtype), _tensor(ns, dtype)
    (sa, s), (ga, g1), (pa, pg1), (ba, b1), (oa, o1) = odd(ns), odd(ng), odd(ng), odd(ns), odd(ns)
    s.copy_(sph)
    for a, b, c, d, e in ((sph, g, back, pg, out), (s, g1, b1, pg1, o1)):
        p.sphere_to_grid(a, b)
        p.grid_to_sphere(b, c)
        p.apply_potential(a, v, d, e)
    torch.cuda.synchronize()
    for a, b in ((g, g1), (back, b1), (pg, pg1), (out, o1)):
        assert torch.equal(a, b)
    for t in (sa, ga, pa, ba, oa):
        assert t[0].item() == mark and t[-1].item() == mark
    p.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_separate_passes_repeat(dtype, capfd, monkeypatch):
    """Every execution of the y and x passes gives the same bits (60x54x50 with
    more bands than the plane kernel takes: the lengths where a store's data were
    overwritten in one of 15 executions)."""
    import torch
    monkeypatch.setenv("FFTB_LOG", "1")
    w = synth.small_workload((60, 54, 50), (15, 13, 12), [(0.1, 0.2, 0.3)], 64, seed=310, dtype=dtype)
    p = make_plan(w, dtype=dtype)
    assert "one launch" not in capfd.readouterr().err
    sph = to_device(np.concatenate([c.reshape(-1) for c in w.coeffs]), dtype)
    v = torch.rand(60 * 54 * 50, dtype=sph.real.dtype, device="cuda")

    def results():
        g = p.sphere_to_grid(sph)
        vg = torch.empty_like(g)
        return g, p.grid_to_sphere(g), p.apply_potential(sph, v, vg), vg

    first = results()
    for _ in range(100):
        assert all(torch.equal(torch.view_as_real(a), torch.view_as_real(b)) for a, b in zip(results(), first))
    p.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_graph_replays_follow_the_buffers(dtype, capfd, monkeypatch):
    """A graph plan with more launches than are launched directly: replayed on the
    same buffers and captured again where any one of them changes, in both
    directions and the potential step, beside the plain plan."""
    import torch
    w = synth.small_workload((80, 72, 60), (5, 5, 5), [(0.1, 0.2, -0.3)], 12, seed=92, dtype=dtype)
    plain = make_plan(w, dtype=dtype)
    monkeypatch.setenv("FFTB_LOG", "1")
    monkeypatch.setenv("FFTB_MAX_DEVICE_BYTES", str(1 << 30))   # (small groups: many launches)
    p = make_plan(w, dtype=dtype, flags=4)
    log = capfd.readouterr().err
    assert "axis passes" in log and int(log.split("axis passes, ")[1].split(" groups")[0]) >= 3
    sph = to_device(np.concatenate([c.reshape(-1) for c in w.coeffs]), dtype)
    ng, n = p.info["grid_elems"], 80 * 72 * 60
    s = [sph, sph.flip(0).contiguous()]
    v = [torch.rand(n, dtype=sph.real.dtype, device="cuda") - 0.5 for _ in range(2)]
    g = [_tensor(ng, dtype) for _ in range(2)]
    o = [_tensor(sph.numel(), dtype) for _ in range(2)]
    want_g = [plain.sphere_to_grid(x) for x in s]
    want_o = [plain.grid_to_sphere(x) for x in want_g]
    for i, j in ((0, 0), (0, 0), (1, 0), (1, 1), (1, 1), (0, 1)):
        for t in g + o:
            t.fill_(float("nan"))
        p.sphere_to_grid(s[i], g[j])
        p.grid_to_sphere(want_g[i], o[j])
        assert torch.equal(g[j], want_g[i]) and torch.equal(o[j], want_o[i]), (i, j)
        assert torch.isnan(g[1 - j].real).all() and torch.isnan(o[1 - j].real).all()
    vg = _tensor(ng, dtype)
    for i, k, j, l in ((0, 0, 0, 0), (0, 0, 0, 0), (1, 0, 0, 0), (1, 1, 0, 0), (1, 1, 1, 0), (1, 1, 1, 1), (0, 1, 1, 1)):
        for t in g + o:
            t.fill_(float("nan"))
        p.apply_potential(s[i], v[k], g[j], o[l])
        want = plain.apply_potential(s[i], v[k], vg)
        assert torch.equal(g[j], vg) and torch.equal(o[l], want), (i, k, j, l)
        assert torch.isnan(g[1 - j].real).all() and torch.isnan(o[1 - l].real).all()
    p.close()
    plain.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_plans_of_other_sizes_live_together(dtype):
    """A plan whose kernels take much LDS runs after plans of other sizes, whose
    tiles of the same kernels take little, were made and destroyed."""
    import torch
    nb = 64 if dtype == "c128" else 128
    for dims in ((32, 32, 32), (96, 96, 96)):      # (the plane kernel, the y and x passes)
        big = synth.small_workload(dims, [0.25 * d for d in dims], [(0.1, 0.2, -0.3)], nb, seed=5, dtype=dtype)
        p = make_plan(big, dtype=dtype)
        sph = to_device(np.concatenate([c.reshape(-1) for c in big.coeffs]), dtype)
        v = torch.rand(dims[0] ** 3, dtype=sph.real.dtype, device="cuda")
        pg = _tensor(p.info["grid_elems"], dtype)
        want = p.sphere_to_grid(sph), p.apply_potential(sph, v, pg)
        others = []
        for small in (dims, (8, 6, 4)):
            w = synth.small_workload(small, [0.2 * d for d in small], [(0, 0, 0)], 1, seed=6, dtype=dtype)
            others.append(make_plan(w, dtype=dtype))
        for _ in range(2):
            got = p.sphere_to_grid(sph), p.apply_potential(sph, v, pg)
            assert all(torch.equal(a, b) for a, b in zip(got, want))
            while others:
                others.pop().close()
        p.close()
