"""GPU parity of the axis passes: the lengths where their two stages can go
wrong (single stage, the smallest and the largest splits, odd and unbalanced
radices), band counts around a piece, several rows per tile, several spheres
of different sizes, groups of planes, and the general kernels on the same
inputs. Bars: those of the other parity tests."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import TOL, check_workload, make_plan, rel, to_device

pytestmark = pytest.mark.gpu

# dims, k-points, bands
SHAPES = [
    ((16, 18, 20), 1, 3),       # one stage, then the shortest two-stage splits
    ((18, 25, 27), 2, 1),       # odd radices, one band: many rows per tile
    ((512, 4, 3), 1, 3),        # 32 x 16 along x (more bands are refused, as by the general kernels)
    ((3, 512, 4), 1, 9),
    ((4, 3, 512), 1, 8),
    ((125, 6, 5), 1, 7),        # 25 x 5
    ((5, 243, 6), 1, 2),        # 27 x 9
    ((6, 5, 486), 1, 3),        # 27 x 18
    ((48, 45, 64), 2, 37),      # ragged bands, several band tiles
    ((60, 54, 50), 1, 16),
    ((72, 96, 100), 1, 2),      # many lines per tile: tables too long to stage
]


def _workload(dims, nk, nb, dtype, seed):
    ks = np.random.default_rng(seed).uniform(-0.5, 0.5, (nk, 3))
    semi = [max(0.25 * d, 0.6) for d in dims]
    ks = [tuple(float(k) if d > 6 else 0.0 for k, d in zip(kk, dims)) for kk in ks]
    return synth.small_workload(dims, semi, ks, nb, seed=seed, dtype=dtype, shuffle=True)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_pass_shapes(i, dtype, capfd, monkeypatch):
    dims, nk, nb = SHAPES[i]
    monkeypatch.setenv("FFTB_LOG", "1")
    w = _workload(dims, nk, nb, dtype, 300 + i)
    make_plan(w, dtype=dtype).close()
    assert capfd.readouterr().err.count("axis passes") == 2
    e = check_workload(w, dtype, flags=(0, 1, 4, 5)[i % 4], reps=2)
    assert max(e) <= TOL[dtype], (dims, e)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("static", [False, True])
def test_pass_groups_spheres_and_general_path(dtype, static, capfd, monkeypatch):
    """Spheres with other maps and band counts in several groups of planes
    (the bound makes the groups small), with the potential, against the oracle
    and against the LDS-stage kernels."""
    import torch
    from paper_2406_05577_amd import Plan
    dims, nbs = (30, 27, 20), [3, 11, 8]
    ws = [synth.small_workload(dims, (7, 6, 5), [(0.1 * s, -0.2, 0.3)], nb, seed=50 + s, dtype=dtype,
                               shuffle=True) for s, nb in enumerate(nbs)]
    maps, coeffs = [w.spheres[0].lin for w in ws], [w.coeffs[0] for w in ws]
    maps[1] = maps[1][: maps[1].shape[0] // 2]      # a sphere with missing columns
    coeffs[1] = coeffs[1][: maps[1].shape[0]]
    v = np.random.default_rng(5).standard_normal(dims[::-1]).astype("f8" if dtype == "c128" else "f4")
    monkeypatch.setenv("FFTB_LOG", "1")
    monkeypatch.setenv("FFTB_MAX_DEVICE_BYTES", str(1 << 30))
    p = Plan(dims, maps, nbs, dtype=dtype)
    assert "inverse: axis passes, 1 groups" not in capfd.readouterr().err
    q = Plan(dims, maps, nbs, dtype=dtype, tuning=dict(path=1))
    sph = to_device(np.concatenate([c.reshape(-1) for c in coeffs]), dtype)
    vt = torch.from_numpy(v.reshape(-1)).cuda()
    grid = torch.full((p.info["grid_elems"],), complex(float("nan"), 0.0), dtype=sph.dtype, device="cuda")
    (p.sphere_to_grid_static if static else p.sphere_to_grid)(sph, grid)
    plain = grid.clone()
    out = p.apply_potential(sph, vt, grid=grid)
    gq = q.sphere_to_grid(sph)
    oq = q.apply_potential(sph, vt)
    torch.cuda.synchronize()
    assert rel(plain.cpu().numpy(), gq.cpu().numpy()) <= TOL[dtype]
    assert rel(out.cpu().numpy(), oq.cpu().numpy()) <= TOL[dtype]
    g, o, n = plain.cpu().numpy(), out.cpu().numpy(), dims[0] * dims[1] * dims[2]
    ga = oa = 0
    for m, c, nb in zip(maps, coeffs, nbs):
        c = c.astype(np.complex128)
        gg, oo = g[ga:ga + n * nb], o[oa:oa + c.size]
        ga, oa = ga + n * nb, oa + c.size
        assert rel(gg, oracle.sphere_to_grid(dims, m, c).ravel()) <= TOL[dtype]
        assert rel(oo, oracle.apply_potential(dims, m, c, v.astype("f8")).ravel()) <= TOL[dtype]
    p.close()
    q.close()


@pytest.mark.parametrize("dtype,nb", [("c64", 8), ("c64", 9), ("c64", 3), ("c128", 3)])
def test_pass_buffers_at_any_value(dtype, nb):
    """Buffers that start at an odd complex value (8-byte aligned complex64):
    the passes' 16-byte accesses take any address a value may have; the bytes
    around the buffers stay as they were."""
    import torch
    w = _workload((36, 30, 25), 2, nb, dtype, 77)
    p = make_plan(w, dtype=dtype)
    sph = to_device(np.concatenate([c.reshape(-1) for c in w.coeffs]), dtype)
    grid = p.sphere_to_grid(sph)
    back = p.grid_to_sphere(grid)
    mark = complex(7.0, -7.0)

    def odd(n):
        t = torch.full((n + 2,), mark, dtype=sph.dtype, device="cuda")
        return t, t[1:-1]

    s_all, s = odd(sph.numel())
    g_all, g = odd(grid.numel())
    b_all, b = odd(sph.numel())
    s.copy_(sph)
    p.sphere_to_grid(s, g)
    p.grid_to_sphere(g, b)
    torch.cuda.synchronize()
    assert torch.equal(g, grid) and torch.equal(b, back)
    for t in (s_all, g_all, b_all):
        assert t[0].item() == mark and t[-1].item() == mark
    p.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_pass_repeats(dtype):
    """Every execution gives the same bits (a hazard between a store and the
    next use of its registers showed in one of 15 executions)."""
    import torch
    w = _workload((60, 54, 50), 1, 16, dtype, 309)
    sph = torch.from_numpy(w.sphere_concat()).to("cuda").to(
        torch.complex128 if dtype == "c128" else torch.complex64)
    p = make_plan(w, dtype=dtype)
    pot = torch.rand(60 * 54 * 50, dtype=sph.real.dtype, device="cuda")

    def results():
        g = p.sphere_to_grid(sph)
        vg = torch.empty_like(g)
        return g, p.grid_to_sphere(g), p.apply_potential(sph, pot, vg), vg

    first = results()
    for _ in range(200):
        assert all(torch.equal(torch.view_as_real(a), torch.view_as_real(b))
                   for a, b in zip(results(), first))
    p.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_pass_potential(i, dtype):
    """The potential step's x pass (both transforms of a row in one workgroup)
    against the two directions run one after the other, which the oracle checks."""
    import torch
    dims, nk, nb = SHAPES[i]
    w = _workload(dims, nk, nb, dtype, 500 + i)
    sph = torch.from_numpy(w.sphere_concat()).to("cuda").to(
        torch.complex128 if dtype == "c128" else torch.complex64)
    p = make_plan(w, dtype=dtype, flags=(0, 4)[i % 2])
    v = torch.rand(dims[0] * dims[1] * dims[2], dtype=sph.real.dtype, device="cuda") - 0.25
    g = torch.full((p.info["grid_elems"],), complex(float("nan"), 0.0), dtype=sph.dtype, device="cuda")
    out = torch.full_like(sph, complex(float("nan"), 0.0))
    for _ in range(2):
        p.apply_potential(sph, v, g, out)
    want = p.sphere_to_grid(sph)
    at = 0
    for s in w.spheres:
        n = v.numel() * s.nbands
        want[at:at + n] *= v.repeat_interleave(s.nbands)
        at += n
    assert rel(g.cpu().numpy(), want.cpu().numpy()) <= TOL[dtype]
    assert rel(out.cpu().numpy(), p.grid_to_sphere(want).cpu().numpy()) <= TOL[dtype]
    p.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("mode", ["plain", "stream", "graph", "capture"])
def test_pass_two_streams(mode, dtype, capfd, monkeypatch):
    """The planes on two streams: the same bits as on one, on the caller's
    stream, replayed and captured, with the caller's work queued behind each
    call (a spoiled or freed buffer shows a missing wait)."""
    import torch
    w = synth.small_workload((80, 72, 60), (5, 5, 5), [(0.1, 0.2, -0.3), (0, 0, 0)], 12, seed=91, dtype=dtype)
    sph = to_device(np.concatenate([c.reshape(-1) for c in w.coeffs]), dtype)
    v = torch.rand(80 * 72 * 60, dtype=sph.real.dtype, device="cuda") - 0.5
    one = make_plan(w, dtype=dtype)
    want = one.sphere_to_grid(sph)
    back = one.grid_to_sphere(want)
    vg = torch.empty_like(want)
    vout = one.apply_potential(sph, v, vg)
    monkeypatch.setenv("FFTB_LOG", "1")
    monkeypatch.setenv("FFTB_MAX_DEVICE_BYTES", str(1 << 30))   # (small groups)
    p = make_plan(w, dtype=dtype, flags=4 if mode == "graph" else 0)
    assert "on two streams" in capfd.readouterr().err
    monkeypatch.delenv("FFTB_MAX_DEVICE_BYTES")
    s_in, g, s, pg, po = sph.clone(), torch.empty_like(want), torch.empty_like(sph), torch.empty_like(want), torch.empty_like(sph)

    def step():
        p.sphere_to_grid(s_in, g)
        p.grid_to_sphere(g, s)
        p.apply_potential(s_in, v, pg, po)

    st = torch.cuda.Stream() if mode != "plain" else torch.cuda.current_stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        if mode == "capture":
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=st):
                step()
            step = graph.replay
        for _ in range(5):
            for t in (g, s, pg, po):
                t.fill_(float("nan"))
            s_in.copy_(sph)
            step()
            s_in.fill_(float("nan"))
            for t, r in ((g, want), (s, back), (pg, vg), (po, vout)):
                assert torch.equal(t, r)
    torch.cuda.synchronize()
    p.close()
    one.close()


PLANE_LENGTHS = [1, 2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64]


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("i", range(len(PLANE_LENGTHS)))
def test_plane_kernel(i, dtype, capfd, monkeypatch):
    """Planes in one launch: every length on both axes, whole and cut band tiles,
    spheres of other band counts, both directions against the oracle and the
    potential step against them."""
    import torch
    from paper_2406_05577_amd import Plan
    dims = (PLANE_LENGTHS[i], PLANE_LENGTHS[(7 * i + 5) % len(PLANE_LENGTHS)], 3 + i % 3)
    nbs = [((1, 4), (3, 6), (16, 10), (33, 2))[i % 4], (2,)][i % 5 == 4]
    ws = [_workload(dims, 1, nb, dtype, 700 + 10 * i + s) for s, nb in enumerate(nbs)]
    monkeypatch.setenv("FFTB_LOG", "1")
    p = Plan(dims, [w.spheres[0].lin for w in ws], list(nbs), dtype=dtype, flags=(0, 4)[i % 2])
    assert capfd.readouterr().err.count("planes in one launch") == 2
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    sph = to_device(np.concatenate([w.coeffs[0].reshape(-1) for w in ws]), dtype)
    nan = complex(float("nan"), 0.0)
    g = torch.full((p.info["grid_elems"],), nan, dtype=tdt, device="cuda")
    back = torch.full_like(sph, nan)
    for _ in range(2):
        p.sphere_to_grid(sph, g)
        p.grid_to_sphere(g, back)
    n = dims[0] * dims[1] * dims[2]
    v = torch.rand(n, dtype=g.real.dtype, device="cuda") - 0.25
    want, at, soff = g.clone(), 0, 0
    for w, nb in zip(ws, nbs):
        s = w.spheres[0]
        c = sph[soff:soff + s.ns * nb].cpu().numpy().reshape(s.ns, nb).astype(np.complex128)
        got = g[at:at + n * nb].cpu().numpy()
        assert rel(got, oracle.sphere_to_grid(dims, s.lin, c).ravel()) <= TOL[dtype], (dims, nb)
        assert rel(back[soff:soff + s.ns * nb].cpu().numpy(), c.ravel()) <= TOL[dtype], (dims, nb)
        want[at:at + n * nb] *= v.repeat_interleave(nb)
        at, soff = at + n * nb, soff + s.ns * nb
    pg, out = torch.full_like(g, nan), torch.full_like(sph, nan)
    for _ in range(2):
        p.apply_potential(sph, v, pg, out)
    assert rel(pg.cpu().numpy(), want.cpu().numpy()) <= TOL[dtype]
    assert rel(out.cpu().numpy(), p.grid_to_sphere(want).cpu().numpy()) <= TOL[dtype]
    p.close()
