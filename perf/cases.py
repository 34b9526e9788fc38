"""The transforms whose speed this framework is judged by.

A case is one piece of work of a plane-wave electronic-structure program: some
k-points' cutoff spheres on one FFT grid, a number of bands, a precision, the
plan's flags, and what is done with them:

    inverse     Plan.sphere_to_grid: coefficients to the grid (a density build)
    forward     Plan.grid_to_sphere: the grid back to coefficients
    round_trip  both, one after the other (what the benchmark times)
    potential   Plan.apply_potential: c' = P V P^-1 c, the Hamiltonian's local part
    cuboid      the plain batched 3D FFT and back (Plan.cuboid)

Sizes are this repository's own workloads (32^3, 96^3, 128^3, 144x160x180 and
256^3 with their spheres) and generic grids with factors 2, 3 and 5, since a
grid follows from the cell and the cutoff and is rarely a power of two. The
sphere's diameter is about half of the grid's edge, as a wavefunction cutoff
gives it for an alias-free density.
"""
import math

import numpy as np
import torch

from paper_2406_05577_amd import Plan

DTYPES = {"c128": torch.complex128, "c64": torch.complex64}
REALS = {"c128": torch.float64, "c64": torch.float32}
FLAGS = {"plain": 0, "batched": 1, "graph": 4, "batched_graph": 5}


def _case(name, op, dims, bands, dtype, kpoints=1, kseed=0, mode="plain", ratio=0.25):
    c = {"name": name} if name else {}
    c.update(op=op, nx=dims[0], ny=dims[1], nz=dims[2], bands=bands, dtype=dtype,
             kpoints=kpoints, kseed=kseed, mode=mode, ratio=ratio)
    return c


def listed():
    return [
        # the smallest call: a few bands of a small molecule's box at Gamma, where
        # launches and host time count
        _case("small_box_32_c128", "round_trip", (32, 32, 32), 4, "c128"),
        # many bands of the small box in single precision, replayed as a graph
        # (an eigensolver's inner loop)
        _case("many_bands_32_c64_graph", "round_trip", (32, 32, 32), 256, "c64", mode="graph"),
        # several k-points of a bulk crystal in one batched plan (96^3, 8 k-points x 64 bands)
        _case("kpoints_96_c64_batched", "round_trip", (96, 96, 96), 64, "c64", kpoints=8, kseed=4,
              mode="batched_graph"),
        # the density build of a 256-band supercell: the inverse alone, double precision
        _case("inverse_128_c128", "inverse", (128, 128, 128), 256, "c128"),
        # projecting real-space products of the same cell back: the forward alone, single precision
        _case("forward_128_c64", "forward", (128, 128, 128), 256, "c64"),
        # the Hamiltonian's local part on one k-point of the orthorhombic cell
        _case("hamiltonian_144x160x180_c128", "potential", (144, 160, 180), 128, "c128", kseed=5),
        # the same cell's batched single-precision form over two k-points (the benchmark's other half)
        _case("kpoints_144x160x180_c64_batched", "round_trip", (144, 160, 180), 128, "c64",
              kpoints=2, kseed=5, mode="batched_graph"),
        # the paper's experiment shape, the largest grid, with a block of bands
        _case("large_256_c128", "round_trip", (256, 256, 256), 24, "c128"),
        # a surface slab: a short and wide cell with a long vacuum axis, two k-points, odd band count
        _case("surface_60x72x180_c128", "potential", (60, 72, 180), 37, "c128", kpoints=2, kseed=9),
        # an ordinary cell whose grid is no benchmark size, ragged bands
        _case("cell_108x100x120_c64", "round_trip", (108, 100, 120), 50, "c64", kseed=10),
        # a large cell on such a grid, a block of bands of a Davidson step
        _case("supercell_200x192x216_c128", "round_trip", (200, 192, 216), 20, "c128", kseed=11),
        # densities and potentials: the dense batched 3D FFT, every point a coefficient
        _case("dense_fft_90x80x72_c128", "cuboid", (90, 80, 72), 24, "c128"),
    ]


def _smooth(lo, hi):
    out = []
    for n in range(lo, hi + 1):
        k = n
        for p in (2, 3, 5):
            while k % p == 0:
                k //= p
        if k == 1:
            out.append(n)
    return out


def draw(rng):
    """A cell of any size and shape the listed ones lie between."""
    while True:
        edge = math.exp(rng.uniform(math.log(24), math.log(216)))
        dims = []
        for axis in range(3):
            stretch = rng.uniform(0.8, 1.25) * (rng.uniform(1.0, 2.5) if axis == 2 and rng.random() < 0.25 else 1.0)
            e = min(max(edge * stretch, 24), 240)
            dims.append(rng.choice(_smooth(max(24, int(0.95 * e)), int(1.08 * e) + 2)))
        dtype = rng.choice(["c128", "c64"])
        op = rng.choice(["inverse", "forward", "round_trip", "potential", "round_trip", "potential", "cuboid"])
        kpoints = 1 if op == "cuboid" else rng.choice([1, 1, 1, 2, 3, 4, 8])
        n = dims[0] * dims[1] * dims[2]
        per_band = n * kpoints * (16 if dtype == "c128" else 8)
        most = min(256, int(4e9 / per_band / (4 if op == "cuboid" else 1)))
        if most < 1:
            continue
        bands = int(math.exp(rng.uniform(0, math.log(most + 1))))
        c = _case(None, op, dims, max(1, min(bands, most)), dtype, kpoints=kpoints,
                  kseed=0 if kpoints == 1 and rng.random() < 0.3 else rng.randrange(1, 1000),
                  mode=rng.choice(["plain", "plain", "batched", "graph", "batched_graph"]),
                  ratio=round(rng.choice([0.25, 0.25, rng.uniform(0.17, 0.33)]), 3))
        return c


def _dims(case):
    return case["nx"], case["ny"], case["nz"]


def _maps(case):
    """The spheres' maps: the wrapped linear index of each G with
    sum(((m_i + k_i) / a_i)^2) <= 1, x-major with z fastest."""
    dims = _dims(case)
    if case["op"] == "cuboid":
        return [np.arange(dims[0] * dims[1] * dims[2], dtype=np.int32)]
    if case["kseed"]:
        ks = np.random.default_rng(case["kseed"]).uniform(-0.5, 0.5, (case["kpoints"], 3))
    else:
        ks = np.zeros((case["kpoints"], 3))
    maps = []
    for k in ks:
        terms, wrapped = [], []
        for n, ki in zip(dims, k):
            r = int(math.ceil(case["ratio"] * n)) + 1
            m = np.arange(-r, r + 1)
            terms.append(((m + ki) / (case["ratio"] * n)) ** 2)
            wrapped.append(m % n)
        inside = (terms[0][:, None, None] + terms[1][:, None]) + terms[2] <= 1.0
        ix, iy, iz = np.nonzero(inside)
        lin = wrapped[0][ix] + dims[0] * (wrapped[1][iy] + dims[1] * wrapped[2][iz].astype(np.int64))
        maps.append(lin.astype(np.int32))
    return maps


def _random(n, dtype, gen):
    return torch.randn(n, dtype=dtype, device="cuda", generator=gen)


def _inputs(case, seed, ncoef):
    """The input buffer, band fastest, and the potential (or None)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n = case["nx"] * case["ny"] * case["nz"]
    bands = case["bands"]
    count = n * bands * case["kpoints"] if case["op"] in ("forward", "cuboid") else ncoef * bands
    data = _random(count, DTYPES[case["dtype"]], gen)
    pot = _random(n, REALS[case["dtype"]], gen) if case["op"] == "potential" else None
    return data, pot


def prepare(case, seed):
    maps = _maps(case)
    flags = FLAGS[case["mode"]]
    if case["op"] == "cuboid":
        plan = Plan.cuboid(_dims(case), case["bands"], dtype=case["dtype"], flags=flags)
    else:
        plan = Plan(_dims(case), maps, case["bands"], dtype=case["dtype"], flags=flags)
    data, pot = _inputs(case, seed, sum(m.shape[0] for m in maps))
    dt = DTYPES[case["dtype"]]
    grid = None if case["op"] == "forward" else torch.empty(plan.info["grid_elems"], dtype=dt, device="cuda")
    out = None if case["op"] == "inverse" else torch.empty(plan.info["sphere_elems"], dtype=dt, device="cuda")
    return {"op": case["op"], "plan": plan, "in": data, "pot": pot, "grid": grid, "out": out}


def run(state):
    op, plan = state["op"], state["plan"]
    if op == "inverse":
        return plan.sphere_to_grid(state["in"], state["grid"])
    if op == "forward":
        return plan.grid_to_sphere(state["in"], state["out"])
    if op == "potential":
        out = plan.apply_potential(state["in"], state["pot"], grid=state["grid"], out=state["out"])
        return state["grid"], out
    grid = plan.sphere_to_grid(state["in"], state["grid"])  # round_trip, cuboid
    return grid, plan.grid_to_sphere(grid, state["out"])


def work(case):
    """Bytes: what each entry point reads and writes once. Operations:
    5 n log2 n per line, z lines on the occupied columns, y lines on the
    occupied (x, z), x lines on the whole grid."""
    nx, ny, nz = _dims(case)
    n, size = nx * ny * nz, 16 if case["dtype"] == "c128" else 8
    ncoef, flops = 0, 0.0
    for lin in _maps(case):
        ncoef += lin.shape[0]
        columns = np.unique(lin % (nx * ny))
        slabs = np.unique(lin % nx)
        flops += 5.0 * (len(columns) * nz * math.log2(nz) + len(slabs) * nz * ny * math.log2(ny)
                        + n * math.log2(nx))
    both = case["op"] in ("round_trip", "cuboid", "potential")
    points = n * case["kpoints"]
    moved = (ncoef + points) * case["bands"] * size * (2 if case["op"] in ("round_trip", "cuboid") else 1)
    if case["op"] == "potential":
        moved += ncoef * case["bands"] * size + n * size // 2
    return {"bytes": moved, "flops": flops * case["bands"] * (2 if both else 1)}


def _dft(n, sign):
    j = torch.arange(n, dtype=torch.int64)
    ang = (2.0 * math.pi / n) * ((j[:, None] * j) % n).to(torch.float64)
    return torch.complex(torch.cos(ang), sign * torch.sin(ang)).cuda()


def _axes(a, mats):
    """The dense transform of a[z][y][x][b] along each axis."""
    nz, ny, nx, nb = a.shape
    a = (mats[2] @ a.reshape(nz, -1)).reshape(nz, ny, nx * nb)
    for z in range(nz):
        a[z] = mats[1] @ a[z]
    a = a.reshape(nz, ny, nx, nb)
    for z in range(nz):
        a[z] = torch.matmul(mats[0], a[z])
    return a


def exact(case, seed):
    """The definition in 64 bits: dense DFT matrices along the three axes."""
    nx, ny, nz = _dims(case)
    n, bands, op = nx * ny * nz, case["bands"], case["op"]
    maps = [torch.from_numpy(m.astype(np.int64)).cuda() for m in _maps(case)]
    data, pot = _inputs(case, seed, sum(m.shape[0] for m in maps))
    inv = [_dft(k, +1) for k in (nx, ny, nz)]
    fwd = [_dft(k, -1) for k in (nx, ny, nz)]
    data = data.to(torch.complex128)
    if pot is not None:
        pot = pot.to(torch.float64).reshape(nz, ny, nx, 1)
    grids, outs, at = [], [], 0
    for lin in maps:
        count = (n if op == "forward" else lin.shape[0]) * bands
        block = data[at:at + count].reshape(-1, bands)
        at += count
        grid = block.new_empty((nz, ny, nx, bands))
        back = block.new_empty((lin.shape[0], bands))
        for b in range(0, bands, 16):
            e = min(bands, b + 16)
            if op == "forward":
                g = block[:, b:e].reshape(nz, ny, nx, e - b)
            else:
                g = block.new_zeros((n, e - b))
                g[lin] = block[:, b:e]
                g = _axes(g.reshape(nz, ny, nx, e - b), inv)
                if pot is not None:
                    g = g * pot
                grid[..., b:e] = g
            if op != "inverse":
                back[:, b:e] = _axes(g, fwd).reshape(n, e - b)[lin] / float(n)
        grids.append(grid.reshape(-1))
        outs.append(back.reshape(-1))
        del block, grid, back
    join = lambda parts: parts[0] if len(parts) == 1 else torch.cat(parts)  # noqa: E731
    if op == "inverse":
        return join(grids)
    if op == "forward":
        return join(outs)
    return join(grids), join(outs)
