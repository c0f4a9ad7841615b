"""Energies at the edges of the spline kernels' rules, through the C ABI: points without a finite energy beside equal
ones, flat tetrahedra exactly on a grid energy, a point far off the others. Against the FP64 oracle, gate 1e-5 of the
largest value (FP32 energies and additions)."""
import numpy as np
import pytest

import synth
from gates import dos_err

pytestmark = pytest.mark.gpu

KINDS = ["dos", "exact", "batched", "nos", "binned"]


def _both(oracle_lib, kind, eps, w, grid, e0, de, ne, flat):
    """The oracle's result and the library's. A tetrahedron that is flat at a grid energy counts there (E_j >= E4),
    in the oracle only above it (E_j > E1): it gets that energy one step down."""
    import torch
    import paper_1710_10789_amd as tetra

    te, tw = torch.from_numpy(eps).cuda(), torch.from_numpy(w).cuda()
    args = (te, tw, grid, e0, de, ne)
    if flat is not None:
        eps = np.where(eps == np.float32(flat), np.nextafter(np.float32(flat), np.float32(-np.inf)), eps)
    if kind == "nos":
        ref, got = oracle_lib.nos(eps, w, grid, e0, de, ne), tetra.nos_forward(*args)
    elif kind == "binned":
        ref, got = oracle_lib.dos_binned(eps, w, grid, e0, de, ne), tetra.dos_binned(*args)
    else:
        ref = oracle_lib.dos(eps, w, grid, e0, de, ne)
        if kind == "batched":
            got = tetra.dos_batched([args + (None,), args + (None,)])[1]
        else:
            got = tetra.dos_forward(*args, deterministic=kind == "exact")
    return np.asarray(ref[0] if isinstance(ref, tuple) else ref), got.double().cpu().numpy()


def _check(oracle_lib, kind, eps, w, grid, e0, de, ne, flat=None):
    ref, got = _both(oracle_lib, kind, eps, w, grid, e0, de, ne, flat)
    assert np.isfinite(got).all()
    assert np.abs(ref).max() > 0.0
    err = dos_err(got, ref)
    print(f"[case] err {err:.2e}", flush=True)
    assert err <= 1e-5


def _bands(grid, nb=2, seed=3):
    """Random energies in [0, 1] that no two points share, and positive weights."""
    rng = np.random.default_rng(seed)
    nk = int(np.prod(grid))
    eps = np.stack([rng.permutation(nk) for _ in range(nb)]).astype(np.float32) / np.float32(nk)
    return eps, rng.random((nb, 3, nk)).astype(np.float32)


# pairs of neighbours with one energy and the point without one that their only tetrahedron of the first tile has
TIED = [((0, 0, 0), (1, 0, 0), (0, 1, 0)), ((0, 0, 0), (0, 0, 1), (1, 0, 1)), ((0, 0, 0), (0, 1, 0), (1, 0, 0))]


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("kind", KINDS)
def test_tie_beside_a_point_without_energy(oracle_lib, kind, bad):
    grid, ne = (16, 16, 16), 120
    for a, b, c in TIED:
        eps, w = _bands(grid)
        cube = eps.reshape(2, *grid)
        cube[:, b[0], b[1], b[2]] = cube[:, a[0], a[1], a[2]]
        for x in range(2):  # the whole neighbourhood but the pair
            for y in range(2):
                for z in range(2):
                    if (x, y, z) not in (a, b) and ((x, y, z) == c or bad == np.inf):
                        cube[:, x, y, z] = bad
        print(f"[case] {kind} {bad} {a} {b}", flush=True)
        _check(oracle_lib, kind, eps, w, grid, -0.02, float(np.float32(1.04 / (ne - 1))), ne)


def _flat(some, e, grid=(16, 9, 8), nb=2):
    """Bands around e, all of them flat there or only a block of 4 x 4 x 4 points."""
    eps, w = _bands(grid, nb)
    eps = (np.float32(e) * (np.float32(0.6) + np.float32(0.8) * eps)).astype(np.float32)
    if some:
        eps.reshape(nb, *grid)[:, 2:6, 3:7, 1:5] = e
    else:
        eps[:] = e
    return eps, w, grid


# (e - e0) / de comes out above the whole number that it is for 7 x 4.6875 and 15 x 1.171875
@pytest.mark.parametrize("some", [True, False])
@pytest.mark.parametrize("kind", ["nos", "binned"])
@pytest.mark.parametrize("step,j", [(4.6875, 7), (0.25, 6), (0.3, 4), (1.171875, 15)])
def test_flat_on_an_inner_grid_energy(oracle_lib, kind, some, step, j):
    de = float(np.float32(step))
    e = float(np.float32(j * de))
    eps, w, grid = _flat(some, e)
    print(f"[case] {kind} some={some} de {de} E {e}", flush=True)
    _check(oracle_lib, kind, eps, w, grid, 0.5 * de if kind == "binned" else 0.0, de, 3 * j, flat=e)


@pytest.mark.parametrize("some", [True, False])
@pytest.mark.parametrize("kind", ["nos", "binned"])
@pytest.mark.parametrize("ne", [1, 2, 7])
def test_flat_on_the_last_grid_energy(oracle_lib, kind, some, ne):
    """The last energy (the upper edge of the last bin) is exactly that of the flat tetrahedra: they count there."""
    de, e = 0.25, 2.0
    eps, w, grid = _flat(some, e)
    eps = np.maximum(eps, np.float32(e)) if some else eps  # nothing below it, so that nothing else hides them
    e0 = e - (ne - 1) * de - (0.5 * de if kind == "binned" else 0.0)
    print(f"[case] {kind} some={some} ne {ne}", flush=True)
    _check(oracle_lib, kind, eps, w, grid, e0, de, ne, flat=e)


@pytest.mark.parametrize("kind", KINDS)
def test_a_point_far_off_the_others(oracle_lib, kind):
    """One energy of another scale on a tile's first point does not coarsen the search for nearly equal energies."""
    grid, ne = (16, 16, 16), 1000
    eps, w = _bands(grid)
    cube = eps.reshape(2, *grid)
    # neighbours one step of FP32 apart, on either side of where their difference from 3000 rounds up
    low = np.float32((4 * np.arange(2 * 4 * 4 * 4).reshape(2, 4, 4, 4) % 2048 * 4 + 1) / 8192)
    cube[:, 1::4, 1::4, 1::4] = low
    cube[:, 1::4, 1::4, 2::4] = np.nextafter(low, np.float32(2.0))
    for far in (3.0e3, 1.0e30):
        cube[:, ::8, ::8, ::8] = far
        print(f"[case] {kind} {far}", flush=True)
        _check(oracle_lib, kind, eps, w, grid, -0.02, float(np.float32(1.04 / (ne - 1))), ne)


@pytest.mark.parametrize("kind", ["dos", "nos", "binned", "chi"])
def test_a_weight_that_is_no_number_adds_nothing(oracle_lib, kind):
    """It takes its tetrahedra out of its own orbital and leaves the others alone."""
    import torch
    import paper_1710_10789_amd as tetra

    grid, nb, ne = (12, 9, 8), 3, 90
    eps, w = synth.band_structure(nb, 10, grid)
    w = np.abs(w) + np.float32(0.05)
    bad, orb = 3 * 72 + 5 * 8 + 4, 1
    gone = eps.copy()
    gone[1, bad] = np.nan
    lo, hi = float(eps.min()), float(eps.max())
    e0, de = float(np.float32(lo - 0.01)), float(np.float32((hi - lo) * 1.05 / (ne - 1)))
    if kind == "chi":
        ef, q = float(np.float32(np.median(eps))), (4, 2, 0)
        f = lambda e, b: oracle_lib.chi(e, b, grid, q, ef, 0.0, de, ne)  # noqa: E731
    else:
        name = {"dos": "dos", "nos": "nos", "binned": "dos_binned"}[kind]
        f = lambda e, b: getattr(oracle_lib, name)(e, b, grid, e0, de, ne)  # noqa: E731
    ref, without = (r[0] if isinstance(r, tuple) else r for r in (f(eps, w), f(gone, w)))
    ref[:, orb] = without[:, orb]
    w[1, orb, bad] = np.nan
    te, tw = torch.from_numpy(eps).cuda(), torch.from_numpy(w).cuda()
    if kind == "chi":
        got = tetra.chi_spectral(te, tw, grid, q, ef, 0.0, de, ne)
    else:
        got = {"dos": tetra.dos_forward, "nos": tetra.nos_forward, "binned": tetra.dos_binned}[kind](te, tw, grid, e0, de, ne)
    got = got.double().cpu().numpy()
    assert np.isfinite(got).all()
    err = dos_err(got, ref)
    print(f"[case] {kind} err {err:.2e}", flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("tile", range(1, 6))
def test_tile_ids_take_the_same_tiles(tile):
    """The forward's tiles are the same for every id: so are the exact mode's sums, bit for bit."""
    import torch
    import paper_1710_10789_amd as tetra

    grid, ne = (17, 16, 24), 700
    eps, w = (torch.from_numpy(x).cuda() for x in _bands(grid))
    args = (eps, w, grid, -0.02, float(np.float32(1.04 / (ne - 1))), ne)
    ref = tetra.dos_forward(*args, deterministic=True)
    assert torch.equal(ref, tetra.dos_forward(*args, deterministic=True, tile=tile))


LATTICES = {  # bands with equal energies by symmetry, some of a tile's tetrahedra or all of them
    "cubic": lambda x, y, z: np.cos(x) + np.cos(y) + np.cos(z),
    "fcc": lambda x, y, z: np.cos(x) + np.cos(y) + np.cos(z) + np.cos(x - y) + np.cos(y - z) + np.cos(z - x),
    "layers": lambda x, y, z: np.cos(x) + np.cos(y) + 0.3 * np.cos(x + y) + 0.0 * z,
    "columns": lambda x, y, z: np.cos(x) + 0.0 * y + 0.0 * z,
}


@pytest.mark.parametrize("grid,norb,ne", [((16, 16, 16), 3, 60), ((9, 17, 8), 9, 700), ((10, 10, 6), 16, 3000),
                                          ((8, 24, 1), 2, 90), ((1, 1, 50), 5, 300)])
@pytest.mark.parametrize("name", sorted(LATTICES))
@pytest.mark.parametrize("kind", KINDS)
def test_equal_energies_by_symmetry(oracle_lib, kind, name, grid, norb, ne):
    """More tetrahedra than the queue holds, all of them, in tiles shorter than eight cubes, with the orbitals in groups
    and with energy ranges beyond the histogram."""
    k = np.meshgrid(*[2 * np.pi * np.arange(n) / n for n in grid], indexing="ij")
    e = LATTICES[name](*k).reshape(-1)
    eps = np.stack([e, 0.7 * e + 0.2]).astype(np.float32)
    w = np.random.default_rng(9).random((2, norb, e.size)).astype(np.float32)
    lo, hi = float(eps.min()), float(eps.max())
    de = float(np.float32(1.0371 * (hi - lo) / (ne - 1)))  # no energy of the band on a grid energy
    print(f"[case] {kind} {name} {grid} {norb} {ne}", flush=True)
    ref, got = _both(oracle_lib, kind, eps, w, grid, float(np.float32(lo - 0.0173 * (hi - lo))), de, ne, None)
    assert np.isfinite(got).all()
    err = dos_err(got, ref)
    print(f"[case] err {err:.2e}", flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("grid,norb,ne", [((16, 16, 16), 3, 60), ((9, 17, 8), 9, 700), ((10, 10, 6), 16, 3000),
                                          ((8, 24, 1), 2, 90), ((1, 1, 50), 5, 300)])
@pytest.mark.parametrize("name", sorted(LATTICES))
def test_susceptibility_of_equal_energies(oracle_lib, name, grid, norb, ne):
    """The same for the differences of two bands, with transitions of both signs."""
    import torch
    import paper_1710_10789_amd as tetra

    k = np.meshgrid(*[2 * np.pi * np.arange(n) / n for n in grid], indexing="ij")
    e = LATTICES[name](*k).reshape(-1)
    eps = np.stack([e, 0.7 * e + 0.2]).astype(np.float32)
    w = np.random.default_rng(9).random((2, norb, e.size)).astype(np.float32)
    wide = float(eps.max() - eps.min())
    ef, q = float(np.float32(0.0613)), (grid[0] // 3, grid[1] // 4, grid[2] // 5)
    de = float(np.float32(2.0371 * wide / (ne - 1)))
    w0 = float(np.float32(-1.0119 * wide))
    print(f"[case] {name} {grid} {norb} {ne}", flush=True)
    ref, _ = oracle_lib.chi(eps, w, grid, q, ef, w0, de, ne)
    got = tetra.chi_spectral(torch.from_numpy(eps).cuda(), torch.from_numpy(w).cuda(), grid, q, ef, w0, de, ne)
    err = dos_err(got.double().cpu().numpy(), ref)
    print(f"[case] err {err:.2e}", flush=True)
    assert err <= 1e-5


# grid, orbitals and energies on either side of the rule for calls with few of them (33^2 = 1089: up to 5 energies, 9
# with more than 8 orbitals, in the exact mode 27 and 19), signed weights, a last tile of one cube
FEW = [("dos", (33, 33, 33), 7, 5), ("dos", (33, 33, 33), 7, 6), ("dos", (36, 29, 33), 16, 9), ("dos", (1, 70, 1), 3, 500),
       ("exact", (33, 33, 33), 7, 27), ("exact", (33, 33, 33), 7, 28), ("exact", (36, 29, 33), 16, 19),
       ("exact", (36, 29, 33), 16, 20), ("exact", (1, 70, 1), 3, 500)]


@pytest.mark.parametrize("kind,grid,norb,ne", FEW)
@pytest.mark.parametrize("storage", ["f32", "signed", "f16", "c64"])
def test_few_energies(oracle_lib, kind, grid, norb, ne, storage):
    import torch
    import paper_1710_10789_amd as tetra

    rng = np.random.default_rng(ne)
    nk = int(np.prod(grid))
    k = np.meshgrid(*[2 * np.pi * np.arange(n) / n for n in grid], indexing="ij")
    e = (np.cos(k[0] + 0.2) + 0.9 * np.cos(k[1] + 0.3 * k[0]) + 0.8 * np.cos(k[2] - k[1])).reshape(-1)
    eps = np.stack([e, 0.6 * e + 0.3 * np.cos(k[2]).reshape(-1)]).astype(np.float32)
    w = rng.random((2, norb, nk)).astype(np.float32) - np.float32(0.4 if storage == "signed" else 0.0)
    scale = None
    tw = torch.from_numpy(w).cuda()
    if storage == "f16":
        tw, scale = tetra.half_weights(tw)
        w = (tw.float() * scale[:, None, None]).cpu().numpy()
    elif storage == "c64":
        tw = torch.polar(tw.sqrt(), tw)
        w = (tw.real.double() ** 2 + tw.imag.double() ** 2).float().cpu().numpy()
    lo, hi = float(eps.min()), float(eps.max())
    e0, de = float(np.float32(lo + 0.01)), float(np.float32((hi - lo) / ne))
    print(f"[case] {kind} {grid} {norb} {ne} {storage}", flush=True)
    call = lambda: tetra.dos_forward(torch.from_numpy(eps).cuda(), tw, grid, e0, de, ne, w_scale=scale,  # noqa: E731
                                     deterministic=kind == "exact")
    got = call()
    if kind == "exact":
        assert torch.equal(got, call())
    ref, _ = oracle_lib.dos(eps, w, grid, e0, de, ne)
    err = dos_err(got.double().cpu().numpy(), ref)
    print(f"[case] err {err:.2e}", flush=True)
    assert err <= 1e-5
