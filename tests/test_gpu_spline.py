"""The kernels in the spline form (tetra_spline.h), through the C ABI, where their routes change: tiles of seven to
nine cubes a side and a last one of a single cube, energy ranges that take the orbitals in groups or leave the
histogram (summed energy by energy), equal corner energies, few (the queue of degenerate tetrahedra) and everywhere
(a grid of one point along an axis), energy grids that start inside or above the bands, both signs of the
susceptibility in one tile. Against the FP64 oracle, gate 1e-5 of the largest value (FP32 energies and additions)."""
import numpy as np
import pytest

import synth
from gates import dos_err

pytestmark = pytest.mark.gpu

CASES = {  # grid, bands = orbitals, energies, first energy and range in units of the band width from its bottom
    "edge_7_8_9": ((7, 8, 9), 5, 90, -0.02, 1.04),
    "edge_17_1": ((17, 16, 8), 1, 150, -0.02, 1.04),
    "groups": ((9, 8, 8), 16, 1500, -0.02, 1.04),
    "long": ((8, 8, 8), 2, 12000, -0.02, 1.04),
    "tied": ((10, 9, 8), 3, 120, -0.02, 1.04),
    "flat": ((20, 18, 1), 3, 100, -0.02, 1.04),
    "inside": ((12, 9, 8), 4, 120, 0.45, 0.3),
    "above": ((9, 8, 10), 2, 50, 1.1, 0.2),
}


def _model(name):
    grid, nb, ne, first, width = CASES[name]
    eps, w = synth.band_structure(nb, 7 + nb, grid)
    if name == "tied":
        cube = eps.reshape(nb, *grid)
        cube[:, 2:5, 3:5, 1:4] = np.round(cube[:, 2:5, 3:5, 1:4] * 8) / 8
    lo, hi = float(eps.min()), float(eps.max())
    de = float(np.float32(width * (hi - lo) / (ne - 1)))
    return grid, nb, ne, eps, w, float(np.float32(lo + first * (hi - lo))), de


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("kind", ["dos", "exact", "batched", "nos", "binned", "chi"])
def test_routes(oracle_lib, kind, name):
    import torch
    import paper_1710_10789_amd as tetra

    grid, nb, ne, eps, w, e0, de = _model(name)
    te, tw = torch.from_numpy(eps).cuda(), torch.from_numpy(w).cuda()
    args = (te, tw, grid, e0, de, ne)
    print(f"[case] {kind} {name}", flush=True)
    if kind == "chi":
        ef, q = float(np.float32(np.median(eps))), (grid[0] // 3, 2, 0)
        e0 = float(np.float32(-0.5 * de * (ne - 1))) if name != "above" else e0  # both signs of the transfer energy
        ref, _ = oracle_lib.chi(eps, w, grid, q, ef, e0, de, ne)
        got = tetra.chi_spectral(te, tw, grid, q, ef, e0, de, ne)
    elif kind == "nos":
        ref, got = oracle_lib.nos(eps, w, grid, e0, de, ne), tetra.nos_forward(*args)
    elif kind == "binned":
        ref, got = oracle_lib.dos_binned(eps, w, grid, e0, de, ne), tetra.dos_binned(*args)
    else:
        ref = oracle_lib.dos(eps, w, grid, e0, de, ne)
        if kind == "batched":
            got = tetra.dos_batched([args + (None,), args + (None,)])[1]
        else:
            got = tetra.dos_forward(*args, deterministic=kind == "exact")
            if kind == "exact":
                assert torch.equal(got, tetra.dos_forward(*args, deterministic=True))
    ref = np.asarray(ref[0] if isinstance(ref, tuple) else ref)
    got = got.double().cpu().numpy()
    if np.abs(ref).max() == 0.0:
        assert not got.any()
    else:
        err = dos_err(got, ref)
        print(f"[case] err {err:.2e}", flush=True)
        assert err <= 1e-5
