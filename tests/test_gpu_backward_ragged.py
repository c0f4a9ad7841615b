"""The adjoint on grids that its tiles do not divide, on either side of the rule for shrinking them: few units, many
with short windows, many with long ones, a grid thinner than the tile. Against the FP64 oracle, the gradient gate."""
import numpy as np
import pytest

import synth
from gates import gate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,nb,norb,ne", [((9, 10, 11), 2, 3, 200), ((20, 18, 22), 8, 3, 60), ((20, 18, 22), 8, 3, 700),
                                             ((33, 18, 5), 8, 2, 600)])
def test_ragged_grids(oracle_lib, grid, nb, norb, ne):
    import torch
    import paper_1710_10789_amd as tetra

    eps, _ = synth.band_structure(nb, 5, grid)
    w = np.random.default_rng(nb).random((nb, norb, eps.shape[1])).astype(np.float32)
    e0, de = synth.energy_grid(eps, ne)
    G = np.random.default_rng(ne).normal(size=(ne, norb)).astype(np.float32)
    print(f"[case] {grid} {nb} {norb} {ne}", flush=True)
    ge, gw = tetra.dos_backward(torch.from_numpy(eps).cuda(), torch.from_numpy(w).cuda(), grid, e0, de,
                                torch.from_numpy(G).cuda())
    re, rw = oracle_lib.dos_backward(eps, w, grid, e0, de, G.astype(np.float64))
    for got, ref in ((ge, re), (gw, rw)):
        ok, big, norm = gate(got.cpu().numpy(), ref)
        print(f"[case] {big:.2e} {norm:.2e}", flush=True)
        assert ok
