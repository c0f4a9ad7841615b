"""The susceptibility on a grid with more units than one launch may hold: a line of 2^27 points with a band that crosses
E_F in 4096 points near its end, below E_F elsewhere, adds what the same 4096 points add on a line of 8192. Against the
FP64 oracle on these, gate 1e-5 of the largest value (FP32 energies and additions; a few hundred workgroups add)."""
import numpy as np
import pytest

from gates import dos_err

pytestmark = pytest.mark.gpu


def test_more_units_than_one_launch_holds(oracle_lib):
    import torch
    import paper_1710_10789_amd as tetra

    n, m, p, ne, q = 1 << 27, 8192, 4096, 40, 13
    k = 2 * np.pi * np.arange(p) / 64
    band = np.cos(k) + 0.3 * np.cos(2 * k + 0.4) + 0.1 * np.cos(k / 37)
    weight = 0.6 + 0.3 * np.cos(k + 1.0)
    de = float(np.float32(2.9 / ne))

    def line(total):
        eps = torch.full((1, total), -1.5, device="cuda")
        w = torch.full((1, 1, total), 0.5, device="cuda")
        at = total - p - 1000
        eps[0, at:at + p] = torch.from_numpy(band.astype(np.float32)).cuda()
        w[0, 0, at:at + p] = torch.from_numpy(weight.astype(np.float32)).cuda()
        return eps, w

    eps, w = line(m)
    ref, _ = oracle_lib.chi(eps.cpu().numpy(), w.cpu().numpy(), (1, 1, m), (0, 0, q), 0.0617, -1.337, de, ne)
    print(f"[case] {n}", flush=True)
    got = tetra.chi_spectral(*line(n), (1, 1, n), (0, 0, q), 0.0617, -1.337, de, ne)
    err = dos_err(got.double().cpu().numpy() * (n / m), ref)
    print(f"[case] err {err:.2e}", flush=True)
    assert err <= 1e-5
