"""The work that users of this package have it do, as cases that can be timed and checked.

A case is a dict of plain values: ``kind`` names the entry point, the rest its sizes and options.

* Inputs: a seeded random tight-binding model (a Hermitian on-site matrix with levels in [-2, 2] eV and
  complex Gaussian hoppings to nearest and in-plane diagonal neighbours), diagonalised on every point
  of a periodic k-grid: ascending band energies and the orbital weights |a|^2 (or the amplitudes a).
  Neighbouring points therefore have nearby energies, bands cross and avoid each other, and the weights
  of a band sum to one where every orbital is kept.
* Energy grids: uniform, over ``span`` times the range of the bands, centred on it (1.2: the whole band
  range with 10 % on either side; below one: a part of it, for a closer look). Susceptibilities: from
  zero to ``span`` times the band width, the Fermi energy at half filling.
* ``exact`` forms the same results in FP64 with torch alone: sections and clipped volumes of every
  tetrahedron as sums over the triangles and tetrahedra they split into, and autograd for gradients.
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

import paper_1710_10789_amd as tetra

DTYPES = ("f32", "f16", "c64")  # weights as FP32, as FP16 with a scale per band, or as complex amplitudes


def listed():
    return [
        # a quick look at a small model, the sizes of the parity tests: launches and latency
        _case("fwd_small", "forward", (16, 16, 16), 8, 8, 200),
        # the paper's FeSe set-up: a flat grid, eigenvector amplitudes, the five 3d orbitals of eight bands
        _case("fwd_paper", "forward", (60, 60, 10), 8, 5, 1024, dtype="c64"),
        # the headline DOS of the benchmark
        _case("fwd_64", "forward", (64, 64, 64), 8, 8, 1000),
        # the precision workload: many orbitals, many energies, FP16 weights; the largest single DOS
        _case("fwd_96_half", "forward", (96, 96, 96), 16, 16, 2000, dtype="f16"),
        # a bitwise reproducible DOS on a fine energy grid
        _case("fwd_48_exact", "exact", (48, 48, 48), 8, 8, 2000),
        # one step of fitting a model to a DOS: forward, loss, adjoint
        _case("fit_64", "step", (64, 64, 64), 8, 8, 500),
        # the same through eigenvector amplitudes, a small model with ten orbitals
        _case("fit_small_amp", "step", (24, 24, 24), 10, 10, 400, dtype="c64"),
        # the adjoint alone, on a grid whose sides fit no tile
        _case("bwd_ragged", "backward", (50, 42, 34), 8, 8, 1000),
        # orbital filling as a function of the Fermi energy
        _case("nos_64", "nos", (64, 64, 64), 8, 8, 1000),
        # bin averages with bins much narrower than the tetrahedra
        _case("binned_fine", "binned", (24, 24, 24), 8, 8, 4096),
        # susceptibility of the benchmark's model for a transfer in the plane
        _case("chi_64", "chi", (64, 64, 64), 8, 8, 500, span=1.0, q1=16, q2=16, q3=0),
        # models of very different sizes in one call (a scan over parameters)
        _case("batch_12", "batched", (96, 96, 96), 8, 8, 1950, models=12, pick=3),
    ]


def _case(name, kind, grid, nb, norb, ne, dtype="f32", span=1.2, **more):
    c = {"name": name, "kind": kind, "n1": grid[0], "n2": grid[1], "n3": grid[2], "nb": nb, "norb": norb, "ne": ne,
         "dtype": dtype, "span": span, **more}
    if not name:
        del c["name"]
    return c


def draw(rng):
    """One more case: any entry point, sides 5 to 96 (odd ones among them), 1 to 16 bands and orbitals, 32 to
    4096 energies, every storage of the weights, the whole band range or a part of it."""
    kind = rng.choice(["forward", "forward", "forward", "exact", "step", "step", "backward", "nos", "binned", "chi",
                       "batched"])
    top = {"chi": 64, "step": 72, "backward": 72}.get(kind, 96)

    def log_int(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    side = log_int(5, top)
    grid = [min(top, max(5, int(round(side * rng.uniform(0.6, 1.4))))) for _ in range(3)]
    if rng.random() < 0.4:  # the even sides that users type
        grid = [min(top, max(8, 8 * ((g + 4) // 8))) for g in grid]
    norb = rng.choice([1, 3, 5, 6, 8, 8, 10, 16])
    nb = norb if rng.random() < 0.7 else rng.randint(1, 16)
    ne = log_int(32, 4096)
    dtype = rng.choice(["f32", "f32", "f16", "c64"])
    span = 1.2 if rng.random() < 0.75 else rng.choice([0.3, 0.6])
    if kind in ("batched", "chi"):
        dtype = rng.choice(["f32", "f32", "f16"])
    more = {}
    if kind == "chi":
        span = rng.choice([1.0, 0.4])
        more = {"q%d" % (i + 1): rng.randrange(grid[i]) for i in range(3)}
    elif kind == "batched":
        more = {"models": rng.randint(2, 10), "pick": rng.randrange(1000)}
        grid = [max(grid)] * 3
    # no dearer than the largest listed: grid points x (bands, or band pairs) x orbitals, and the
    # (tetrahedron, band, energy) triples, of which a share that falls with the grid's side is in a window
    while True:
        nk = grid[0] * grid[1] * grid[2]
        bands = nb * nb / 4 if kind == "chi" else nb
        if nk * bands * max(norb, 4) <= 1.6e7 and nk ** (2 / 3) * bands * ne * norb <= 4.0e9:
            break
        grid = [max(5, int(0.85 * g)) for g in grid]
    return _case("", kind, grid, nb, norb, ne, dtype=dtype, span=span, **more)


def work(case):
    """Bytes: every input read once, every output written once. Operations: each corner of each
    tetrahedron-band (of each band pair) meets each orbital once."""
    total = {"bytes": 0.0, "flops": 0.0}
    for c in _models(case):
        nk, nb, norb, ne = c["n1"] * c["n2"] * c["n3"], c["nb"], c["norb"], c["ne"]
        wsize = {"f32": 4, "f16": 2, "c64": 8}[c["dtype"]]
        inputs = nk * nb * (4 + norb * wsize) + (4 * nb if c["dtype"] == "f16" else 0)
        outputs = 4 * ne * norb
        corners = 6 * 4 * nk * norb * (nb * nb if c["kind"] == "chi" else nb)
        if c["kind"] in ("step", "backward"):
            outputs = nk * nb * (4 + norb * (8 if c["dtype"] == "c64" else 4))
            inputs += 4 * ne * norb
            total["flops"] += 2.0 * corners  # the adjoint: one product each for the energies and the weights
            if c["kind"] == "step":
                inputs += inputs  # the adjoint needs the whole DOS first: the inputs are read again
                outputs += 4 * ne * norb
        total["bytes"] += inputs + outputs
        total["flops"] += 2.0 * corners
    return total


def prepare(case, seed):
    if case["kind"] == "batched":
        states = [_inputs(c, seed * 1000 + i) for i, c in enumerate(_models(case))]
        problems = [(s["eps"], s["w"], s["grid"], s["e0"], s["de"], s["ne"], s["scale"]) for s in states]
        # a program that scans parameters keeps the workspace
        ws = torch.empty(tetra.batched_workspace_bytes(problems), dtype=torch.uint8, device="cuda")
        return {"kind": "batched", "problems": problems, "ws": ws}
    s = _inputs(case, seed)
    g = torch.Generator().manual_seed(seed * 7 + 1)
    if case["kind"] == "backward":
        s["G"] = torch.randn(case["ne"], case["norb"], generator=g).to(_device())
    if case["kind"] == "step":  # the DOS to fit: of the bands' energy scale, not the model's own
        s["target"] = _target(case, g)
        s["eps"].requires_grad_()
        s["w"].requires_grad_()
    return s


def run(s):
    kind = s["kind"]
    if kind == "batched":
        return tetra.dos_batched(s["problems"], workspace=s["ws"])
    args = (s["eps"], s["w"], s["grid"])
    if kind == "forward":
        return tetra.dos_forward(*args, s["e0"], s["de"], s["ne"], w_scale=s["scale"])
    if kind == "exact":
        return tetra.dos_forward(*args, s["e0"], s["de"], s["ne"], w_scale=s["scale"], deterministic=True)
    if kind == "backward":
        return tetra.dos_backward(*args, s["e0"], s["de"], s["G"], w_scale=s["scale"])
    if kind == "step":
        dos = tetra.dos(*args, s["e0"], s["de"], s["ne"], w_scale=s["scale"])
        loss = (dos - s["target"]).square().sum()
        ge, gw = torch.autograd.grad(loss, (s["eps"], s["w"]))
        return dos.detach(), ge, gw
    if kind == "nos":
        return tetra.nos_forward(*args, s["e0"], s["de"], s["ne"], w_scale=s["scale"])
    if kind == "binned":
        return tetra.dos_binned(*args, s["e0"], s["de"], s["ne"], w_scale=s["scale"])
    return tetra.chi_spectral(*args, s["q"], s["ef"], s["e0"], s["de"], s["ne"], w_scale=s["scale"])


# ---------------------------------------------------------------------------------------------
# Inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _models(case):
    """The single problems of a case: itself, or the models of a batch (uneven cubic grids and energy grids)."""
    if case["kind"] != "batched":
        return [case]
    r = np.random.default_rng(case["pick"])
    sides = [n for n in (24, 32, 48, 64, 96) if n <= case["n1"]] or [case["n1"]]
    out = []
    for i in range(case["models"]):
        n = int(r.choice(sides)) if i else case["n1"]
        ne = int(r.integers(min(256, case["ne"]), case["ne"] + 1))
        out.append({**case, "n1": n, "n2": n, "n3": n, "ne": ne})
    return out


def _inputs(case, seed):
    grid = (case["n1"], case["n2"], case["n3"])
    n = max(case["nb"], case["norb"])
    eps, amp = _bands(n, case["nb"], case["norb"], seed, grid)
    lo, hi = float(eps.min()), float(eps.max())
    s = {"kind": case["kind"], "grid": grid, "ne": case["ne"], "eps": eps, "scale": None}
    if case["kind"] == "chi":
        ef = float(eps.reshape(-1)[:: max(1, eps.numel() // 100003)].median())
        s.update(q=(case["q1"], case["q2"], case["q3"]), ef=float(np.float32(ef)), e0=0.0)
        s["de"] = float(np.float32(max(case["span"] * (hi - lo), 1e-3) / max(case["ne"] - 1, 1)))
    else:
        width = case["span"] * max(hi - lo, 1e-3)
        s["e0"] = float(np.float32(0.5 * (lo + hi) - 0.5 * width))
        s["de"] = float(np.float32(width / max(case["ne"] - 1, 1)))
    if case["dtype"] == "c64":
        s["w"] = amp
    else:
        s["w"] = amp.real.square() + amp.imag.square()
        if case["dtype"] == "f16":
            s["w"], s["scale"] = tetra.half_weights(s["w"])
    return s


def _target(case, g):
    """A smooth DOS on the case's energy grid, about the height of the model's own: a few Gaussians per orbital."""
    x = torch.linspace(-1.2, 1.2, case["ne"], dtype=torch.float64)[:, None, None]
    at = torch.rand(1, case["norb"], 3, generator=g, dtype=torch.float64) * 1.6 - 0.8
    wide = torch.rand(1, case["norb"], 3, generator=g, dtype=torch.float64) * 0.3 + 0.15
    return (0.2 * torch.exp(-((x - at) / wide) ** 2)).sum(2).float().to(_device())


HOPS = ((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, -1, 0))


def _bands(n, nb, norb, seed, grid, sigma=0.3):
    """eps [nb, nk] (FP32, ascending per point) and amplitudes [nb, norb, nk] (complex64) of the seeded model."""
    r = np.random.default_rng(seed)

    def gauss():
        return (r.standard_normal((n, n)) + 1j * r.standard_normal((n, n))) * (sigma / math.sqrt(2))

    a = gauss()
    t0 = (a + a.conj().T) / 2 + np.diag(r.uniform(-2.0, 2.0, n))
    hops = [(R, gauss()) for R in HOPS]
    nk = grid[0] * grid[1] * grid[2]
    dev = _device()
    eps = torch.empty(nb, nk, dtype=torch.float32, device=dev)
    amp = torch.empty(nb, norb, nk, dtype=torch.complex64, device=dev)
    chunk = max(4096, 8_000_000 // (n * n))
    for lo in range(0, nk, chunk):
        k = torch.arange(lo, min(nk, lo + chunk), device=dev)
        kf = (k // (grid[1] * grid[2]) / grid[0], (k // grid[2]) % grid[1] / grid[1], k % grid[2] / grid[2])
        h = torch.tensor(t0, dtype=torch.complex64, device=dev)[:, :, None].repeat(1, 1, k.numel())
        for R, t in hops:
            ph = 2 * math.pi * (kf[0] * R[0] + kf[1] * R[1] + kf[2] * R[2])
            half = torch.tensor(t, dtype=torch.complex64, device=dev)[:, :, None] * torch.polar(torch.ones_like(ph), ph)
            h += half + half.conj().transpose(0, 1)
        e, v = _eigh(h)
        eps[:, lo:lo + chunk] = e[:nb]
        amp[:, :, lo:lo + chunk] = v[:norb, :nb].transpose(0, 1)
    return eps, amp


def _eigh(h):
    """Ascending eigenvalues [n, K] and eigenvectors [n, n, K] (columns) of Hermitian h [n, n, K]: cyclic Jacobi,
    disjoint pairs of a round-robin tournament at once, every matrix of the batch alongside the others."""
    n = h.shape[0]
    v = torch.eye(n, dtype=h.dtype, device=h.device)[:, :, None].repeat(1, 1, h.shape[2])
    players = list(range(n + n % 2))
    for _ in range(6 if n <= 8 else 7):
        for _ in range(len(players) - 1):
            half = len(players) // 2
            pairs = [(min(a, b), max(a, b)) for a, b in zip(players[:half], reversed(players[half:])) if max(a, b) < n]
            players = [players[0], players[-1]] + players[1:-1]
            if not pairs:
                continue
            p, q = (torch.tensor(x, device=h.device) for x in zip(*pairs))
            apq = h[p, q]
            mod = apq.abs()
            phase = torch.where(mod > 0, apq / mod.clamp_min(1e-30), torch.ones_like(apq))
            tau = (h[q, q].real - h[p, p].real) / (2 * mod.clamp_min(1e-30))
            t = torch.where(tau >= 0, 1.0, -1.0) / (tau.abs() + torch.sqrt(1 + tau * tau))
            t = torch.where(mod > 0, t, torch.zeros_like(t))
            c = torch.rsqrt(1 + t * t)
            s, c = (t * c) * phase, c[:, None].to(h.dtype)
            s = s[:, None]
            a, b = h[p], h[q]  # rows
            h[p], h[q] = c * a - s * b, s.conj() * a + c * b
            hv = torch.cat((h, v))  # columns of both
            a, b = hv[:, p].transpose(0, 1), hv[:, q].transpose(0, 1)
            hv[:, p] = (c * a - s.conj() * b).transpose(0, 1)
            hv[:, q] = (s * a + c * b).transpose(0, 1)
            h, v = hv[:n], hv[n:]
    e, order = torch.diagonal(h).real.T.sort(0)
    return e, torch.gather(v, 1, order[None].expand(n, n, -1))


# ---------------------------------------------------------------------------------------------
# The same in FP64 with torch alone

# Corner offsets of a cube by slot (bits 0, 1, 2: axes 1, 2, 3) and its six tetrahedra (Table I of the paper, less one)
TETS = ((0, 1, 2, 5), (1, 2, 3, 5), (0, 2, 4, 5), (2, 3, 5, 7), (2, 4, 5, 6), (2, 5, 6, 7))


def exact(case, seed):
    if case["kind"] == "batched":
        return [_exact_one({**c, "kind": "forward"}, seed * 1000 + i) for i, c in enumerate(_models(case))]
    return _exact_one(case, seed)


def _exact_one(case, seed):
    if case["ne"] * case["norb"] > 2_000_000:
        return None
    s = prepare(case, seed)
    eps = s["eps"].detach().double()
    w = s["w"].detach()
    if case["dtype"] == "c64":
        b = w.real.double() ** 2 + w.imag.double() ** 2
    else:
        b = w.double() * (s["scale"].double()[:, None, None] if s["scale"] is not None else 1.0)
    g = _Grid(s["grid"], s["e0"], s["de"], s["ne"])
    if case["kind"] == "chi":
        return g.chi(eps, b, s["q"], s["ef"])
    if case["kind"] in ("nos", "binned"):
        return g.states(eps, b, case["kind"] == "binned")
    if case["kind"] in ("forward", "exact"):
        return g.dos(eps, b)
    if case["kind"] == "backward":
        dos, G = None, s["G"].double()
    else:
        dos = g.dos(eps, b)
        G = 2.0 * (dos - s["target"].double())
    ge, gb = g.gradients(eps, b, G)
    if case["dtype"] == "c64":
        gw = 2.0 * torch.complex(w.real.double() * gb, w.imag.double() * gb)
    elif case["dtype"] == "f16" and case["kind"] == "step":  # of the stored values
        gw = gb * s["scale"].double()[:, None, None]
    else:
        gw = gb
    return (ge, gw) if dos is None else (dos, ge, gw)


class _Grid:
    """Sums over the tetrahedra of a periodic grid at E_j = e0 + j de, in FP64."""

    def __init__(self, grid, e0, de, ne):
        self.grid, self.e0, self.de, self.ne = grid, e0, de, ne
        self.vol = 1.0 / (6.0 * grid[0] * grid[1] * grid[2])

    def corners(self, x, t):
        """x [..., nk] at the four corners of tetrahedron t of every cube: [nk, 4, ...]."""
        y = x.reshape(x.shape[:-1] + tuple(self.grid))
        at = [torch.roll(y, [-(s & 1), -(s >> 1 & 1), -(s >> 2)], (-3, -2, -1)).reshape(x.shape) for s in TETS[t]]
        return torch.stack(at, -1).movedim((-2, -1), (0, 1))

    def chunks(self, e, steps):
        """Ranges of the tetrahedra e [N, 4] (ascending) with at most `steps` energies in their windows each."""
        j0, j1 = self.window(e)
        total = torch.cumsum((j1 - j0 + 2).clamp_min(0), 0)
        lo, n = 0, e.shape[0]
        while lo < n:
            base = int(total[lo - 1]) if lo else 0
            hi = max(lo + 1, int(torch.searchsorted(total, torch.tensor(base + steps, device=total.device), right=True)))
            yield slice(lo, min(hi, n))
            lo = hi

    def window(self, e, shift=0.0):
        """First and last j with E1 < E_j < E4."""
        big = self.ne + 2.0
        j0 = torch.floor(((e[:, 0] - self.e0) / self.de - shift).clamp(-2.0, big)).long() - 1
        j1 = torch.ceil(((e[:, 3] - self.e0) / self.de - shift).clamp(-2.0, big)).long() + 1
        at = lambda j: self.e0 + (j.double() + shift) * self.de  # noqa: E731
        for _ in range(3):
            j0 = torch.where(at(j0) <= e[:, 0], j0 + 1, j0)
            j1 = torch.where(at(j1) >= e[:, 3], j1 - 1, j1)
        return j0.clamp_min(0), j1.clamp_max(self.ne - 1)

    def updates(self, e):
        """(tetrahedron, j) of every energy inside a window."""
        j0, j1 = self.window(e.detach())
        count = (j1 - j0 + 1).clamp_min(0)
        tet = torch.repeat_interleave(torch.arange(e.shape[0], device=e.device), count)
        j = torch.arange(tet.numel(), device=e.device) - (torch.cumsum(count, 0) - count)[tet] + j0[tet]
        return tet, j

    def density(self, e, b, vol, tet, j):
        """sum_l b_l dw_l/dE at E_j of tetrahedron `tet`: [len(tet), norb]; the three kinds of section apart."""
        E = self.e0 + j.double() * self.de
        out, where = [], []
        for kind in range(3):
            e_ = e.detach()[tet]
            sel = (E <= e_[:, 1], (E > e_[:, 1]) & (E <= e_[:, 2]), E > e_[:, 2])[kind]
            i = sel.nonzero()[:, 0]
            if not i.numel():
                continue
            et, bt, v = e.index_select(0, tet[i]), b.index_select(0, tet[i]), vol[tet[i]]
            e1, e2, e3, e4 = et.unbind(1)
            b1, b2, b3, b4 = bt.unbind(1)
            f = lambda lo, hi: (E[i] - lo) / (hi - lo)  # noqa: E731  where E cuts the edge lo-hi
            on = lambda r, lo, hi: lo + r[:, None] * (hi - lo)  # noqa: E731
            if kind == 0:  # a triangle on the edges of corner 1
                r2, r3, r4 = f(e1, e2), f(e1, e3), f(e1, e4)
                d = v * r2 * r3 / (e4 - e1)
                val = d[:, None] * (on(r2, b1, b2) + on(r3, b1, b3) + on(r4, b1, b4))
            elif kind == 2:  # a triangle on the edges of corner 4
                r1, r2, r3 = 1 - f(e1, e4), 1 - f(e2, e4), 1 - f(e3, e4)
                d = v * r2 * r3 / (e4 - e1)
                val = d[:, None] * (on(r1, b4, b1) + on(r2, b4, b2) + on(r3, b4, b3))
            else:  # a quadrilateral: two triangles that share the side from edge 13 to edge 24
                r13, r14, r23, r24 = f(e1, e3), f(e1, e4), f(e2, e3), f(e2, e4)
                p13, p14, p23, p24 = on(r13, b1, b3), on(r14, b1, b4), on(r23, b2, b3), on(r24, b2, b4)
                d1 = v * r14 * (1 - r24) / (e3 - e1)
                d2 = v * r24 * (1 - r23) / (e3 - e1)
                val = d1[:, None] * (p13 + p14 + p24) + d2[:, None] * (p13 + p24 + p23)
            out.append(val)
            where.append(i)
        return out, where

    def add_density(self, e, b, vol, out):
        e, order = e.sort(1)
        b = torch.gather(b, 1, order[:, :, None].expand_as(b))
        for part in self.chunks(e, 4_000_000 // max(4, b.shape[2])):
            tet, j = self.updates(e[part])
            if tet.numel():
                for val, i in zip(*self.density(e[part], b[part], vol[part], tet, j)):
                    out.index_add_(0, j[i], val)

    def dos(self, eps, b):
        out = torch.zeros(self.ne, b.shape[1], dtype=torch.float64, device=eps.device)
        vol = torch.full((eps.shape[1],), self.vol, dtype=torch.float64, device=eps.device)
        for n, t in itertools.product(range(eps.shape[0]), range(6)):
            self.add_density(self.corners(eps[n], t), self.corners(b[n], t).contiguous(), vol, out)
        return out

    def gradients(self, eps, b, G):
        ge, gb = torch.zeros_like(eps), torch.zeros_like(b)
        nk = eps.shape[1]
        k = torch.arange(nk, device=eps.device).double()
        vol = torch.full((nk,), self.vol, dtype=torch.float64, device=eps.device)
        for t in range(6):
            at = self.corners(k, t).long()
            for n in range(eps.shape[0]):
                e0, b0 = self.corners(eps[n], t), self.corners(b[n], t).contiguous()
                e0, order = e0.sort(1)
                b0 = torch.gather(b0, 1, order[:, :, None].expand_as(b0))
                points = torch.gather(at, 1, order)
                for part in self.chunks(e0, 3_000_000 // max(4, b.shape[1])):
                    e, bb = e0[part].requires_grad_(), b0[part].requires_grad_()
                    tet, j = self.updates(e)
                    if not tet.numel():
                        continue
                    loss = sum((val * G[j[i]]).sum() for val, i in zip(*self.density(e, bb, vol[part], tet, j)))
                    if not torch.is_tensor(loss):
                        continue
                    de, db = torch.autograd.grad(loss, (e, bb))
                    ge[n].index_add_(0, points[part].reshape(-1), de.reshape(-1))
                    gb[n].index_add_(1, points[part].reshape(-1), db.reshape(-1, b.shape[1]).T.contiguous())
        return ge, gb

    def volume(self, e, b, E):
        """int b over the part of a tetrahedron (unit volume, e ascending) below E, for E1 < E < E4: [n, norb]."""
        out = torch.empty(b.shape[0], b.shape[2], dtype=torch.float64, device=b.device)
        kinds = (E <= e[:, 1], (E > e[:, 1]) & (E <= e[:, 2]), E > e[:, 2])
        for kind, sel in enumerate(kinds):
            i = sel.nonzero()[:, 0]
            e1, e2, e3, e4 = e[i].unbind(1)
            b1, b2, b3, b4 = b[i].unbind(1)
            f = lambda lo, hi: (E[i] - lo) / (hi - lo)  # noqa: E731
            on = lambda r, lo, hi: lo + r[:, None] * (hi - lo)  # noqa: E731
            if kind == 0:
                r2, r3, r4 = f(e1, e2), f(e1, e3), f(e1, e4)
                out[i] = (r2 * r3 * r4 / 4)[:, None] * (b1 + on(r2, b1, b2) + on(r3, b1, b3) + on(r4, b1, b4))
            elif kind == 2:
                r1, r2, r3 = 1 - f(e1, e4), 1 - f(e2, e4), 1 - f(e3, e4)
                above = (r1 * r2 * r3 / 4)[:, None] * (b4 + on(r1, b4, b1) + on(r2, b4, b2) + on(r3, b4, b3))
                out[i] = (b1 + b2 + b3 + b4) / 4 - above
            else:
                r13, r14, r23, r24 = f(e1, e3), f(e1, e4), f(e2, e3), f(e2, e4)
                p13, p14, p23, p24 = on(r13, b1, b3), on(r14, b1, b4), on(r23, b2, b3), on(r24, b2, b4)
                out[i] = ((r13 * r14 * (1 - r24) / 4)[:, None] * (b1 + p13 + p14 + p24)
                          + (r13 * r24 * (1 - r23) / 4)[:, None] * (b1 + p13 + p24 + p23)
                          + (r23 * r24 / 4)[:, None] * (b1 + b2 + p23 + p24))
        return out

    def states(self, eps, b, binned):
        """Number of states at E_j, or its difference quotient over the bins of width de around them."""
        shift, ne = (-0.5, self.ne + 1) if binned else (0.0, self.ne)
        grid = _Grid(self.grid, self.e0 + shift * self.de, self.de, ne)
        inside = torch.zeros(ne, b.shape[1], dtype=torch.float64, device=eps.device)
        above = torch.zeros(ne + 1, b.shape[1], dtype=torch.float64, device=eps.device)
        for n, t in itertools.product(range(eps.shape[0]), range(6)):
            e, order = self.corners(eps[n], t).sort(1)
            bb = self.corners(b[n], t)
            bb = torch.gather(bb, 1, order[:, :, None].expand_as(bb))
            full = torch.ceil(((e[:, 3] - grid.e0) / grid.de).clamp(-2.0, ne + 2.0)).long() - 1
            for _ in range(3):
                full = torch.where(grid.e0 + full.double() * grid.de < e[:, 3], full + 1, full)
            above.index_add_(0, full.clamp(0, ne), self.vol * bb.mean(1))
            for part in grid.chunks(e, 4_000_000 // max(4, b.shape[1])):
                tet, j = grid.updates(e[part])
                if tet.numel():
                    E = grid.e0 + j.double() * grid.de
                    inside.index_add_(0, j, self.vol * grid.volume(e[part][tet], bb[part][tet], E))
        total = inside + torch.cumsum(above, 0)[:ne]
        return (total[1:] - total[:-1]) / self.de if binned else total

    def chi(self, eps, b, q, ef):
        out = torch.zeros(self.ne, b.shape[1], dtype=torch.float64, device=eps.device)
        shifted = lambda x: torch.roll(x.reshape(x.shape[:-1] + tuple(self.grid)),  # noqa: E731
                                       [-q[0], -q[1], -q[2]], (-3, -2, -1)).reshape(x.shape)
        eq, bq = shifted(eps), shifted(b)
        for n, m in itertools.product(range(eps.shape[0]), repeat=2):
            if not (eps[n].min() <= ef <= eq[m].max() or eq[m].min() <= ef <= eps[n].max()):
                continue
            weight = b[n] * bq[m]
            for t in range(6):
                e, ep = self.corners(eps[n], t), self.corners(eq[m], t)
                for sign in (1.0, -1.0):
                    f1, f2 = sign * (e - ef), sign * (ef - ep)  # both <= 0 inside
                    some = ((f1 <= 0).any(1) & (f2 <= 0).any(1)).nonzero()[:, 0]
                    if some.numel():
                        W = self.corners(weight, t)[some]
                        data = torch.cat((f1[some][:, :, None], f2[some][:, :, None], (ep - e)[some][:, :, None], W), 2)
                        vol = torch.full((some.numel(),), sign * self.vol, dtype=torch.float64, device=eps.device)
                        for plane in (0, 1):
                            data, vol = self.clip(data, vol, plane)
                        if vol.numel():
                            self.add_density(data[:, :, 2].contiguous(), data[:, :, 3:].contiguous(), vol, out)
        return out

    @staticmethod
    def clip(data, vol, plane):
        """The part of the tetrahedra with data[..., plane] <= 0, as tetrahedra (vertex data [N, 4, C], volumes)."""
        f, order = data[:, :, plane].sort(1)
        data = torch.gather(data, 1, order[:, :, None].expand_as(data))
        inside = (f <= 0).sum(1)
        keep, vols = [data[inside == 4]], [vol[inside == 4]]
        for k in (1, 2, 3):
            d, v = data[inside == k], vol[inside == k]
            if not v.numel():
                continue
            z = d[:, :, plane]

            def cut(i, o):  # the point of the edge from inside i to outside o on the plane
                r = (z[:, i] / (z[:, i] - z[:, o])).nan_to_num(0.0)
                return r, d[:, i] + r[:, None] * (d[:, o] - d[:, i])

            if k == 1:
                (r1, p1), (r2, p2), (r3, p3) = cut(0, 1), cut(0, 2), cut(0, 3)
                parts = [((d[:, 0], p1, p2, p3), r1 * r2 * r3)]
            elif k == 2:
                (r02, p02), (r03, p03), (r12, p12), (r13, p13) = cut(0, 2), cut(0, 3), cut(1, 2), cut(1, 3)
                parts = [((d[:, 0], p02, p03, p13), r02 * r03 * (1 - r13)),
                         ((d[:, 0], p02, p13, p12), r02 * r13 * (1 - r12)),
                         ((d[:, 0], d[:, 1], p12, p13), r12 * r13)]
            else:  # all but the corner tetrahedron at 3, a prism
                (r0, p0), (r1, p1), (r2, p2) = cut(0, 3), cut(1, 3), cut(2, 3)
                parts = [((d[:, 0], d[:, 1], d[:, 2], p2), r2),
                         ((d[:, 0], d[:, 1], p1, p2), r1 * (1 - r2)),
                         ((d[:, 0], p0, p1, p2), r0 * (1 - r1) * (1 - r2))]
            for corners, share in parts:
                keep.append(torch.stack(corners, 1))
                vols.append(v * share)
        data, vol = torch.cat(keep), torch.cat(vols)
        some = vol != 0
        return data[some], vol[some]
