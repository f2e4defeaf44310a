"""Timing cases of the H/S builder: what a program that sets up FLAPW matrices has it do.

A case names an entry point of `HSBuilder` (or the autograd function), a synthetic cell and a
basis size.  The cells are those of this repository's workloads: orthorhombic boxes of 8 to 30
bohr, 1 to 4 atom types of up to 32 atoms, l_max 4 to 10, bases from some two hundred plane waves
(one formula unit, a quick look) to 12000 (the largest the benchmark sets up).  Positions are
random with non-overlapping muffin tins, radial boundary values and T blocks have the
distributions of the synthetic cells, and the basis holds the N_G shortest k+G of a random k.

`exact` evaluates the paper's formulas in 64-bit torch: matching coefficients, stacked products.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1712_07206_amd import HSB_FP64, HSB_SPLIT_CRT, HSB_SPLIT_CRT_BF16
from paper_1712_07206_amd.autograd import hs_build
from paper_1712_07206_amd.hsbuild import HSBuilder

PRECISION = {"fp64": HSB_FP64, "residue_int8": HSB_SPLIT_CRT, "residue_bf16": HSB_SPLIT_CRT_BF16}
MODULI = 11  # the residue forms' usual number of moduli (about 1e-11 of the FP64 result)

# side lengths (bohr), atoms per type, muffin-tin radii, l_max
CELLS = {
    "tiny": ((8.0, 8.0, 8.0), (2,), (1.2,), 4),
    "ragged": ((13.0, 15.5, 11.0), (5, 1, 3), (1.9, 2.1, 1.7), 7),
    "tetragonal": ((14.0, 14.0, 20.0), (8, 8), (2.0, 2.3), 8),
    "orthorhombic": ((20.0, 20.0, 24.0), (16, 16), (2.0, 2.3), 8),
    "cubic64": ((24.0, 24.0, 24.0), (32, 32), (2.2, 2.2), 10),
    "cubic128": ((30.0, 30.0, 30.0), (32, 32, 32, 32), (2.2, 2.2, 2.2, 2.2), 10),
}


def listed():
    return [
        # the smallest call: one k-point of a two-atom cell, where launches and latency are the time
        dict(name="forward_tiny_256", op="forward", cell="tiny", ng=256, precision="fp64"),
        # an ordinary small cell with uneven types and a size that is no multiple of anything
        dict(name="forward_ragged_1237", op="forward", cell="ragged", ng=1237, precision="fp64"),
        # one k-point of a medium cell: too few tiles to fill the GPU by themselves
        dict(name="forward_tetragonal_3000", op="forward", cell="tetragonal", ng=3000, precision="fp64"),
        # the benchmark's workload: the largest cell, bound by the matrix cores
        dict(name="forward_cubic128_12000", op="forward", cell="cubic128", ng=12000, precision="fp64"),
        # split precision on the 16-bit matrix cores at a medium size
        dict(name="residue_bf16_tetragonal_3000", op="forward", cell="tetragonal", ng=3000, precision="residue_bf16"),
        # split precision on the int8 matrix cores at the benchmark's size
        dict(name="residue_int8_cubic128_12000", op="forward", cell="cubic128", ng=12000, precision="residue_int8"),
        # the type-factored build: a medium cell, odd size
        dict(name="factored_orthorhombic_3101", op="factored", cell="orthorhombic", ng=3101, precision="fp64"),
        # the type-factored build at the benchmark's size
        dict(name="factored_cubic128_12000", op="factored", cell="cubic128", ng=12000, precision="fp64"),
        # an inversion-symmetric cell: real symmetric matrices, odd size
        dict(name="real_cubic64_6001", op="real", cell="cubic64", ng=6001, precision="fp64"),
        # a set of k-points with uneven bases in one call
        dict(name="batch_orthorhombic_16x3100", op="batch", cell="orthorhombic", ng=3100, nk=16, precision="fp64"),
        # the adjoint alone, for forces and T derivatives, at the size of the loss workload
        dict(name="backward_cubic64_6000", op="backward", cell="cubic64", ng=6000, precision="fp64"),
        # forward and backward through autograd, a step of a fit on a small cell, odd size
        dict(name="autograd_ragged_801", op="autograd", cell="ragged", ng=801, precision="fp64"),
    ]


# op -> cells it is drawn on, N_G range
_RANGES = {
    "forward": (("tiny", "ragged", "tetragonal", "orthorhombic", "cubic64"), (180, 6000)),
    "residue": (("tetragonal", "orthorhombic", "cubic64", "cubic128"), (1500, 9000)),
    "factored": (("ragged", "tetragonal", "orthorhombic", "cubic64", "cubic128"), (800, 12000)),
    "real": (("ragged", "tetragonal", "orthorhombic", "cubic64"), (800, 7000)),
    "batch": (("tiny", "ragged", "tetragonal", "orthorhombic"), (200, 3400)),
    "backward": (("ragged", "tetragonal", "orthorhombic", "cubic64"), (400, 6000)),
    "autograd": (("tiny", "ragged", "tetragonal"), (180, 2000)),
}
# the largest basis drawn for a cell: about what its volume holds at a cut-off of 5 / bohr
_MOST = {"tiny": 900, "ragged": 2600, "tetragonal": 5000, "orthorhombic": 9000, "cubic64": 9000, "cubic128": 12000}


def draw(rng):
    op = rng.choice(("forward", "forward", "residue", "factored", "real", "batch", "backward", "autograd"))
    cells, (lo, hi) = _RANGES[op]
    cell = rng.choice(cells)
    hi = min(hi, _MOST[cell])
    lo = min(lo, hi // 2)
    ng = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    precision = "fp64"
    if op == "residue":
        op, precision = "forward", rng.choice(("residue_int8", "residue_int8", "residue_bf16"))
    case = dict(op=op, cell=cell, ng=ng, precision=precision)
    if op == "batch":
        case["nk"] = rng.randint(2, 16)
    return case


# ---- inputs ------------------------------------------------------------------------------


def _basis(side, k, ng):
    """The ng integer triples g with the shortest |2 pi (g + k) / side|."""
    b = 2.0 * np.pi / np.asarray(side)
    radius = 1.15 * (6.0 * np.pi ** 2 * ng / float(np.prod(side))) ** (1.0 / 3.0) + float(b.max())
    axes = [np.arange(-int(radius / bi) - 1, int(radius / bi) + 2) for bi in b]
    grid = np.stack(np.meshgrid(*axes, indexing="ij"), axis=-1).reshape(-1, 3)
    norm = (((grid + k) * b) ** 2).sum(axis=1)
    order = np.argsort(norm, kind="stable")[:ng]
    assert norm[order[-1]] <= radius ** 2
    return np.ascontiguousarray(grid[order].astype(np.int32))


def _positions(rng, side, counts, radii, inversion):
    """Fractional positions, type by type, with non-overlapping spheres; with `inversion` in pairs
    (f, -f), an odd atom of a type at the origin (the first such type) or on another fixed point."""
    side = np.asarray(side)
    frac, rad, partner = [], [], []
    fixed = [np.array(p) for p in ((0.0, 0.0, 0.0), (0.5, 0.5, 0.5), (0.5, 0.0, 0.0), (0.0, 0.5, 0.5))]

    def free(f, r):
        if not frac:
            return True
        d = f - np.asarray(frac)
        d -= np.round(d)
        return bool((np.sqrt(((d * side) ** 2).sum(axis=1)) >= r + np.asarray(rad)).all())

    def put(f, r):
        frac.append(f)
        rad.append(r)

    for n, r in zip(counts, radii):
        left = n
        if inversion and n % 2:
            # only the origin is its own image exactly (no lattice vector between f and -f)
            f = fixed[0]
            if not free(f, r):
                raise RuntimeError("origin taken")
            partner.append(len(frac))
            put(f, r)
            left -= 1
        while left > 0:
            f = rng.uniform(-0.5, 0.5, 3)
            if inversion:
                d = 2.0 * f - np.round(2.0 * f)
                if not free(f, r) or not free(-f, r) or np.sqrt(((d * side) ** 2).sum()) < 2.0 * r:
                    continue
                i = len(frac)
                partner.extend([i + 1, i])
                put(f, r)
                put(-f, r)
                left -= 2
            elif free(f, r):
                put(f, r)
                left -= 1
    return np.asarray(frac), np.asarray(partner if inversion else np.arange(len(frac)), dtype=np.int32)


def _symmetric(T, l_max):
    """T's mean with its time-reversal image, without the entries of odd l + l'."""
    n_l = (l_max + 1) ** 2
    lv = np.concatenate([[l] * (2 * l + 1) for l in range(l_max + 1)])
    mv = np.concatenate([np.arange(-l, l + 1) for l in range(l_max + 1)])
    at = lv * lv + lv - mv
    flip, sign = np.concatenate([at, n_l + at]), np.tile((-1.0) ** mv, 2)
    image = sign[:, None] * sign[None, :] * np.conj(T[np.ix_(flip, flip)])
    ll = np.tile(lv, 2)
    return np.where((ll[:, None] + ll[None, :]) % 2, 0.0, 0.5 * (T + image))


def _inputs(case, seed):
    """Host arrays of a case: everything a program reads from its own set-up."""
    side, counts, radii, l_max = CELLS[case["cell"]]
    rng = np.random.Generator(np.random.PCG64([20171207, int(seed)]))
    inversion = case["op"] == "real"
    if inversion:  # one odd type at most: the origin is the one fixed point with tau = -tau
        counts = tuple(c if i == 0 else c + c % 2 for i, c in enumerate(counts))
    frac, partner = _positions(rng, side, counts, radii, inversion)
    n_t, n_l = len(counts), (l_max + 1) ** 2
    m = 2 * n_l
    radial = rng.uniform(0.5, 1.5, (n_t, l_max + 1, 4))
    while True:
        bad = np.abs(radial[..., 0] * radial[..., 3] - radial[..., 2] * radial[..., 1]) < 0.1
        if not bad.any():
            break
        radial[bad, 2:] = rng.uniform(0.5, 1.5, (int(bad.sum()), 2))
    T = rng.normal(0.0, 0.05 / math.sqrt(2.0), (n_t, m, m, 2)).view(np.complex128)[..., 0]
    T = np.triu(T, 1)
    T = T + np.conj(np.swapaxes(T, 1, 2))
    T[:, np.arange(m), np.arange(m)] = rng.uniform(-2.0, 2.0, (n_t, m))
    if inversion:
        T = np.stack([_symmetric(t, l_max) for t in T])
    nk = case.get("nk", 1)
    k = rng.uniform(-0.5, 0.5, (nk, 3))
    ng = case["ng"]
    # the k-points' basis sizes belong to the case (a set-up of its own), the rest is drawn anew
    spread = np.random.Generator(np.random.PCG64([ng, nk]))
    sizes = [ng] if nk == 1 else [int(x) for x in spread.integers(int(0.9 * ng), int(1.1 * ng) + 1, nk)]
    return dict(
        side=side, l_max=l_max, r_mt=np.asarray(radii), types=np.repeat(np.arange(n_t), counts).astype(np.int32),
        tau=frac * np.asarray(side), partner=partner, radial=radial, udot=rng.uniform(0.01, 0.1, (n_t, l_max + 1)),
        T=T, k=k, g=[_basis(side, k[i], sizes[i]) for i in range(nk)], sizes=sizes)


def _gradients(ng, seed, device):
    """Two Hermitian matrices dL/dH and dL/dS, entries of size 1 / ng."""
    gen = torch.Generator(device=device).manual_seed(int(seed) + 77)

    def one():
        z = torch.randn(ng, ng, 2, dtype=torch.float64, device=device, generator=gen) / ng
        z = torch.view_as_complex(z)
        return (0.5 * (z + z.conj().transpose(0, 1))).contiguous()

    return one(), one()


def prepare(case, seed):
    d = _inputs(case, seed)
    op, ng = case["op"], d["sizes"]
    prec = PRECISION[case["precision"]]
    b = HSBuilder(np.diag(d["side"]), d["types"], d["r_mt"], d["radial"], d["udot"], d["l_max"], max(ng),
                  precision=prec, n_slices=0 if prec == HSB_FP64 else MODULI)
    state = dict(op=op, builder=b, k=d["k"], partner=d["partner"],
                 g=[torch.as_tensor(x, device="cuda") for x in d["g"]],
                 tau=torch.as_tensor(d["tau"], device="cuda"), T=torch.as_tensor(d["T"], device="cuda").contiguous())
    kind = torch.float64 if op == "real" else torch.complex128
    if op in ("forward", "factored", "real"):  # a program's own matrices; only their upper triangles are written
        state["H"] = torch.zeros(ng[0], ng[0], dtype=kind, device="cuda")
        state["S"] = torch.zeros(ng[0], ng[0], dtype=kind, device="cuda")
    elif op == "batch":
        total = sum(n * n for n in ng)
        state["H"] = torch.zeros(total, dtype=kind, device="cuda")
        state["S"] = torch.zeros(total, dtype=kind, device="cuda")
    else:
        state["gH"], state["gS"] = _gradients(ng[0], seed, "cuda")
        if op == "autograd":
            state["tau"].requires_grad_(True)
            state["T"].requires_grad_(True)
    return state


def run(s):
    b, op = s["builder"], s["op"]
    if op == "forward":
        return b.forward(s["k"][0], s["g"][0], s["tau"], s["T"], H=s["H"], S=s["S"])
    if op == "factored":
        return b.forward_factored(s["k"][0], s["g"][0], s["tau"], s["T"], H=s["H"], S=s["S"])
    if op == "real":
        return b.forward_real(s["k"][0], s["g"][0], s["tau"], s["partner"], s["T"], H=s["H"], S=s["S"])
    if op == "batch":
        H, S, _ = b.batch(s["k"], s["g"], s["tau"], s["T"], H=s["H"], S=s["S"])
        return H, S
    if op == "backward":
        return b.backward(s["k"][0], s["g"][0], s["tau"], s["T"], s["gH"], s["gS"])
    H, S = hs_build(s["tau"], s["T"], b, s["k"][0], s["g"][0])
    gtau, gT = torch.autograd.grad((H, S), (s["tau"], s["T"]), (s["gH"], s["gS"]))
    return H.detach(), S.detach(), gT, gtau


def work(case):
    """Inputs read once, outputs written once; the complex products with three real ones each.

    forward, batch, residue: H by the stacked contraction over all atoms, the upper triangle; S by its
    sum over atom pairs' phases and l.  factored: one product per type.  real: half the atoms, two real
    products.  backward: the adjoint of the type-factored form."""
    side, counts, _, l_max = CELLS[case["cell"]]
    n_l, n_a = (l_max + 1) ** 2, sum(counts)
    m, n_t, nk, n = 2 * n_l, len(counts), case.get("nk", 1), case["ng"]
    op = case["op"]
    tri = n * (n + 1) / 2.0
    small = 16.0 * n_t * m * m + 24.0 * n_a + 12.0 * n * nk
    s_flops = tri * (6.0 * n_a + 8.0 * n_t * (l_max + 1))
    per_type = 4.0 * n_t * m * m * n
    fact = tri * (6.0 * n_a + 4.0 * n_t * m)
    if op in ("forward", "batch"):
        return dict(bytes=nk * 32.0 * tri + small, flops=nk * (6.0 * m * n_a * tri + s_flops + per_type))
    if op == "real":
        return dict(bytes=16.0 * tri + small, flops=4.0 * m * (n_a / 2.0) * tri + s_flops / 2.0 + per_type)
    if op == "factored":
        return dict(bytes=32.0 * tri + small, flops=fact + s_flops + per_type)
    back = 2.0 * fact + tri * (6.0 * n_a + 4.0 * n_t * m)
    if op == "backward":
        return dict(bytes=32.0 * n * n + small + 16.0 * n_t * m * m, flops=back)
    return dict(bytes=64.0 * n * n + 2 * small + 16.0 * n_t * m * m, flops=back + 6.0 * m * n_a * tri + s_flops)


# ---- the paper's formulas in 64 bits ------------------------------------------------------


def _bessel(l_top, x):
    """j_0 .. j_l_top at x > 0: series for small x, downward recurrence otherwise."""
    out = np.zeros((l_top + 1, x.size))
    low = x < 2.0
    xs = x[low]
    pref = np.ones_like(xs)
    for l in range(l_top + 1):
        if l:
            pref = pref * xs / (2 * l + 1)
        t, s = np.ones_like(xs), np.ones_like(xs)
        for q in range(1, 40):
            t = t * (-0.5 * xs * xs) / (q * (2 * l + 2 * q + 1))
            s = s + t
        out[l, low] = pref * s
    xb = x[~low]
    if xb.size:
        top = l_top + 30 + int(xb.max())
        f = np.zeros((top + 2, xb.size))
        f[top] = 1e-290
        for i in range(top, 0, -1):
            f[i - 1] = (2 * i + 1) / xb * f[i] - f[i + 1]
            big = np.abs(f[i - 1]) > 1e200
            if big.any():
                f[i - 1:, big] *= 1e-200
        j0, j1 = np.sin(xb) / xb, np.sin(xb) / xb ** 2 - np.cos(xb) / xb
        peak = np.maximum(np.abs(f[0]), np.abs(f[1]))
        a, c = f[0] / peak, f[1] / peak
        out[:, ~low] = f[:l_top + 1] / peak * ((j0 * a + j1 * c) / (a * a + c * c))
    return out


def _harmonics(l_max, K, kn):
    """Y_lm of the directions of K, rows L = l^2 + l + m, Condon-Shortley phase."""
    n = kn.size
    ct = np.where(kn > 0, K[:, 2] / np.where(kn > 0, kn, 1.0), 1.0)
    w = np.where(kn > 0, (K[:, 0] + 1j * K[:, 1]) / np.where(kn > 0, kn, 1.0), 0.0)
    Y = np.zeros(((l_max + 1) ** 2, n), dtype=np.complex128)
    diag = np.full(n, math.sqrt(0.25 / math.pi))
    wm = np.ones(n, dtype=np.complex128)
    for m in range(l_max + 1):
        if m:
            diag = -diag * math.sqrt((2 * m + 1) / (2.0 * m))
            wm = wm * w
        p0, p1 = np.zeros(n), diag
        for l in range(m, l_max + 1):
            if l > m:
                al = math.sqrt((4.0 * l * l - 1) / (l * l - m * m))
                bl = math.sqrt(((l - 1.0) ** 2 - m * m) / (4.0 * (l - 1) ** 2 - 1))
                p0, p1 = p1, al * (ct * p1 - bl * p0)
            Y[l * l + l + m] = p1 * wm
            Y[l * l + l - m] = (-1) ** m * np.conj(p1 * wm)
    return Y


def _coefficients(d, i, device):
    """Per type [A; B] at the origin (complex, [2 N_L][N_G]), the weights of S, the K vectors."""
    side, l_max = np.asarray(d["side"]), d["l_max"]
    K = (d["g"][i] + d["k"][i]) * (2.0 * np.pi / side)
    kn = np.sqrt((K ** 2).sum(axis=1))
    lv = np.concatenate([[l] * (2 * l + 1) for l in range(l_max + 1)])
    ang = 4.0 * np.pi / math.sqrt(float(np.prod(side))) * (1j ** lv)[:, None] * np.conj(_harmonics(l_max, K, kn))
    per_type = []
    for t in range(len(d["r_mt"])):
        j = _bessel(l_max + 1, np.maximum(kn * d["r_mt"][t], 1e-300))
        dj = np.stack([-j[1]] + [(l * j[l - 1] - (l + 1) * j[l + 1]) / (2 * l + 1) for l in range(1, l_max + 1)])
        u, du, ud, dud = (d["radial"][t, :, q][:, None] for q in range(4))
        W = u * dud - ud * du
        a = (j[:-1] * dud - kn * dj * ud) / W
        b = (kn * dj * u - j[:-1] * du) / W
        per_type.append(torch.as_tensor(np.concatenate([ang * a[lv], ang * b[lv]]), device=device))
    lam = [torch.as_tensor(np.concatenate([np.ones(lv.size), d["udot"][t][lv]]), device=device)
           for t in range(len(d["r_mt"]))]
    return per_type, lam, torch.as_tensor(K, device=device)


def _atoms(d, i, device):
    """For every atom: its type, phases and [A; B]."""
    per_type, lam, K = _coefficients(d, i, device)
    tau = torch.as_tensor(d["tau"], device=device)
    for a, t in enumerate(d["types"]):
        arg = K @ tau[a]
        yield a, int(t), torch.complex(torch.cos(arg), torch.sin(arg)) * per_type[t], lam[t], K


def _matrices(d, i, device):
    n = d["sizes"][i]
    H = torch.zeros(n, n, dtype=torch.complex128, device=device)
    S = torch.zeros_like(H)
    T = torch.as_tensor(d["T"], device=device)
    for _, t, W, lam, _ in _atoms(d, i, device):
        Wh = W.conj().transpose(0, 1).resolve_conj().contiguous()
        H.addmm_(Wh, T[t] @ W)
        S.addmm_(Wh, lam[:, None] * W)
    return H, S


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    d = _inputs(case, seed)
    op = case["op"]
    if op in ("forward", "factored"):
        H, S = _matrices(d, 0, device)
        return torch.triu(H), torch.triu(S)
    if op == "real":
        H, S = _matrices(d, 0, device)
        return torch.triu(H.real).contiguous(), torch.triu(S.real).contiguous()
    if op == "batch":
        Hs, Ss = [], []
        for i in range(case["nk"]):
            H, S = _matrices(d, i, device)
            Hs.append(torch.triu(H).reshape(-1))
            Ss.append(torch.triu(S).reshape(-1))
        return torch.cat(Hs), torch.cat(Ss)
    n = d["sizes"][0]
    gH, gS = _gradients(n, seed, device)
    T = torch.as_tensor(d["T"], device=device)
    gT = torch.zeros_like(T)
    gtau = torch.zeros(len(d["types"]), 3, dtype=torch.float64, device=device)
    for a, t, W, lam, K in _atoms(d, 0, device):
        PH, PS = W @ gH, W @ gS
        gT[t] += PH @ W.conj().transpose(0, 1).resolve_conj().contiguous()
        c = (PH.conj() * (T[t] @ W) + PS.conj() * (lam[:, None] * W)).sum(dim=0)
        gtau[a] = -2.0 * (K * c.imag[:, None]).sum(dim=0)
    if op == "backward":
        return gT, gtau
    H, S = _matrices(d, 0, device)
    up = lambda M: torch.triu(M) + torch.triu(M, 1).conj().transpose(0, 1)  # noqa: E731
    return up(H), up(S), gT, gtau
