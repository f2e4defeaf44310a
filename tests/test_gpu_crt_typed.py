"""The residue form of the type-factored build (H by residues per type, S in FP64) at the sizes where its
tiles, chunks and matrix-core steps change, and the stacked residue contraction it leaves to
hsbuild_forward_coefficients.

Bar for H, element by element: a column of R_t or Y_t (M = 2 N_L rows) is scaled to a 2-norm of at least
(bound - sqrt(2 M) / 2) / 2 and its entries rounded by at most 1/2 (1/sqrt(2) for the complex Y), so
|dR| <= sqrt(M) / 2 and |dY| <= sqrt(M / 2), and a type's entry is off by at most
e |R| |Y|, e = (sqrt(M) / 2 + sqrt(M / 2)) * 2 / (bound - sqrt(2 M) / 2) (1 + a second-order term); times |P_t| <= the
atoms of the type, |R| = |W_a|, |Y| = |T W_a|.  On top of that the FP64 path's 1e-12 of the norm; S: that alone."""
import numpy as np
import pytest
import torch

from oracle import hs_oracle as o
from test_gpu_crt import _wide_case
from test_gpu_typed import TOL, _case, _full, _rel

pytestmark = pytest.mark.gpu

MODULI = (241, 233, 229, 197, 193, 181, 173, 169, 157, 149, 137, 125, 113)


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1712_07206_amd import _native
    _native.lib()
    yield


def _bound(case, n_mod):
    m = 2 * case["n_l"]
    bound = np.sqrt(0.5 * np.prod(np.array(MODULI[:n_mod], dtype=float)) * (1 - 2.0 ** -10))
    e = 1.01 * (np.sqrt(m) / 2 + np.sqrt(m / 2)) * 2 / (bound - np.sqrt(2 * m) / 2)
    W = o.coefficients(case).reshape(case["n_atoms"], m, case["n_g"])
    norm = lambda x: np.sqrt((np.abs(x) ** 2).sum(axis=0))  # noqa: E731
    return e * sum(np.outer(norm(W[a]), norm(case["T"][t] @ W[a])) for a, t in enumerate(case["atom_type"]))


def _check(case, real=False, n_mod=11):
    from paper_1712_07206_amd import HSB_SPLIT_CRT, HSB_SPLIT_CRT_BF16, HSB_SPLIT_CRT_FP16
    from paper_1712_07206_amd.hsbuild import HSBuilder, case_tensors
    n = case["n_g"]
    print("atoms", np.bincount(case["atom_type"]), "l_max", case["l_max"], "N_G", n, "moduli", n_mod, flush=True)
    Hr, Sr = o.hs(case)
    if real:
        Hr, Sr = Hr.real, Sr.real
    bar = _bound(case, n_mod) + TOL * np.linalg.norm(Hr)
    iu, il = np.triu_indices(n), np.tril_indices(n, -1)
    first = None
    for prec in (HSB_SPLIT_CRT, HSB_SPLIT_CRT_BF16, HSB_SPLIT_CRT_FP16):
        b = HSBuilder.from_case(case, precision=prec, n_slices=n_mod)
        g, tau, T = case_tensors(case)
        H = torch.full((n, n), float("nan"), dtype=torch.float64 if real else torch.complex128, device="cuda")
        S = H.clone()
        if real:
            b.forward_real(case["k_frac"], g, tau, case["partner"], T, H, S)
        else:
            b.forward(case["k_frac"], g, tau, T, H, S)
        torch.cuda.synchronize()
        H, S = H.cpu().numpy(), S.cpu().numpy()
        b.close()
        for M in (H, S):
            assert np.all(np.isnan(M[il])), "strict lower triangle was written"
        if first is None:
            first = H, S
            assert np.all(np.abs(H - Hr)[iu] <= bar[iu])
            assert _rel(_full(S), Sr) <= TOL
        else:  # the same integers on the 16-bit matrix cores
            assert np.array_equal(H[iu], first[0][iu]) and np.array_equal(S[iu], first[1][iu])


@pytest.mark.parametrize("n_g", [1, 31, 33, 63, 64, 65, 129])
def test_basis_around_the_tiles(n_g):
    _check(_case((3, 1), 2, n_g))


@pytest.mark.parametrize("atoms", [(1,), (11, 12, 13), (1,) * 16])
def test_atom_counts_around_the_chunks(atoms):
    _check(_case(atoms, 1, 70))


@pytest.mark.parametrize("l_max", [0, 3, 5, 7, 12])  # 2, 32, 72, 128, 338 rows
def test_rows_around_the_steps(l_max):
    _check(_case((2, 2), l_max, 70))


@pytest.mark.parametrize("n_mod", [8, 13])  # fewest and most; an odd and an even number of steps
def test_moduli(n_mod):
    _check(_case((2, 3), 4, 66), n_mod=n_mod)


@pytest.mark.parametrize("atoms,l_max,n_g", [((1,), 0, 40), ((25, 2), 3, 65), ((3, 4), 7, 129)])
def test_real_form(atoms, l_max, n_g):
    _check(_case(atoms, l_max, n_g, inversion=True), real=True)


def test_stacked_layouts_past_the_reduction_window():
    """hsbuild_forward_coefficients on the coefficients of a 288-atom cell, 69696 stacked rows: the byte form's
    8-wave layout reduces its int32 sums after 65536 rows, its 4-wave layout not at all, the 16-bit forms every
    1024: the same H and S, to the split path's 1e-10."""
    from paper_1712_07206_amd import HSB_SPLIT_CRT, HSB_SPLIT_CRT_BF16, HSB_SPLIT_CRT_FP16
    from paper_1712_07206_amd import _native as N
    from paper_1712_07206_amd.hsbuild import HSBuilder
    n = 96
    case = _wide_case(n, 40)
    coef = o.coefficients(case)
    assert 65536 < 2 * case["n_atoms"] * case["n_l"] <= 131072
    Hr, Sr = o.hs(case)
    iu = np.triu_indices(n)
    first = None
    for prec, waves in ((HSB_SPLIT_CRT, 4), (HSB_SPLIT_CRT, 8), (HSB_SPLIT_CRT_BF16, 8), (HSB_SPLIT_CRT_FP16, 8)):
        print("precision", prec, "waves", waves, flush=True)
        b = HSBuilder.from_case(case, precision=prec, n_slices=11)
        b.set_option(N.HSB_OPT_HS_WAVES, waves)
        H, S = b.forward_from_coefficients(torch.as_tensor(coef, device="cuda"), torch.as_tensor(case["T"], device="cuda"))
        H, S = H.cpu().numpy(), S.cpu().numpy()
        b.close()
        if first is None:
            first = H, S
            assert _rel(_full(H), Hr) <= 1e-10 and _rel(_full(S), Sr) <= 1e-10
        assert np.array_equal(H[iu], first[0][iu]) and np.array_equal(S[iu], first[1][iu])
