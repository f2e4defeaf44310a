"""The stacked contractions on the coefficients of a cell (hsbuild_forward_coefficients), where they run whatever form
the builds take: FP64 in stream-K form, in segments and in one pass, and the residues in both layouts; and the
type-factored builds against them where no oracle reaches."""
import numpy as np
import pytest
import torch

from flapw_cells import make_case
from oracle import hs_oracle as o

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    yield


def _full(M):
    return np.triu(M) + np.triu(M, 1).conj().T


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _nan(n):
    return torch.full((n, n), complex(float("nan"), float("nan")), dtype=torch.complex128, device="cuda")


def _from_coefficients(b, coef, T):
    """Upper triangles of H and S; the lower ones untouched."""
    n = coef.shape[-1]
    H, S = _nan(n), _nan(n)
    b.forward_from_coefficients(coef, T, H, S)
    H, S = H.cpu().numpy(), S.cpu().numpy()
    il = np.tril_indices(n, -1)
    assert np.all(np.isnan(H[il])) and np.all(np.isnan(S[il])), "strict lower triangle written"
    return H, S


@pytest.mark.parametrize("idx,n_g", [(1, 1), (1, 7), (1, 129), (1, 513), (0, None), (4, 800), (1, 3000)])
def test_stream_k_and_segments_match_one_pass(idx, n_g):
    """HSB_OPT_SPLIT_K 1 (stream-K at these sizes, but for the 100 rows of the two-atom cell: its slots show in the
    workspace) and 2 (two segments) against 0 (one pass), each bitwise equal across runs; one pass against the oracle's
    Eqs. 4-5 to 1e-12.  Bars between the forms: relative Frobenius 1e-14, and 1e-13 of the largest entry (the shared
    tiles sum the same products in pieces, over up to 15488 rows, so single entries move by a few ulps of the terms)."""
    from paper_1712_07206_amd import _native as N
    from paper_1712_07206_amd.hsbuild import HSBuilder, case_tensors
    case = make_case(idx, n_g=n_g)
    n = case["n_g"]
    b = HSBuilder.from_case(case)
    g, tau, T = case_tensors(case)
    coef = b.coefficients(case["k_frac"], g, tau)
    iu = np.triu_indices(n)
    out, need = {}, {}
    for mode in (0, 1, 1, 2, 2):
        b.set_option(N.HSB_OPT_SPLIT_K, mode)
        need[mode] = b.workspace_bytes(N.HSB_MODE_FORWARD, [n])
        H, S = _from_coefficients(b, coef, T)
        out.setdefault(mode, []).append((H[iu], S[iu]))
    b.close()
    print("idx", idx, "N_G", n, "workspace", need, flush=True)
    assert (need[1] > need[0]) == (idx != 0)
    Hr, Sr = o.hs(case)
    ref = out[0][0]
    assert _rel(ref[0], Hr[iu]) <= 1e-12 and _rel(ref[1], Sr[iu]) <= 1e-12
    for mode in (1, 2):
        first, again = out[mode]
        for x, y, r in zip(first, again, ref):
            assert np.array_equal(x, y), mode
            assert np.linalg.norm(x - r) <= 1e-14 * np.linalg.norm(r), mode
            assert np.abs(x - r).max() <= 1e-13 * np.abs(r).max(), mode


def _one_atom():
    case = dict(make_case(0))
    case["atom_type"], case["tau"], case["n_atoms"] = case["atom_type"][:1], case["tau"][:1], 1
    return case


# stacked widths of one, two and three 64-row chunks (50, 100, 160 rows), fewer than the copy ring's four stages; one block of
# 256 columns; and 12 of them a side at 30976 rows
@pytest.mark.parametrize("which", ["one atom", "two atoms", "five atoms", "16 atoms, N_G 129", "128 atoms, N_G 3000"])
def test_residue_layouts_match_the_oracle_and_each_other(which):
    """Bytes in 4 and 8 waves, and the 16-bit kinds: bitwise the same H and S, at the split path's 1e-10."""
    from paper_1712_07206_amd import _native as N
    from paper_1712_07206_amd.hsbuild import HSBuilder, case_tensors
    case = {"one atom": _one_atom, "two atoms": lambda: make_case(0), "five atoms": lambda: make_case(8),
            "16 atoms, N_G 129": lambda: make_case(1, n_g=129),
            "128 atoms, N_G 3000": lambda: make_case(2, n_g=3000)}[which]()
    g, tau, T = case_tensors(case)
    b = HSBuilder.from_case(case)
    coef = b.coefficients(case["k_frac"], g, tau)
    b.close()
    Hr, Sr = o.hs(case)
    iu = np.triu_indices(case["n_g"])
    first = None
    for prec, waves in ((N.HSB_SPLIT_CRT, 4), (N.HSB_SPLIT_CRT, 8), (N.HSB_SPLIT_CRT_BF16, 8), (N.HSB_SPLIT_CRT_FP16, 8)):
        print(which, "precision", prec, "waves", waves, flush=True)
        b = HSBuilder.from_case(case, precision=prec, n_slices=11)
        b.set_option(N.HSB_OPT_HS_WAVES, waves)
        H, S = _from_coefficients(b, coef, T)
        b.close()
        if first is None:
            first = H, S
            eh, es = _rel(_full(H), Hr), _rel(_full(S), Sr)
            print("rel err H %.3e S %.3e" % (eh, es), flush=True)
            assert eh <= 1e-10 and es <= 1e-10
        assert np.array_equal(H[iu], first[0][iu]) and np.array_equal(S[iu], first[1][iu])


def test_type_factored_builds_against_the_stacked_contraction_at_full_size():
    """N_G = 12000, 128 atoms, l_max = 10: the FP64 and byte-residue builds against the one-pass stacked contraction of
    the same call, over the upper triangles; FP64's 1e-12 (S of the residue form too), the split path's 1e-10 for H."""
    from paper_1712_07206_amd import _native as N
    from paper_1712_07206_amd.hsbuild import HSBuilder, case_tensors
    case = make_case(2)
    n = case["n_g"]
    g, tau, T = case_tensors(case)
    b = HSBuilder.from_case(case)
    b.set_option(N.HSB_OPT_SPLIT_K, 0)
    ref = [torch.triu(M) for M in b.forward(case["k_frac"], g, tau, T)]
    b.close()
    del b
    torch.cuda.empty_cache()
    for prec, bars in ((N.HSB_FP64, (1e-12, 1e-12)), (N.HSB_SPLIT_CRT, (1e-10, 1e-12))):
        print("N_G", n, "precision", prec, flush=True)
        b = HSBuilder.from_case(case, precision=prec, n_slices=11)
        for M, R, bar in zip(b.forward(case["k_frac"], g, tau, T), ref, bars):
            e = (torch.linalg.norm(torch.triu(M) - R) / torch.linalg.norm(R)).item()
            print("rel %.3e" % e, flush=True)
            assert e <= bar
        b.close()
        del b
        torch.cuda.empty_cache()


def test_static_forward_in_the_stacked_form():
    """16 types of one atom, l_max = 2, N_G = 14000: the padded rows of the type-factored form need more than the static
    scratch, the stacked ones less; the call runs these, and agrees with hsbuild_forward to FP64 rounding."""
    from paper_1712_07206_amd import _native as N
    from paper_1712_07206_amd.hsbuild import HSBuilder, case_tensors
    from test_gpu_typed import _case
    n = 14000
    case = _case((1,) * 16, 2, n)
    g, tau, T = case_tensors(case)
    b = HSBuilder.from_case(case)
    need = b.workspace_bytes(N.HSB_MODE_FORWARD, [n])
    b.set_option(N.HSB_OPT_SPLIT_K, 0)
    stacked = b.workspace_bytes(N.HSB_MODE_FORWARD, [n])
    b.set_option(N.HSB_OPT_SPLIT_K, 1)
    print("workspace", need, "stacked", stacked, flush=True)
    assert stacked <= 256 << 20 < need
    ref = b.forward(case["k_frac"], g, tau, T)
    H, S = _nan(n), _nan(n)
    b.forward_static(case["k_frac"], g, tau, T, H, S)
    low = torch.ones((n, n), dtype=torch.bool, device="cuda").tril_(-1)
    for M, R in zip((H, S), ref):
        assert bool(torch.isnan(M.real[low]).all()), "strict lower triangle written"
        R = R.masked_fill(low, 0.0)
        assert (torch.linalg.norm(M.masked_fill(low, 0.0) - R) / torch.linalg.norm(R)).item() <= 1e-12
