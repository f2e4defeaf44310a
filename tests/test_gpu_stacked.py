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
