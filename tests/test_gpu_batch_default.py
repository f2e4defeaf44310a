"""The batch tests and the one at k = 0 with the default options, which run the type-factored form; the tests themselves pin the
stacked one with HSB_OPT_SPLIT_K = 0.  Their k-points of about 3000 plane waves take the larger tiles and blocks over all k-points
(half tiles, 64 x 64 blocks of T' R), the small ones the smaller."""
import numpy as np
import pytest
import torch

import test_gpu_batch as batch
import test_gpu_gamma as gamma
from flapw_cells import make_batch_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    yield


def _default(case):
    from paper_1712_07206_amd.hsbuild import HSBuilder
    b = HSBuilder.from_case(case)
    tau = torch.as_tensor(case["tau"], device="cuda")
    T = torch.as_tensor(case["T"], device="cuda")
    return b, tau, T, [torch.as_tensor(g, device="cuda") for g in case["g"]]


@pytest.mark.parametrize("name", ["equals_sequential_bitwise", "graph_reuse_and_recapture", "sees_g_lists_changed_in_place",
                                  "small_uneven_bases_against_oracle", "full_64k_against_oracle"])
def test_batch(name, monkeypatch):
    monkeypatch.setattr(batch, "_setup", _default)
    getattr(batch, "test_batch_" + name)()


def test_gamma_in_batch(monkeypatch):
    from paper_1712_07206_amd.hsbuild import HSBuilder
    monkeypatch.setattr(HSBuilder, "set_option", lambda *_: None)
    gamma.test_gamma_in_batch()


def test_batch_against_the_stacked_batch():
    """Bar: FP64 rounding of two forms, 1e-12 relative over each block's upper triangle; the graph replayed after other
    work, with T changed in place."""
    from paper_1712_07206_amd import _native as N
    case = make_batch_case(3, n_k=4)
    b, tau, T, gl = _default(case)
    r, _, _, _ = _default(case)
    r.set_option(N.HSB_OPT_SPLIT_K, 0)
    H = S = None
    for scale in (1.0, 0.5, -2.0):
        T.mul_(scale)
        H, S, off = b.batch(case["k_frac"], gl, tau, T, H, S)
        Hr, Sr, _ = r.batch(case["k_frac"], gl, tau, T)
        for k, n in enumerate(int(x) for x in case["n_g"]):
            iu = torch.triu_indices(n, n, device="cuda")
            for M, R in ((H, Hr), (S, Sr)):
                x, y = (batch._block(m, off[k], n)[iu[0], iu[1]] for m in (M, R))
                assert (torch.linalg.norm(x - y) / torch.linalg.norm(y)).item() <= 1e-12, (scale, k)
    assert np.all(np.asarray(case["n_g"]) >= 2800)
