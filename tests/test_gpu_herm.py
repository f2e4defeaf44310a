"""hsbuild_mirror and hsbuild_hermitian_part at the edges of their 32 x 32 tiles, bitwise against torch."""
import pytest
import torch

from test_gpu_typed import _case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1712_07206_amd import _native
    _native.lib()
    yield


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 65])
def test_full_matrices(n):
    from paper_1712_07206_amd.hsbuild import HSBuilder, hermitian_full
    b = HSBuilder.from_case(_case((1,), 0, n))
    gen = torch.Generator().manual_seed(n)
    rand = lambda: torch.randn(n, n, dtype=torch.complex128, generator=gen).cuda()  # noqa: E731
    H, S = rand(), rand()
    H[torch.ones(n, n, dtype=torch.bool).tril(-1)] = float("nan")  # what a build leaves there
    want = [torch.where(torch.ones(n, n, dtype=torch.bool, device="cuda").tril(-1), M.conj().T, M) for M in (H, S)]
    assert torch.equal(want[1], hermitian_full(S))
    H, S = b.mirror(H, S)
    assert torch.equal(H, want[0]) and torch.equal(S, want[1])
    part = lambda g: 0.5 * (g + g.conj().transpose(0, 1))  # noqa: E731
    x, y = rand(), rand()
    for gH, gS in ((x, y), (x.T, y.conj()), (None, y), (x.real.to(torch.complex128), None), (x[:1].expand(n, n), y)):
        oH, oS = b.hermitian_part(n, gH, gS)
        zero = torch.zeros(n, n, dtype=torch.complex128, device="cuda")
        assert torch.equal(oH, zero if gH is None else part(gH)) and torch.equal(oS, zero if gS is None else part(gS))
