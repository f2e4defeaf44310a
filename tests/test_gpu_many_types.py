"""Cells of many atom types with few atoms each, where a pass over the types costs more than the atoms of each save."""
import numpy as np
import pytest
import torch

import test_gpu_typed as typed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_1712_07206_amd import _native
    _native.lib()
    yield


def _stacked_adjoint_bytes(n_types, n_atoms, l_max, n):
    """Workspace of the adjoint on the rows of all atoms: tables, T^T, lam, five arrays of the stacked rows, gH and gS padded,
    and the partial sums, each rounded up to 256 bytes."""
    up = lambda v, m: (v + m - 1) // m * m  # noqa: E731
    n_l = (l_max + 1) ** 2
    m, k = 2 * n_l, 2 * n_atoms * n_l
    kp, np_ = (k + 30) // 16 * 16, up(n, 128)
    sizes = [16 * 13 * 5 * 8, np_ * 32, n_l * np_ * 16, n_types * (l_max + 1) * np_ * 16, n_types * up(m, 16) * up(m, 128) * 16,
             kp * 8] + [kp * np_ * 16] * 4 + [np_ * up(kp, 128) * 16] + [np_ * np_ * 16] * 2
    return sum(up(s, 256) for s in sizes + [n_atoms * m * m * 16, n_atoms * ((n + 255) // 256) * 24])


@pytest.mark.parametrize("atoms,l_max", [((1,) * 16, 0), ((1,) * 16, 2), ((1,) * 16, 6), ((2,) * 16, 1), ((1,) * 8, 1)])
def test_adjoint_workspace_is_no_larger_than_the_stacked_operands(atoms, l_max):
    """hsbuild_backward asks for no more than the rows of all atoms take, and so doesn't go over the types one by one
    for want of it (16 types of one atom at N_G = 100: 48 launches, 0.32 ms where the stacked rows take 0.12)."""
    from paper_1712_07206_amd import _native as N
    from paper_1712_07206_amd.hsbuild import HSBuilder
    b = HSBuilder.from_case(typed._case(atoms, l_max, 20), max_ng=6000)
    for n in (1, 100, 5000):
        need, bar = b.workspace_bytes(N.HSB_MODE_BACKWARD, [n]), _stacked_adjoint_bytes(len(atoms), sum(atoms), l_max, n)
        print("types", len(atoms), "l_max", l_max, "N_G", n, "bytes", need, "stacked", bar, flush=True)
        assert need <= bar


# on both sides of the rule between the stacked and the type-factored adjoint; a type without atoms
@pytest.mark.parametrize("atoms,l_max,n_g", [((1,) * 16, 0, 1), ((1,) * 16, 2, 70), ((2,) * 8, 0, 129),
                                             ((1,) * 7 + (0,) + (2,) * 8, 1, 128), ((1,) * 16, 6, 65), ((1,) * 16, 1, 1100),
                                             ((12, 1) * 6, 6, 70), ((1,) * 6, 3, 300)])
def test_adjoint_of_general_matrices(atoms, l_max, n_g):
    typed.test_adjoint_of_general_matrices(atoms, l_max, n_g)
