"""The autotuner's default candidates and its cache, whose entries of earlier builds named 4 waves as a layout: now that
pins the stacked contraction."""
import json

import pytest
import torch

from flapw_cells import make_batch_case, make_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    yield


def test_entries_of_an_earlier_form_are_not_reused(tmp_path):
    from paper_1712_07206_amd import autotune
    from paper_1712_07206_amd.hsbuild import HSBuilder
    b = HSBuilder.from_case(make_case(1, n_g=300))
    path = str(tmp_path / "tune.json")
    old = autotune._key(b, 300, 0).split("/", 1)[1]
    assert old.startswith("gfx950/")
    with open(path, "w") as f:
        json.dump({old: {"waves": 4, "tile_group": 8}}, f)
    assert autotune.cached_options(b, 300, path=path) is None


@pytest.mark.parametrize("precision,waves", [("HSB_FP64", 8), ("HSB_SPLIT_CRT", 4), ("HSB_SPLIT_CRT", 8),
                                             ("HSB_SPLIT_CRT_BF16", 8)])
def test_default_candidates_leave_the_form_alone(precision, waves):
    """FP64: the library's choice, also where the caller had pinned the stacked form; a residue handle: the layout
    it has."""
    from paper_1712_07206_amd import _native as N
    from paper_1712_07206_amd import autotune
    from paper_1712_07206_amd.hsbuild import HSBuilder, case_tensors
    case = make_case(1, n_g=300)
    g, tau, T = case_tensors(case)
    b = HSBuilder.from_case(case, precision=getattr(N, precision), n_slices=11)
    b.set_option(N.HSB_OPT_HS_WAVES, 4 if precision == "HSB_FP64" else waves)
    res = autotune.tune(b, case["k_frac"], g, tau, T, precision=getattr(N, precision), reps=1, path=None)
    assert set(res["candidates_ms"]) == {"w%d_g%d" % (waves, gr) for gr in autotune.TILE_GROUPS}
    assert b.get_option(N.HSB_OPT_HS_WAVES) == res["waves"] == waves


def test_default_candidates_of_the_batch():
    from paper_1712_07206_amd import _native as N
    from paper_1712_07206_amd import autotune
    from paper_1712_07206_amd.hsbuild import HSBuilder
    case = make_batch_case(3, n_k=2)
    b = HSBuilder.from_case(case)
    tau, T = torch.as_tensor(case["tau"], device="cuda"), torch.as_tensor(case["T"], device="cuda")
    res = autotune.tune_batch(b, case["k_frac"], [torch.as_tensor(x, device="cuda") for x in case["g"]], tau, T)
    assert set(res["candidates_ms"]) == {"w8_g8", "w8_g4"} and b.get_option(N.HSB_OPT_HS_WAVES) == 8
