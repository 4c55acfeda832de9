"""The narrow kernels' walk over their output tiles: runs of one to five tiles, odd and even, of equal and of
unequal length side by side, the last tile ragged -- those of up to three (two of 128 rows), and any of a
lone token tile, straight from registers, longer ones through LDS -- both token tiles, both widths, with
the first contraction fused in and from slabs, against the fp64 oracle."""
import pytest

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import check_all, sk, tuning  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("plan", [1, 3], ids=["fused", "split_expand"])
@pytest.mark.parametrize("bm", [64, 128])
@pytest.mark.parametrize("R", [48, 128])
@pytest.mark.parametrize("slices", [1, 2, 3, 5])
def test_runs_of_output_tiles(sk, tuning, plan, bm, R, slices):  # noqa: F811
    # 592 = 4 tiles of 128 and 80 columns: runs of 5 | 3 + 2 | 2 + 2 + 1 | 1; the other direction, 464: 4 | 2 | 2 | 1
    # bound: the repository's bf16 bar (the intermediate and the result rounded to 8 bits once each)
    tuning(sk.SK_TUNE_BM, bm)
    tuning(sk.SK_TUNE_SLICES, slices)
    check_all(sk, W.Workload("chain_runs", 203, 464, 592, 1, R, "bf16", seed=50 + slices), plan)


@pytest.mark.parametrize("plan", [1, 3], ids=["fused", "split_expand"])
def test_long_run_of_a_lone_token_tile(sk, tuning, plan):  # noqa: F811
    # bound: as above
    tuning(sk.SK_TUNE_SLICES, 1)
    check_all(sk, W.Workload("chain_lone_tile", 40, 464, 592, 1, 48, "bf16", seed=57), plan)
