"""The fp32 GEMM's tiles and splits at their edges: one row past a tile, a k chunk of 16, odd and even
numbers of chunks, ranges of a split contraction that end inside a chunk -- against the fp64 oracle."""
import pytest

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import check_all, sk, tuning  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [1, 4], ids=["128x128", "64x64"])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("shape", [(1, 16, 16, 1, 16), (65, 48, 80, 1, 16), (129, 464, 144, 3, 48), (641, 416, 272, 1, 144)],
                         ids=lambda s: "T%d_%dx%d_l%dk%d" % s)
def test_f32_tiles_and_splits(sk, tuning, tile, splits, shape):  # noqa: F811
    # bound: the repository's fp32 bar; sums of at most 641 products carry about 641 * 2^-24 = 4e-5
    # of their terms' magnitude at worst, and sqrt of that length in practice
    tuning(sk.SK_TUNE_TILE, tile)
    tuning(sk.SK_TUNE_SSPLITS, splits)
    tuning(sk.SK_TUNE_WSPLITS, splits)
    T, d_in, d_out, l, k = shape
    check_all(sk, W.Workload("f32_tiles", T, d_in, d_out, l, k, "f32", seed=40 + T), 0, single_call=True)
