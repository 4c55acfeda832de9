"""The 256 x 256 GEMM tile at its edges, forced onto shapes small enough for a full oracle pass: contractions
shorter than the four chunks its loop runs, ending inside a chunk and inside a pair of chunks, one row past
a tile, several tiles per work-group, and the token contraction in ranges -- against the fp64 oracle."""
import pytest

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import check_all, sk, tuning  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("shape", [(1, 16, 16, 1, 16), (257, 80, 272, 1, 48), (300, 336, 528, 3, 112),
                                   (1100, 400, 304, 1, 272), (900, 1040, 784, 2, 264)],
                         ids=lambda s: "T%d_%dx%d_l%dk%d" % s)
def test_big_tile_edges(sk, tuning, splits, shape):  # noqa: F811
    # bound: the repository's bf16 bar (two roundings to 8 bits, 2^-9 each, at up to three standard
    # deviations of the row they are judged against)
    tuning(sk.SK_TUNE_TILE, 0)
    tuning(sk.SK_TUNE_WTILE, 0)
    tuning(sk.SK_TUNE_WSPLITS, splits)
    T, d_in, d_out, l, k = shape
    check_all(sk, W.Workload("big_tile", T, d_in, d_out, l, k, "bf16", seed=60 + T), 2, single_call=True)


def test_more_big_tiles_than_cus(sk, tuning):  # noqa: F811
    """A work-group walks several tiles: the streams of loads cross from one into the next."""
    tuning(sk.SK_TUNE_TILE, 0)
    check_all(sk, W.Workload("big_tile_crew", 4100, 272, 4624, 1, 272, "bf16", seed=77), 2)


@pytest.mark.parametrize("shape", [(11383, 464, 336, 3, 240), (6000, 2064, 1040, 1, 1552)], ids=lambda s: "T%d_%dx%d_l%dk%d" % s)
def test_single_call_agrees_whichever_tile_its_first_products_take(sk, shape):  # noqa: F811
    """sk_linear_bwd puts the first two products beside each other on 128 x 128 tiles where the separate calls
    may take this one: the factor and bias gradients are the same bit for bit, as the header says."""
    import torch
    from test_gpu_parity import DeviceLayer
    T, d_in, d_out, l, k = shape
    sk.sk_set_plan(0)
    t = W.generate(W.Workload("single_call_tiles", T, d_in, d_out, l, k, "bf16", seed=T))
    one, sep = DeviceLayer(t, sk), DeviceLayer(t, sk)
    sk.check(one.bwd())
    sk.check(sep.bwd_input())
    sk.check(sep.bwd_weight())
    torch.cuda.synchronize()
    assert torch.equal(one.dU.view(torch.int32), sep.dU.view(torch.int32))
    assert torch.equal(one.db.view(torch.int32), sep.db.view(torch.int32))
    assert torch.allclose(one.dX.float(), sep.dX.float(), rtol=2e-2, atol=2e-2 * float(sep.dX.float().std()))
