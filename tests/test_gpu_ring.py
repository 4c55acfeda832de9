"""The GEMM tiles on a ring of chunks in LDS, which launches of one round take: contractions of fewer chunks than the
ring has slots, ending inside a chunk, one chunk past a turn of the ring, ragged rows and columns, split
contractions, column sums, two products in one launch -- against the fp64 oracle, and on either side of the round
against the staged tile, bit for bit (the same sums in the same order)."""
import pytest
import torch

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import DeviceLayer, _kernels_of, check_all, sk, tuning  # noqa: F401

pytestmark = pytest.mark.gpu


def _rings(names):
    return [n for n in names if n.startswith("gemm_bf16_kernel<") and n.count(",") == 6]


@pytest.mark.parametrize("tile", [1, 2, 4], ids=["128x128", "128x64", "64x64"])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("shape", [(300, 16, 48, 1, 16), (129, 272, 336, 1, 272), (1300, 400, 208, 3, 112), (515, 1040, 80, 1, 144)],
                         ids=lambda s: "T%d_%dx%d_l%dk%d" % s)
def test_ring_edges(sk, tuning, tile, splits, shape):  # noqa: F811
    # bound: the repository's bf16 bar (two roundings to 8 bits, 2^-9 each, at up to three standard
    # deviations of the row they are judged against)
    tuning(sk.SK_TUNE_TILE, tile)
    tuning(sk.SK_TUNE_WTILE, tile)
    tuning(sk.SK_TUNE_WSPLITS, splits)
    T, d_in, d_out, l, k = shape
    w = W.Workload("ring", T, d_in, d_out, l, k, "bf16", seed=70 + T)
    check_all(sk, w, 2, single_call=True)
    sk.sk_set_plan(2)
    try:
        names = _kernels_of(sk, DeviceLayer(W.generate(w), sk), ("fwd", "bwd_weight"))
    finally:
        sk.sk_set_plan(0)
    assert len(_rings(names)) >= (1 if tile == 2 else 3), names


@pytest.mark.parametrize("tokens", [512 * 64, 512 * 64 + 64])
def test_either_side_of_a_round(sk, tuning, tokens):  # noqa: F811
    """x . S and G . S^T of 64 x 64 tiles, R = in = 64: 512 tiles on the ring, 513 staged."""
    tuning(sk.SK_TUNE_TILE, 4)
    t = W.generate(W.Workload("ring_round", tokens, 64, 64, 1, 64, "bf16", seed=5))
    dev = DeviceLayer(t, sk)
    sk.sk_set_plan(2)
    try:
        names = _kernels_of(sk, dev, ("fwd",))
        sk.check(dev.fwd())
    finally:
        sk.sk_set_plan(0)
    torch.cuda.synchronize()
    assert len(_rings(names)) == (2 if tokens == 512 * 64 else 0), names
    n = 512 * 64
    x, S, U, b = (torch.from_numpy(t.value[k].astype("float32")).cuda() for k in ("x", "S", "U", "b"))
    Z = (x[:n].double() @ S.reshape(64, 64).double()).bfloat16().double()
    want = Z @ U.reshape(64, 64).double() + b.double()
    assert float((dev.y[:n].double() - want).abs().max() / want.std()) < 5e-2   # two roundings to 8 bits at up to six deviations


def test_two_products_on_rings(sk):  # noqa: F811
    for shape in ((568, 640, 352, 1, 48), (1500, 768, 768, 1, 192)):
        T, d_in, d_out, l, k = shape
        w = W.Workload("ring_pair", T, d_in, d_out, l, k, "bf16", seed=T)
        check_all(sk, w, 0, single_call=True)
