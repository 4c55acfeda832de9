"""Few tokens: the kernel that streams the weights once per 64 rows, at the edges of its row and column
tiles and of its chunks (one to five chunks over four waves, a contraction that ends inside a chunk, more
chunks than its ring holds, ranges by XCD) -- against the fp64 oracle."""
import pytest
import torch

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import _kernels_of, check_all, DeviceLayer, sk  # noqa: F401

pytestmark = pytest.mark.gpu

# shape, and the ranges of the forward's and of the input gradient's first contraction: eight, four (two
# XCDs to a range) and two (four), one row tile and several
SHAPES = [((1, 16, 16, 1, 16), 1, 1), ((8, 272, 144, 1, 48), 1, 1), ((9, 336, 2064, 2, 40), 1, 1), ((16, 3088, 80, 1, 160), 8, 1),
          ((33, 4112, 4128, 1, 272), 8, 8), ((64, 1040, 9232, 3, 16), 1, 8), ((65, 784, 3088, 2, 64), 1, 8), ((131, 768, 768, 2, 16), 1, 1),
          ((256, 2048, 528, 1, 256), 1, 1), ((40, 3136, 96, 1, 2064), 4, 1), ((20, 3136, 3152, 1, 4112), 2, 2),
          ((131, 3152, 80, 1, 80), 8, 1), ((130, 80, 3152, 1, 64), 1, 8)]


def _launches(sk, call):  # noqa: F811
    sk.sk_trace_begin()
    try:
        sk.check(call())
        return sk.sk_trace_kernels()
    finally:
        sk.sk_trace_end()


@pytest.mark.parametrize("shape,fwd_ranges,bwd_ranges", SHAPES, ids=lambda s: "T%d_%dx%d_l%dk%d" % s if isinstance(s, tuple) else str(s))
def test_few_rows(sk, shape, fwd_ranges, bwd_ranges):  # noqa: F811
    # bound: the repository's bf16 bar (the intermediate and the result rounded to 8 bits once each)
    T, d_in, d_out, l, k = shape
    w = W.Workload("few_rows", T, d_in, d_out, l, k, "bf16", seed=90 + T)
    sk.sk_set_plan(2)   # (by itself the planner fuses the shortest of these)
    dev = DeviceLayer(W.generate(w), sk)
    for call, ranges, second in (("fwd", fwd_ranges, d_out), ("bwd_input", bwd_ranges, d_in)):
        tiles = [(T + 63) // 64 * ((n + 63) // 64) for n in (l * k, second)]
        got = _launches(sk, getattr(dev, call))
        kernels = [n.split("<")[0] for n, _ in got]
        assert kernels == ["gemm_bf16_few_rows_kernel"] + ["reduce_to_bf16_kernel"] * (ranges > 1) + ["gemm_bf16_few_rows_kernel"], (call, got)
        if ranges > 1:
            per = 8 // ranges   # XCDs to a range; whole rounds of the eight
            assert got[0][1] == (tiles[0] + per - 1) // per * 8, (call, got)
    names = _kernels_of(sk, dev, ("fwd", "bwd_input"))
    assert len([n for n in names if "few_rows" in n]) == 4, names
    check_all(sk, w, 0, single_call=True)
    check_all(sk, w, 0, with_bias=False)
    check_all(sk, w, 2)
    # bit for bit from run to run
    y, dX = dev.y.clone(), dev.dX.clone()
    for t in (dev.y, dev.dX, dev.ws):
        t.fill_(0x55 if t is dev.ws else float("nan"))
    sk.check(dev.fwd())
    sk.check(dev.bwd_input())
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), dev.y.view(torch.int16)) and torch.equal(dX.view(torch.int16), dev.dX.view(torch.int16))
