"""The backward pass of a wide sketch in shared launches, over the pairs of products it is made of: dY . U^T and x . S whole or in
ranges on either tile, dX on each of its tiles, one range of tokens and several, all sizes ragged -- against the fp64 oracle, dU and
db bit for bit those of the separate call, run to run the same."""
import pytest
import torch

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import DeviceLayer, _kernels_of, check_all, sk  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,launches", [
    # both whole: 64 x 64 tiles, 128 x 128 tiles, one range of tokens, dX on 64 x 64 tiles
    ((735, 560, 592, 2, 216), 3), ((3642, 1360, 784, 1, 496), 3), ((556, 1136, 1232, 1, 176), 2), ((281, 80, 80, 1, 784), 2),
    # dY . U^T in ranges, x . S, both
    ((339, 1200, 3824, 1, 464), 3), ((1212, 3920, 608, 1, 272), 4), ((861, 2240, 3568, 1, 144), 3), ((2803, 1792, 3888, 2, 176), 4),
    ((597, 2288, 112, 1, 272), 4),
], ids=lambda v: "T%d_%dx%d_l%dk%d" % v if isinstance(v, tuple) else "")
def test_against_the_oracle_and_the_separate_call(sk, shape, launches):  # noqa: F811
    T, d_in, d_out, l, k = shape
    w = W.Workload("wide_pairs", T, d_in, d_out, l, k, "bf16", seed=T)
    check_all(sk, w, 0, single_call=True)   # bound: the repository's bf16 bar (two roundings to 8 bits)
    t = W.generate(w)
    names = _kernels_of(sk, DeviceLayer(t, sk), ("bwd",))
    assert len(names) == launches and sum(n.startswith("dual_gemm_kernel") for n in names) == 2, names
    one, again, sep = DeviceLayer(t, sk), DeviceLayer(t, sk), DeviceLayer(t, sk)
    again.ws.fill_(255)
    sk.check(one.bwd())
    sk.check(again.bwd())
    sk.check(sep.bwd_weight())
    torch.cuda.synchronize()
    bits = lambda x: x.view(torch.int16 if x.element_size() == 2 else torch.int32)
    for n in ("dU", "db"):
        assert torch.equal(bits(getattr(one, n)), bits(getattr(sep, n))), n
    for n in ("dX", "dU", "db"):
        assert torch.equal(bits(getattr(one, n)), bits(getattr(again, n))), n
