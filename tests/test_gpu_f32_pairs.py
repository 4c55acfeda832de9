"""fp32: the single-call backward pass, whose products share launches in pairs, against the fp64 oracle and bit
for bit against the separate calls: no product split, either of the first two or both, the token contraction
split, pairs of unequal tiles (which go out apart), one token, a tile's edges."""
import pytest
import torch

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import DeviceLayer, _kernels_of, check_all, sk  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,launches", [
    ((1, 16, 16, 1, 16), 2), ((64, 256, 256, 1, 16), None), ((65, 80, 1040, 1, 48), None), ((129, 1040, 80, 3, 16), None),
    ((700, 2064, 1552, 2, 32), 4), ((4111, 208, 336, 1, 112), None), ((1300, 528, 2064, 1, 528), None),
    ((4367, 6016, 32, 1, 224), 5),   # the first pair on unequal tiles
], ids=lambda v: "T%d_%dx%d_l%dk%d" % v if isinstance(v, tuple) else "")
def test_shared_launches(sk, shape, launches):  # noqa: F811
    # bound of check_all: the repository's fp32 bar (4111 products carry at most 4111 * 2^-24 = 2.5e-4 of their
    # terms' magnitude, and the square root of that length in practice)
    T, d_in, d_out, l, k = shape
    w = W.Workload("f32_pairs", T, d_in, d_out, l, k, "f32", seed=90 + T)
    check_all(sk, w, 0, single_call=True)
    t = W.generate(w)
    one, sep = DeviceLayer(t, sk), DeviceLayer(t, sk)
    sk.check(one.bwd())
    sk.check(sep.bwd_input())
    sk.check(sep.bwd_weight())
    torch.cuda.synchronize()
    for name in ("dX", "dU", "db"):
        assert torch.equal(getattr(one, name).view(torch.int32), getattr(sep, name).view(torch.int32)), name
    names = _kernels_of(sk, DeviceLayer(t, sk), ("bwd",))
    assert launches is None or len(names) == launches, names
