"""The single-call backward pass of a narrow sketch over a long input, whose recomputed x . S is cut into ranges and
shares a launch with dY . U^T: against the fp64 oracle, the factor and bias gradients bit for bit those of
the separate call, ragged in every dimension, with and without the bias gradient."""
import pytest
import torch

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import DeviceLayer, _kernels_of, check_all, sk  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(300, 4112, 1040, 1, 16), (1030, 2064, 2320, 2, 32), (515, 3088, 1552, 1, 80), (1500, 2576, 1296, 1, 96),
                                   (2049, 4096, 528, 1, 128), (3652, 3376, 1088, 1, 80)], ids=lambda s: "T%d_%dx%d_l%dk%d" % s)
def test_split_recomputation_beside_the_other_product(sk, shape):  # noqa: F811
    # bound of check_all: the repository's bf16 bar (two roundings to 8 bits)
    T, d_in, d_out, l, k = shape
    w = W.Workload("long_narrow", T, d_in, d_out, l, k, "bf16", seed=T)
    check_all(sk, w, 0, single_call=True)
    t = W.generate(w)
    names = _kernels_of(sk, DeviceLayer(t, sk), ("bwd",))
    # (300 tokens are one range: no sums behind the factor gradient beside the expansion)
    assert [n.split("<")[0] for n in names[:2]] == ["dual_gemm_kernel", "reduce_to_bf16_kernel"] and len(names) == (3 if T == 300 else 4), names
    one, sep = DeviceLayer(t, sk), DeviceLayer(t, sk)
    sk.check(one.bwd())
    sk.check(sep.bwd_weight())
    torch.cuda.synchronize()
    assert torch.equal(one.dU.view(torch.int32), sep.dU.view(torch.int32))
    assert torch.equal(one.db.view(torch.int32), sep.db.view(torch.int32))
