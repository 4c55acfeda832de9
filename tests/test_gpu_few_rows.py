"""Few tokens: the kernel that streams the weights once per 64 rows, at the edges of its row and column
tiles and of its chunks (one to five chunks over four waves, a contraction that ends inside a chunk, more
chunks than its ring holds, ranges by XCD) -- against the fp64 oracle."""
import pytest

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import _kernels_of, check_all, DeviceLayer, sk  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(1, 16, 16, 1, 16), (8, 272, 144, 1, 48), (9, 336, 2064, 2, 40), (16, 3088, 80, 1, 160),
          (33, 4112, 4128, 1, 272), (64, 1040, 9232, 3, 16), (65, 784, 3088, 2, 64), (131, 768, 768, 2, 16),
          (256, 2048, 528, 1, 256)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "T%d_%dx%d_l%dk%d" % s)
def test_few_rows(sk, shape):  # noqa: F811
    # bound: the repository's bf16 bar (the intermediate and the result rounded to 8 bits once each)
    T, d_in, d_out, l, k = shape
    w = W.Workload("few_rows", T, d_in, d_out, l, k, "bf16", seed=90 + T)
    names = _kernels_of(sk, DeviceLayer(W.generate(w), sk), ("fwd", "bwd_input"))
    assert any("few_rows" in n for n in names), names
    check_all(sk, w, 0, single_call=True)
    check_all(sk, w, 0, with_bias=False)
