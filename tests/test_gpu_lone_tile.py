"""Products of 128 x 64 or 64 x 128 tiles in more than a round that take 128 x 128 ones in one: first contractions and expansions, ragged rows, columns
and contractions, on either side of a round of either -- against the fp64 oracle, and bit for bit the smaller tiles'."""
import pytest

from paper_2601_15473_amd import libsk
from paper_2601_15473_amd import workloads as W


def _kernels(call, T, d_in, d_out, R):
    P = [i << 44 for i in range(1, 9)]
    args = (T, d_in, d_out, 1, R, libsk.SK_BF16)
    op, pointers = {"fwd": (libsk.SK_OP_FWD, 5), "bwd_input": (libsk.SK_OP_BWD_INPUT, 4), "bwd_weight": (libsk.SK_OP_BWD_WEIGHT, 5)}[call]
    libsk.sk_trace_begin()
    try:
        libsk.check(getattr(libsk, "sk_linear_" + call)(*P[:pointers], *args, P[7], libsk.sk_linear_workspace_bytes(op, *args)))
        return [n for n, _ in libsk.sk_trace_kernels()]
    finally:
        libsk.sk_trace_end()


@pytest.mark.parametrize("call,shape,which,taken", [
    # (tokens, in, out, R): one row tile more than a round of 128 x 64 and exactly a round (128 of 128 x 128: 1.03 to 1.08 of the time, measured over 160 to 1536)
    ("fwd", (4224, 320, 64, 512), 0, True), ("fwd", (4096, 320, 64, 512), 0, False), ("fwd", (8192, 320, 64, 512), 0, True), ("fwd", (8193, 320, 64, 512), 0, False),
    ("fwd", (2049, 64, 1024, 160), 1, True), ("fwd", (2048, 64, 1024, 160), 1, False),
    # ... but forward over 2048 and more (0.88 to 0.97); not for the gradients
    ("fwd", (4096, 2048, 64, 512), 0, True), ("fwd", (4096, 2032, 64, 512), 0, False), ("fwd", (1024, 64, 2048, 2048), 1, True),
    ("bwd_input", (4096, 64, 2048, 512), 0, False), ("bwd_input", (4097, 64, 2048, 512), 0, True), ("bwd_input", (4075, 512, 256, 1200), 1, False),
    ("bwd_weight", (4096, 2560, 1536, 512), 0, False), ("bwd_weight", (4097, 2560, 1536, 512), 0, True),
    # a result at most 64 wide or high
    ("fwd", (32700, 512, 64, 400), 1, False), ("bwd_input", (32700, 64, 256, 256), 1, False), ("bwd_weight", (32768, 1024, 512, 64), 0, False),
    # a contraction of 128; 64 x 64 tiles; on either side of a round of 128 x 128
    ("fwd", (4224, 128, 64, 512), 0, False), ("fwd", (1000, 64, 1024, 160), 1, False),
    ("fwd", (2048, 64, 2048, 160), 1, True), ("fwd", (2049, 64, 2048, 160), 1, False),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_which_products_take_it(call, shape, which, taken):
    names = _kernels(call, *shape)
    kinds = {"fwd": "true, false", "bwd_input": "true, true", "bwd_weight": "false, true"}[call]
    assert (names[which] == f"gemm_bf16_kernel<128, 128, {kinds}, bf16, false, true>") == taken, names


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(3146, 272, 1168, 2, 384), (2425, 144, 1296, 1, 848), (4119, 336, 368, 2, 400), (863, 1040, 3664, 1, 544)],
                         ids=lambda v: "T%d_%dx%d_l%dk%d" % v)
def test_against_the_oracle_and_the_small_tiles(shape):
    import torch
    from test_gpu_parity import DeviceLayer, _kernels_of, check_all
    T, d_in, d_out, l, k = shape
    w = W.Workload("lone_tile", T, d_in, d_out, l, k, "bf16", seed=T)
    check_all(libsk, w, 0)                    # bound: the repository's bf16 bar (two roundings to 8 bits)
    t = W.generate(w)
    big, small = DeviceLayer(t, libsk), None
    names = _kernels_of(libsk, big, ("fwd", "bwd_input", "bwd_weight"))
    assert any(n.startswith("gemm_bf16_kernel<128, 128,") and n.endswith("true>") for n in names), names
    for call in ("fwd", "bwd_input"):
        libsk.check(getattr(big, call)())
    libsk.sk_set_tuning(libsk.SK_TUNE_TILE, 2)
    try:
        small = DeviceLayer(t, libsk)   # (its workspace for that plan)
        for call in ("fwd", "bwd_input"):
            libsk.check(getattr(small, call)())
    finally:
        libsk.sk_set_tuning(libsk.SK_TUNE_TILE, -1)
    torch.cuda.synchronize()
    for n in ("y", "dX")[:1 if d_out > 2048 else 2]:   # (over 3664 dY . U^T comes in ranges by itself, other sums)
        assert torch.equal(getattr(big, n).view(torch.int16), getattr(small, n).view(torch.int16)), n
