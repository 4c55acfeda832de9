"""The 256 x 128 tile that expansions of one round take: contractions of three to eight chunks, ending inside one, rows and columns
ragged, both operand orders, with and without a bias -- against the fp64 oracle, and bit for bit the 128 x 128 tile's."""
import pytest

from paper_2601_15473_amd import libsk
from paper_2601_15473_amd import workloads as W


def _kernels(call, T, d_in, d_out, R):
    P = [i << 44 for i in range(1, 9)]
    args = (T, d_in, d_out, 1, R, libsk.SK_BF16)
    libsk.sk_trace_begin()
    try:
        if call == "fwd":
            libsk.check(libsk.sk_linear_fwd(*P[:5], *args, P[7], libsk.sk_linear_workspace_bytes(libsk.SK_OP_FWD, *args)))
        else:
            libsk.check(libsk.sk_linear_bwd_input(*P[:4], *args, P[7], libsk.sk_linear_workspace_bytes(libsk.SK_OP_BWD_INPUT, *args)))
        return [n for n, _ in libsk.sk_trace_kernels()]
    finally:
        libsk.sk_trace_end()


@pytest.mark.parametrize("call,shape,taken", [
    # one round of 256 x 128 tiles, more than one of 128 x 128 ones
    ("fwd", (2048, 64, 4096, 256), True), ("fwd", (2049, 64, 4096, 256), False), ("fwd", (2048, 64, 2048, 256), False), ("fwd", (2049, 64, 2048, 256), True),
    ("fwd", (2048, 64, 4096, 128), False), ("fwd", (2048, 64, 4096, 144), True), ("bwd_input", (1100, 3856, 80, 208), True),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_which_expansions_take_it(call, shape, taken):
    names = _kernels(call, *shape)
    assert names[-1].startswith("gemm_bf16_kernel<256, 128, true,") == taken, names


@pytest.mark.gpu
@pytest.mark.parametrize("call,shape", [("fwd", (1100, 64, 3856, 1, 144)), ("fwd", (2060, 80, 2064, 2, 136)), ("fwd", (700, 48, 5520, 1, 496)),
                                        ("bwd_input", (1100, 3856, 80, 1, 208)), ("bwd_input", (2060, 2064, 64, 1, 320))],
                         ids=lambda v: "T%d_%dx%d_l%dk%d" % v if isinstance(v, tuple) else v)
def test_against_the_oracle_and_the_small_tile(call, shape):
    import torch
    from test_gpu_parity import DeviceLayer, _kernels_of, check_all
    T, d_in, d_out, l, k = shape
    w = W.Workload("expansion_tile", T, d_in, d_out, l, k, "bf16", seed=T + k)
    check_all(libsk, w, 0)                    # bound: the repository's bf16 bar (two roundings to 8 bits)
    check_all(libsk, w, 0, with_bias=False)
    t = W.generate(w)
    big = DeviceLayer(t, libsk)
    assert _kernels_of(libsk, big, (call,))[-1].startswith("gemm_bf16_kernel<256, 128, true,")
    libsk.sk_set_tuning(libsk.SK_TUNE_TILE, 1)
    small = DeviceLayer(t, libsk)   # (its workspace for that plan)
    try:
        libsk.check(getattr(small, call)())
    finally:
        libsk.sk_set_tuning(libsk.SK_TUNE_TILE, -1)
    torch.cuda.synchronize()
    out = "y" if call == "fwd" else "dX"
    assert torch.equal(getattr(big, out).view(torch.int16), getattr(small, out).view(torch.int16))
