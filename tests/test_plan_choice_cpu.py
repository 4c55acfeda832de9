"""Which kernels the automatic plans launch on either side of their lines (host trace, no GPU)."""
import pytest

from paper_2601_15473_amd import libsk as sk

BASE = 1 << 44      # made-up device addresses, far apart; never dereferenced


def _kernels(call, *shape):
    args = (*shape[:3], 1, shape[3], sk.SK_BF16)
    op = {"fwd": sk.SK_OP_FWD, "bwd_input": sk.SK_OP_BWD_INPUT, "bwd": sk.SK_OP_BWD}[call]
    P = [i * BASE for i in range(1, 9)]
    ws = (P[7], sk.sk_linear_workspace_bytes(op, *args))
    sk.sk_trace_begin()
    if call == "fwd":
        st = sk.sk_linear_fwd(*P[:5], *args, *ws)
    elif call == "bwd_input":
        st = sk.sk_linear_bwd_input(*P[:4], *args, *ws)
    else:
        st = sk.sk_linear_bwd(*P[:7], *args, *ws)
    names = [n.split("<")[0].replace("gemm_bf16_", "").replace("_kernel", "") for n, _ in sk.sk_trace_kernels()]
    sk.sk_trace_end()
    assert st == sk.SK_OK
    return names


@pytest.mark.parametrize("call,shape,want", [
    # runs of output tiles
    ("fwd", (2048, 768, 768, 128), ["chain_short"]), ("fwd", (4096, 768, 3072, 128), ["chain_small"]),
    ("fwd", (16384, 384, 384, 128), ["chain_short"]), ("fwd", (16384, 384, 512, 128), ["chain_small"]),
    ("fwd", (40000, 384, 256, 32), ["chain_short"]), ("fwd", (40000, 384, 384, 32), ["chain_small"]),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v if isinstance(v, str) else "")
def test_kernels_on_either_side(call, shape, want):
    got = _kernels(call, *shape)
    assert [n or "kernel" for n in got] == want
