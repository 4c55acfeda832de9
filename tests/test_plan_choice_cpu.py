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


FEW = ["few_rows", "few_rows"]
RANGES = ["few_rows", "reduce_to_bf16", "few_rows"]


@pytest.mark.parametrize("call,shape,want", [
    # few tokens, short first contraction (tokens, in, out, R): one fused launch
    ("fwd", (8, 128, 768, 32), ["chain_short"]), ("fwd", (32, 384, 768, 64), ["chain_short"]), ("fwd", (32, 400, 768, 64), FEW),
    ("fwd", (64, 512, 768, 64), ["chain_short"]), ("fwd", (64, 528, 768, 64), FEW), ("fwd", (8, 256, 768, 128), ["chain_short"]),
    ("fwd", (8, 272, 768, 128), FEW), ("bwd_input", (8, 768, 512, 32), ["chain_short"]), ("bwd_input", (8, 768, 528, 32), FEW),
    ("bwd_input", (64, 768, 640, 32), ["chain_short"]), ("bwd_input", (64, 768, 656, 32), FEW),
    # ... past 32 tokens a narrow sketch of a long input is split
    ("fwd", (32, 2944, 672, 16), FEW), ("fwd", (33, 1792, 672, 64), FEW), ("fwd", (33, 1808, 672, 64), ["kernel", "chain_short"]),
    ("fwd", (33, 1808, 672, 80), FEW), ("fwd", (200, 4096, 672, 16), ["kernel", "chain_short"]), ("fwd", (33, 4096, 64, 16), RANGES),
    # ... and an expansion of more than a round of work-groups is not theirs
    ("fwd", (16, 1024, 32768, 16), FEW), ("fwd", (17, 1024, 32768, 16), ["kernel", "chain_short"]),
    ("fwd", (64, 1024, 16384, 256), FEW), ("fwd", (64, 1024, 16400, 256), ["few_rows", "kernel"]),
    # runs of output tiles
    ("fwd", (2048, 768, 768, 128), ["chain_short"]), ("fwd", (4096, 768, 3072, 128), ["chain_small"]),
    ("fwd", (16384, 384, 384, 128), ["chain_short"]), ("fwd", (16384, 384, 512, 128), ["chain_small"]),
    ("fwd", (40000, 384, 256, 32), ["chain_short"]), ("fwd", (40000, 384, 384, 32), ["chain_small"]),
    # narrow ones over a long input: x . S in ranges beside dY . U^T, unless dX is one fused launch of many tokens
    ("bwd", (9600, 2400, 336, 112), ["dual_gemm", "reduce_to_bf16", "kernel", "chain_small"]),
    ("bwd", (9601, 2400, 336, 112), ["chain_small", "kernel", "reduce_to_bf16", "kernel", "reduce_splits"]),
    ("bwd", (9601, 4992, 336, 64), ["dual_gemm", "reduce_to_bf16", "kernel", "chain_small"]),
    ("bwd", (9601, 2400, 6160, 112), ["dual_gemm", "reduce_to_bf16", "kernel", "chain_small"]),
    # wide sketches: the first two contractions beside each other, or alone on 256 x 256 tiles
    ("bwd", (12288, 768, 768, 768), ["dual_gemm", "dual_gemm", "reduce_splits"]),
    ("bwd", (33222, 208, 48, 544), ["dual_gemm", "dual_gemm", "reduce_splits"]),
    # ... dX on 128 x 128 tiles beside Z^T.dY, or alone on 256 x 256 ones where those are far ahead
    ("bwd", (9153, 7792, 576, 416), ["dual_gemm", "reduce_to_bf16", "dual_gemm", "reduce_splits"]),
    ("bwd", (12520, 7296, 144, 352), ["kernel", "crew", "kernel", "reduce_to_bf16", "kernel", "reduce_splits"]),
    ("bwd", (12288, 4096, 1024, 1024), ["crew", "crew", "crew", "kernel", "reduce_splits"]),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v if isinstance(v, str) else "")
def test_kernels_on_either_side(call, shape, want):
    got = _kernels(call, *shape)
    assert [n or "kernel" for n in got] == want
