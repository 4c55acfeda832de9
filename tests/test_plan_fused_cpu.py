"""Where a narrow sketch's two contractions are fused (host trace, no GPU): on either side of each line of the rule."""
import pytest

from paper_2601_15473_amd import libsk as sk
from test_plan_choice_cpu import _kernels


@pytest.mark.parametrize("call,shape,fused", [
    # (tokens, in, out, R): up to 1536 long in one round of work-groups, at any number of slices
    ("fwd", (257, 1536, 4096, 32), True), ("fwd", (257, 1552, 4096, 32), False), ("bwd_input", (1064, 5168, 1344, 128), True),
    ("fwd", (4096, 1536, 2048, 64), True), ("fwd", (4096, 1552, 2048, 64), False), ("fwd", (4096, 1536, 4096, 64), True),
    # length times slices up to 6144: in one round, or up to 1536 long
    ("fwd", (16384, 3072, 3072, 64), True), ("fwd", (16448, 3072, 3072, 64), False), ("fwd", (16448, 1536, 3072, 64), True),
    ("bwd_input", (10442, 5136, 2928, 64), False), ("bwd_input", (16384, 6144, 768, 32), True), ("bwd_input", (16384, 768, 6144, 32), True),
    ("bwd_input", (16384, 768, 6160, 32), False),
    # a longer walk past a round: above R = 64, or from one and a half rounds on, where no slice repeats it; 64-row tiles ...
    ("fwd", (16448, 3072, 3072, 80), True), ("fwd", (24576, 3072, 3072, 64), False), ("fwd", (24577, 3072, 3072, 64), True),
    ("bwd_input", (20000, 768, 3072, 128), True), ("fwd", (16448, 3072, 3088, 128), False), ("bwd_input", (24747, 4576, 2864, 96), False),
    # ... and 128-row ones
    ("bwd_input", (65536, 768, 3072, 128), True), ("fwd", (262144, 3072, 768, 64), True), ("fwd", (32832, 3072, 768, 96), True),
    ("fwd", (49152, 1552, 768, 64), False), ("fwd", (49153, 1552, 768, 64), True), ("fwd", (65536, 2048, 3088, 128), False),
    ("fwd", (65536, 6144, 768, 128), True), ("fwd", (65536, 6160, 768, 128), False),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_fused_or_split(call, shape, fused):
    names = _kernels(call, *shape)
    assert (len(names) == 1) == fused and names[-1] in ("chain_short", "chain_small"), names


@pytest.mark.parametrize("call,shape,taken", [
    # long walks in more than a round, which a workspace would have split, and walks too long for any
    ("fwd", (16448, 3072, 3072, 64), True), ("bwd_input", (10442, 5136, 1152, 64), True), ("bwd_input", (16448, 768, 6144, 32), True),
    ("bwd_input", (16448, 768, 6160, 32), False), ("fwd", (257, 1552, 4096, 32), False), ("fwd", (257, 6160, 768, 32), False),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_calls_without_a_workspace(call, shape, taken):
    args = (*shape[:3], 1, shape[3], sk.SK_BF16)
    P = [i << 44 for i in range(1, 6)]
    sk.sk_trace_begin()
    st = sk.sk_linear_fwd(*P, *args, None, 0) if call == "fwd" else sk.sk_linear_bwd_input(*P[:4], *args, None, 0)
    names = [n for n, _ in sk.sk_trace_kernels()]
    sk.sk_trace_end()
    assert st == (sk.SK_OK if taken else sk.SK_ERR_WORKSPACE) and len(names) == int(taken), (st, names)
