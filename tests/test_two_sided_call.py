"""sk_linear_bwd_two_sided: every access inside the caller's buffers and the reported workspace (host trace), arguments
it refuses, and its outputs on the GPU against sk_linear_bwd and sk_linear_bwd_weight_first -- over the schedules that
keep dY . U_cat^T (narrow sketches, wide ones in shared launches and apart, fp32) and those that do not."""
import numpy as np
import pytest

from paper_2601_15473_amd import libsk as sk
from test_workspace_bounds_cpu import Buffers, _forced, _shape


def _call(P, shape, need):
    return sk.sk_linear_bwd_two_sided(P["x"], P["dY"], P["S"], P["U"], P["dX"], P["dU"], P["db"], P["dA"], *shape, P["ws"], need)


def test_accesses_stay_inside_the_buffers():
    r = np.random.default_rng(7)
    for _ in range(4000):
        shape, plan, forced = _shape(r), int(r.integers(0, 4)), _forced(r)
        R = shape[3] * shape[4]
        need = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_TWO_SIDED, *shape)
        if R % 32:
            assert need == 2 ** 64 - 1
            continue
        sk.sk_set_plan(plan)
        for knob, value in forced:
            sk.sk_set_tuning(knob, value)
        try:
            need = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_TWO_SIDED, *shape)
            buf = Buffers(*shape, R // 2)
            sk.sk_trace_begin()
            try:
                st = _call(buf.base, shape, need)
            finally:
                trace, launches = sk.sk_trace_end()
            assert st == sk.SK_OK, (shape, st)
            buf.check(trace, launches, need, ("dX", "dU", "db", "dA"), (shape, plan, forced))
        finally:
            for knob, _ in forced:
                sk.sk_set_tuning(knob, -1)
            sk.sk_set_plan(0)


def test_refusals():
    shape = (64, 64, 96, 2, 16, sk.SK_BF16)
    P = Buffers(*shape, 16).base
    need = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_TWO_SIDED, *shape)
    assert _call(P, shape, need - 1) == sk.SK_ERR_WORKSPACE
    for name in ("x", "dY", "S", "U", "dX", "dU", "dA", "ws"):
        assert _call({**P, name: None}, shape, need) == sk.SK_ERR_INVALID_ARG, name
        assert _call({**P, name: P[name] + 4}, shape, need) == sk.SK_ERR_INVALID_ARG, name
    assert _call(P, (64, 64, 96, 3, 16, sk.SK_BF16), 1 << 30) == sk.SK_ERR_UNSUPPORTED   # R = 48: halves of 24 columns


@pytest.mark.gpu
@pytest.mark.parametrize("T,d_in,d_out,l,k,dtype,shares", [
    (1000, 256, 1040, 2, 32, "bf16", True), (4096, 768, 3072, 2, 64, "bf16", True), (700, 2576, 1296, 2, 48, "bf16", True),   # narrow
    (1500, 768, 768, 2, 96, "bf16", True), (300, 272, 2064, 2, 144, "bf16", None),                                            # wide
    (600, 320, 208, 2, 16, "bf16", False),                                                                                    # one pass
    (333, 208, 336, 2, 16, "f32", True), (900, 1040, 2064, 4, 64, "f32", True),
], ids=lambda v: str(v))
def test_outputs(T, d_in, d_out, l, k, dtype, shares):
    import torch
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(T)
    R, half = l * k, l * k // 2
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, dY, S, U = rnd(T, d_in).to(td), rnd(T, d_out).to(td), (rnd(d_in, R) / k ** 0.5).to(td), (rnd(R, d_out) / R ** 0.5).to(td)
    shape = (T, d_in, d_out, l, k, sk.DTYPES[dtype])
    f32 = lambda *s: torch.full(s, float("nan"), device="cuda")

    class Out:
        def __init__(self):
            self.dX, self.dU, self.db, self.dA = torch.empty(T, d_in, dtype=td, device="cuda"), f32(R, d_out), f32(d_out), f32(d_in, half)
    one, two = Out(), Out()
    need = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_TWO_SIDED, *shape)
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    call = lambda: sk.sk_linear_bwd_two_sided(x, dY, S, U, one.dX, one.dU, one.db, one.dA, *shape, ws, need)
    sk.check(call())
    apart = max(sk.sk_linear_workspace_bytes(op, *shape) for op in (sk.SK_OP_BWD, sk.SK_OP_BWD_WEIGHT_FIRST))
    ws2 = torch.empty(apart, dtype=torch.uint8, device="cuda")
    sk.check(sk.sk_linear_bwd(x, dY, S, U, two.dX, two.dU, two.db, *shape, ws2, apart))
    sk.check(sk.sk_linear_bwd_weight_first(x, U, dY, two.dA, *shape[:5], half, half, shape[5], ws2, apart))
    torch.cuda.synchronize()
    for name in ("dX", "dU", "db"):
        assert torch.equal(getattr(one, name), getattr(two, name)), name
    want = x.double().cpu().T @ (dY.double().cpu() @ U[half:].double().cpu().T) / l
    # bounds: the repository's bars, here over whole tensors: G rounded to 8 bits once, or fp32 sums
    bar = 1e-2 if dtype == "bf16" else 1e-5
    off = [float((got.double().cpu() - want).norm() / want.norm()) for got in (one.dA, two.dA)]
    assert max(off) < bar
    if dtype == "bf16":
        # The sums of G in another order, before the same single rounding: what the rounding leaves (2^-9 / sqrt(3) of it) is
        # the error of both, and only elements whose fp32 sums lie on either side of a rounding boundary differ.  Twenty-five layers on two
        # seeds: the error 1.000004 times the separate call's on average, at most 1.0003.
        assert off[0] < 1.005 * off[1], off
    if shares is not None:
        sk.sk_profile_begin(32)
        sk.check(call())
        n = len(sk.sk_profile_end(32))
        sk.sk_profile_begin(32)
        sk.check(sk.sk_linear_bwd(x, dY, S, U, two.dX, two.dU, two.db, *shape, ws2, apart))
        n -= len(sk.sk_profile_end(32))
        assert (n <= 2) == shares, n   # x^T . G and the sum of its token ranges, or dY . U^T again as well
