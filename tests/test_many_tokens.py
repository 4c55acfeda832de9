"""The factor gradient over millions of tokens: a row of the recomputed Z^T = S^T . x^T is all tokens long, so
rows of one tile lie far apart -- past 2^22 tokens 256 of them span more than the 2 GB a kernel's 32-bit
offsets reach, past 8.4 million 128 of them do."""
import re

import numpy as np
import pytest
import torch

from oracle import sklinear as O
from paper_2601_15473_amd import libsk as sk
from paper_2601_15473_amd import workloads as W

BASE = 1 << 44      # made-up device addresses, far apart; never dereferenced


@pytest.mark.parametrize("width", [(256, 16), (4096, 4096), (48, 2048)], ids=lambda w: "R%d_out%d" % w)
@pytest.mark.parametrize("tokens", [2 ** 22 - 64, 2 ** 22, 2 ** 22 + 64, 8454656, 8454657, 2 ** 23 + 2 ** 20, 2 ** 24])
@pytest.mark.parametrize("wtile", [-1, 0, 1, 2])
def test_rows_of_a_tile_stay_within_a_window(tokens, width, wtile):
    R, out = width
    args = (tokens, 256, out, 1, R, sk.SK_BF16)
    sk.sk_set_tuning(sk.SK_TUNE_WTILE, wtile)
    try:
        ws = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_WEIGHT, *args)
        sk.sk_trace_begin()
        st = sk.sk_linear_bwd_weight(BASE, 2 * BASE, 3 * BASE, 4 * BASE, 5 * BASE, *args, 6 * BASE, ws)
        names = [n for n, _ in sk.sk_trace_kernels()]
        sk.sk_trace_end()
    finally:
        sk.sk_set_tuning(sk.SK_TUNE_WTILE, -1)
    assert st == sk.SK_OK
    # Z^T . dY: the kernels with a k-contiguous first operand
    rows = [int(m.group(1)) for n in names if (m := re.match(r"gemm_\w+<(\d+), \d+, (?:2, 4, )?true", n.replace("far_kernel<", "far_kernel<256, 256, ")))]
    assert rows, names
    ldz = (tokens + 63) // 64 * 64
    for r in rows:
        assert ((r - 1) * ldz + 64) * 2 < 2 ** 31, (names, ldz)


@pytest.mark.gpu
@pytest.mark.parametrize("blocks,d_in,R,kernel", [
    (1025, 144, 256, "gemm_bf16_far_kernel<false, true, bf16>"),   # Z^T on 256 x 256 tiles
    (2065, 16, 128, "gemm_bf16_kernel<64, 128, true, false, float, true>"),        # Z^T . dY past 8.4 million
], ids=["T4198400_R256", "T8458240_R128"])
def test_factor_gradient_over_millions_of_tokens(blocks, d_in, R, kernel):
    # A block of 4096 tokens repeated: the gradients are the block's, `blocks` times.  Bound: the
    # repository's bf16 bar (Z rounded to 8 bits); the fp32 sums of at most 8.4 M / 32 products add 16-deep
    # MFMA terms one after the other, 2^-24 each: 264 000 / 16 * 6e-8 = 1e-3 at worst.
    from skgpu import TOL, rel_err, to_dev, to_f64
    w = W.Workload("many_tokens", 4096, d_in, 16, 1, R, "bf16", seed=5)
    t = W.generate(w)
    v = {n: a.astype(np.float64) for n, a in t.value.items()}
    x, dY = (to_dev(t.stored[n], "bf16").repeat(blocks, 1) for n in ("x", "dY"))
    S = to_dev(t.S_cat(), "bf16")
    args = (x.shape[0], d_in, 16, 1, R, sk.SK_BF16)
    nbytes = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_WEIGHT, *args)
    ws = torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda")   # (NaN, so that what is not written shows)
    dU = torch.empty((R, 16), dtype=torch.float32, device="cuda")
    db = torch.empty((16,), dtype=torch.float32, device="cuda")
    print(f"case T={x.shape[0]} in={d_in} R={R}", flush=True)
    sk.sk_profile_begin(16)
    sk.check(sk.sk_linear_bwd_weight(x, S, dY, dU, db, *args, ws, nbytes, torch.cuda.current_stream().cuda_stream))
    names = [r[0] for r in sk.sk_profile_end(16)]
    torch.cuda.synchronize()
    assert rel_err(to_f64(dU), blocks * O.grad_factors(v["x"], v["S"], v["dY"]).reshape(R, 16)) <= TOL["bf16"]
    assert rel_err(to_f64(db), blocks * O.grad_bias(v["dY"])) <= TOL["bf16"]
    assert any(n.startswith(kernel) for n in names), names


@pytest.mark.parametrize("tokens,out,R", [(98304, 11008, 2048), (131072, 8192, 2048), (300000, 4096, 4096)])
def test_operands_past_two_gib_keep_their_tile(tokens, out, R):
    assert tokens * out * 2 >= 2 ** 31
    args = (tokens, 256, out, 1, R, sk.SK_BF16)
    sk.sk_trace_begin()
    st = sk.sk_linear_bwd_weight(BASE, 2 * BASE, 3 * BASE, 4 * BASE, 5 * BASE, *args, 6 * BASE,
                                 sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_WEIGHT, *args))
    names = [n for n, _ in sk.sk_trace_kernels()]
    sk.sk_trace_end()
    assert st == sk.SK_OK and not any(n.startswith("gemm_bf16_kernel") for n in names), names


@pytest.mark.gpu
@pytest.mark.parametrize("blocks,rest", [(24, "gemm_bf16_with_colsum_kernel<256, 256, 2, 4, true, false, float>"),
                                         (48, "gemm_bf16_far_with_colsum_kernel<true, false, float>")], ids=["T98376", "T196752"])
def test_factor_gradient_of_operands_past_two_gib(blocks, rest):
    """Z^T . dY with more than 2 GB of dY under one column of tiles: a round of whole-token tiles, and with
    twice the tokens also the split rest.  Blocks of an odd length, repeated; bound as above."""
    from skgpu import TOL, rel_err, to_dev, to_f64
    d_out, R = 11008, 2048
    w = W.Workload("past_two_gib", 4099, 16, d_out, 1, R, "bf16", seed=6)
    t = W.generate(w)
    v = {n: a.astype(np.float64) for n, a in t.value.items()}
    x, dY = (to_dev(t.stored[n], "bf16").repeat(blocks, 1) for n in ("x", "dY"))
    assert dY.numel() * 2 > 2 ** 31
    S = to_dev(t.S_cat(), "bf16")
    args = (x.shape[0], 16, d_out, 1, R, sk.SK_BF16)
    nbytes = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_WEIGHT, *args)
    ws = torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda")
    dU = torch.empty((R, d_out), dtype=torch.float32, device="cuda")
    db = torch.empty((d_out,), dtype=torch.float32, device="cuda")
    print(f"case T={x.shape[0]} out={d_out} R={R}", flush=True)
    sk.sk_profile_begin(16)
    sk.check(sk.sk_linear_bwd_weight(x, S, dY, dU, db, *args, ws, nbytes, torch.cuda.current_stream().cuda_stream))
    names = [r[0] for r in sk.sk_profile_end(16)]
    torch.cuda.synchronize()
    assert rel_err(to_f64(dU), blocks * O.grad_factors(v["x"], v["S"], v["dY"]).reshape(R, d_out)) <= TOL["bf16"]
    assert rel_err(to_f64(db), blocks * O.grad_bias(v["dY"])) <= TOL["bf16"]
    assert names[1:3] == ["gemm_bf16_far_kernel<true, false, float>", rest], names


@pytest.mark.gpu
@pytest.mark.parametrize("tokens,blocks,d_in,nc", [(4099, 65, 4096, 4096), (300, 1, 4112, 3856), (1, 1, 4096, 4096), (63, 1, 8192, 2048)],
                         ids=lambda v: str(v))
def test_first_stage_gradient_on_big_tiles(tokens, blocks, d_in, nc):
    """x^T . G on 256 x 256 tiles, neither operand k-contiguous: what lies past the contraction comes from
    the ends of both arrays.  The first case has more than 2 GB of either.  Bound: G rounded to 8 bits errs
    by 2^-9 / sqrt(6) of its size in the root mean square, the largest of 2^24 such errors by 5.5 times that,
    4.4e-3, against rows whose size varies by a fifth where 256 products make up G: 6e-3."""
    from skgpu import TOL, rel_err, to_dev, to_f64
    w = W.Workload("first_stage_big", tokens, d_in, 256, 1, nc, "bf16", seed=7)
    t = W.generate(w)
    v = {n: a.astype(np.float64) for n, a in t.value.items()}
    x, dY = (to_dev(t.stored[n], "bf16").repeat(blocks, 1) for n in ("x", "dY"))
    U = to_dev(t.U_cat(), "bf16")
    args = (x.shape[0], d_in, 256, 1, nc)
    nbytes = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_WEIGHT_FIRST, *args, sk.SK_BF16)
    ws = torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda")
    dA = torch.full((d_in, nc), float("nan"), dtype=torch.float32, device="cuda")
    print(f"case T={x.shape[0]} in={d_in} columns={nc}", flush=True)
    sk.sk_profile_begin(16)
    sk.check(sk.sk_linear_bwd_weight_first(x, U, dY, dA, *args, 0, nc, sk.SK_BF16, ws, nbytes,
                                           torch.cuda.current_stream().cuda_stream))
    names = [r[0] for r in sk.sk_profile_end(16)]
    torch.cuda.synchronize()
    G = v["dY"] @ v["U"].reshape(nc, 256).T
    assert rel_err(to_f64(dA), blocks * (v["x"].T @ G)) <= TOL["bf16"]
    kernel = "gemm_bf16_far_kernel<" if blocks > 1 else "gemm_bf16_crew_kernel<256, 256, 2, 4, "
    assert kernel + "false, false, float>" in names, names
