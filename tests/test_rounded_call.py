"""sk_linear_bwd_rounded: bit for bit what sk_linear_bwd or sk_linear_bwd_two_sided and sk_round_gradients give, over the schedules that
leave their last sums to it and those that do not, with any of the gradients left out; every access inside the buffers (host
trace); arguments it refuses."""
import pytest

from paper_2601_15473_amd import libsk as sk

BASE = 1 << 44


def _traced(shape, two_sided, need):
    T, d_in, d_out, l, k, _ = shape
    R = l * k
    sizes = dict(x=T * d_in * 2, dY=T * d_out * 2, S=d_in * R * 2, U=R * d_out * 2, dX=T * d_in * 2, dU=R * d_out * 4, db=d_out * 4, dA=d_in * R // 2 * 4,
                 dU2=R * d_out * 2, db2=d_out * 2, dA2=d_in * R // 2 * 2, ws=need)
    P = {n: (i + 1) * BASE for i, n in enumerate(sizes)}
    sk.sk_trace_begin()
    try:
        st = sk.sk_linear_bwd_rounded(*(P[n] for n in ("x", "dY", "S", "U", "dX", "dU", "db")), P["dA"] if two_sided else None, P["dU2"],
                                      R // 2 if two_sided else R, P["db2"], P["dA2"] if two_sided else None, *shape, P["ws"], need)
        names = [n for n, _ in sk.sk_trace_kernels()]
    finally:
        trace, _ = sk.sk_trace_end()
    assert st == sk.SK_OK and names[-1] == "round_gradients_kernel"
    for at, n, write, _ in trace:
        name = list(sizes)[at // BASE - 1]
        assert at % BASE + n <= sizes[name] and (not write or name not in ("x", "dY", "S", "U")), (shape, name, at % BASE, n)
    return names


SHAPES = [(1000, 256, 1040, 2, 32), (4096, 768, 3072, 2, 64), (700, 2576, 1296, 2, 48), (1500, 768, 768, 2, 96), (300, 272, 2064, 2, 144),
          (600, 320, 208, 2, 16), (20, 64, 96, 2, 16), (5000, 1024, 2048, 2, 64), (12288, 4096, 1024, 2, 512)]


@pytest.mark.parametrize("two_sided", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "T%d_%dx%d_l%dk%d" % s)
def test_accesses_stay_inside_the_buffers(shape, two_sided):
    shape = (*shape, sk.SK_BF16)
    _traced(shape, two_sided, sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_TWO_SIDED if two_sided else sk.SK_OP_BWD, *shape))


def test_two_sided_bert_layer_in_four_launches():
    shape = (4096, 768, 3072, 2, 64, sk.SK_BF16)
    names = [n.split("<")[0] for n in _traced(shape, True, sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_TWO_SIDED, *shape))]
    assert names == ["dual_gemm_kernel", "factor_beside_expand_kernel", "gemm_bf16_kernel", "round_gradients_kernel"], names


def test_refusals():
    P = [i * BASE for i in range(1, 14)]
    good = dict(dA=None, dU2=P[8], rows=32, db2=P[9], dA2=None, shape=(64, 64, 96, 2, 16, sk.SK_BF16), ws=1 << 30)

    def call(**change):
        g = {**good, **change}
        return sk.sk_linear_bwd_rounded(*P[:7], g["dA"], g["dU2"], g["rows"], g["db2"], g["dA2"], *g["shape"], P[11], g["ws"])
    for change, want in ((dict(dU2=None, db2=None), sk.SK_ERR_INVALID_ARG), (dict(dU2=P[8] + 4), sk.SK_ERR_INVALID_ARG), (dict(rows=0), sk.SK_ERR_INVALID_ARG),
                         (dict(rows=33), sk.SK_ERR_INVALID_ARG), (dict(dA2=P[10]), sk.SK_ERR_INVALID_ARG), (dict(dA=P[7]), sk.SK_ERR_INVALID_ARG),
                         (dict(shape=(64, 64, 96, 2, 16, sk.SK_F32)), sk.SK_ERR_UNSUPPORTED), (dict(ws=16), sk.SK_ERR_WORKSPACE),
                         (dict(dA=P[7], dA2=P[10], shape=(64, 64, 96, 3, 16, sk.SK_BF16)), sk.SK_ERR_UNSUPPORTED)):
        assert call(**change) == want, change


@pytest.mark.gpu
@pytest.mark.parametrize("two_sided", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "T%d_%dx%d_l%dk%d" % s)
def test_bit_for_bit(shape, two_sided):
    import torch
    T, d_in, d_out, l, k = shape
    R = l * k
    g = torch.Generator(device="cuda").manual_seed(T)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    x, dY, S, U = rnd(T, d_in), rnd(T, d_out), rnd(d_in, R), rnd(R, d_out)
    args = (*shape, sk.SK_BF16)
    need = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_TWO_SIDED if two_sided else sk.SK_OP_BWD, *args)
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    f32 = lambda *s: torch.full(s, float("nan"), device="cuda")
    dX, dU, db, dA = rnd(T, d_in), f32(R, d_out), f32(d_out), f32(d_in, R // 2) if two_sided else None
    if two_sided:
        sk.check(sk.sk_linear_bwd_two_sided(x, dY, S, U, dX, dU, db, dA, *args, ws, need))
    else:
        sk.check(sk.sk_linear_bwd(x, dY, S, U, dX, dU, db, *args, ws, need))
    rows = R // 2 if two_sided else R
    want = [t.bfloat16() for t in (dX, dU[:rows], db) + ((dA,) if two_sided else ())]   # (both round to nearest even)
    for left_out in (None, 0, 1):
        outs = [torch.full(t.shape, float("nan"), dtype=torch.bfloat16, device="cuda") for t in want]
        to = outs[1:]
        given = [None if i == left_out else t for i, t in enumerate(to)]
        ws.fill_(255)
        sk.check(sk.sk_linear_bwd_rounded(x, dY, S, U, outs[0], f32(R, d_out), f32(d_out), f32(d_in, R // 2) if two_sided else None, given[0], rows, given[1],
                                          given[2] if two_sided else None, *args, ws, need))
        torch.cuda.synchronize()
        for i, (got, ref) in enumerate(zip(outs, want)):
            if i - 1 != left_out:
                assert torch.equal(got.view(torch.int16), ref.view(torch.int16)), (i, left_out)
