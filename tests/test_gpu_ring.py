"""The GEMM tiles on a ring of chunks in LDS, which launches of one round take: contractions of fewer chunks than the
ring has slots, ending inside a chunk, one chunk past a turn of the ring, ragged rows and columns, split
contractions, column sums, two products in one launch -- against the fp64 oracle, and on either side of a round
against the staged tile, bit for bit (the same sums in the same order): both results, every tile that has a ring."""
import pytest
import torch

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import DeviceLayer, _kernels_of, check_all, sk, tuning  # noqa: F401

pytestmark = pytest.mark.gpu


def _rings(names):
    return [n for n in names if n.startswith("gemm_bf16_kernel<") and n.count(",") == 6]


@pytest.mark.parametrize("tile", [1, 2, 4], ids=["128x128", "128x64", "64x64"])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("shape", [(300, 16, 48, 1, 16), (129, 272, 336, 1, 272), (1300, 400, 208, 3, 112), (515, 1040, 80, 1, 144)],
                         ids=lambda s: "T%d_%dx%d_l%dk%d" % s)
def test_ring_edges(sk, tuning, tile, splits, shape):  # noqa: F811
    # bound: the repository's bf16 bar (two roundings to 8 bits, 2^-9 each, at up to three standard
    # deviations of the row they are judged against)
    tuning(sk.SK_TUNE_TILE, tile)
    tuning(sk.SK_TUNE_WTILE, tile)
    tuning(sk.SK_TUNE_WSPLITS, splits)
    T, d_in, d_out, l, k = shape
    w = W.Workload("ring", T, d_in, d_out, l, k, "bf16", seed=70 + T)
    check_all(sk, w, 2, single_call=True)
    sk.sk_set_plan(2)
    try:
        names = _kernels_of(sk, DeviceLayer(W.generate(w), sk), ("fwd", "bwd_weight"))
    finally:
        sk.sk_set_plan(0)
    assert len(_rings(names)) >= (1 if tile == 2 else 3), names


def _two_gemms(sk, dev):
    sk.sk_set_plan(2)
    try:
        names = _kernels_of(sk, dev, ("fwd",))
    finally:
        sk.sk_set_plan(0)
    torch.cuda.synchronize()
    return names


@pytest.mark.parametrize("tile,rows,d,R", [(4, 512 * 64, 64, 64), (1, 128 * 128, 208, 256)], ids=["64x64", "128x128"])
def test_either_side_of_a_round(sk, tuning, tile, rows, d, R):  # noqa: F811
    """x . S and Z . U of square tiles, the last work-group of a round and one tile of rows more: ring and staged bit for bit."""
    tuning(sk.SK_TUNE_TILE, tile)
    more = rows + (64 if tile == 4 else 128)
    t = W.generate(W.Workload("ring_round", more, d, R, 1, R, "bf16", seed=5))
    staged, ring = DeviceLayer(t, sk), DeviceLayer(W.generate(W.Workload("ring_round", rows, d, R, 1, R, "bf16", seed=5)), sk)
    ring.x.copy_(staged.x[:rows])
    for n in ("S_cat", "U_cat", "b"):
        getattr(ring, n).copy_(getattr(staged, n))
    for dev, want in ((staged, 0), (ring, 2)):
        names = _two_gemms(sk, dev)
        assert len(names) == 2 and len(_rings(names)) == want, names
    assert torch.equal(ring.y, staged.y[:rows])
    x, S, U, b = (torch.from_numpy(t.value[k].astype("float32")).cuda().double() for k in ("x", "S", "U", "b"))
    want = (x @ S.reshape(d, R)).bfloat16().double() @ U.reshape(R, R) + b
    assert float((staged.y.double() - want).abs().max() / want.std()) < 5e-2   # two roundings to 8 bits at up to six deviations


@pytest.mark.parametrize("tile,R", [(1, 128), (2, 128), (4, 64)], ids=["128x128", "128x64", "64x64"])
def test_factor_gradient_on_either_side_of_a_round(sk, tuning, tile, R):  # noqa: F811
    """Z^T . dY with the column sums, four ragged ranges of tokens, 8192 columns (the last work-group of a round) and a tile more: the
    columns that both have bit for bit, ring and staged."""
    tuning(sk.SK_TUNE_WTILE, tile)
    tuning(sk.SK_TUNE_WSPLITS, 4)
    staged, ring = (DeviceLayer(W.generate(W.Workload("ring_round", 1100, 80, out, 1, R, "bf16", seed=6)), sk) for out in (8192 + 128, 8192))
    ring.x.copy_(staged.x)
    ring.S_cat.copy_(staged.S_cat)
    ring.dY.copy_(staged.dY[:, :8192])
    for dev, want in ((staged, False), (ring, True)):
        names = _kernels_of(sk, dev, ("bwd_weight",))
        assert ["float, true" in n for n in names[:2]] == [False, True] and (len(_rings(names[1:2])) == 1) == want, names
    assert torch.equal(ring.dU, staged.dU[:, :8192]) and torch.equal(ring.db, staged.db[:8192])
    Z = (staged.x.double() @ staged.S_cat.double()).bfloat16().double()
    want = Z.T @ staged.dY.double()
    # (where the library's fp32 sums of Z round the other way, at most one element in a hundred: 0.1 x 2^-8 = 4e-4)
    assert float((staged.dU.double() - want).norm() / want.norm()) < 1e-3
    assert float((staged.db.double() - staged.dY.double().sum(0)).norm() / staged.db.double().norm()) < 1e-5


@pytest.mark.parametrize("shape,ring", [
    # wide sketches: dY . U^T beside Z^T, ragged tokens, widths and k tails, up to the 512 work-groups of a round and past it
    ((1950, 2832, 1568, 1, 240), True), ((2086, 1072, 720, 1, 320), True), ((1507, 3120, 464, 2, 256), True), ((4097, 768, 768, 1, 256), False),
    # narrow ones: dY . U^T in ranges beside Z^T
    ((922, 384, 3552, 1, 48), True), ((2925, 1584, 2480, 2, 32), True), ((3585, 400, 2336, 2, 16), False),
], ids=lambda v: "T%d_%dx%d_l%dk%d" % v if isinstance(v, tuple) else str(v))
def test_two_products_on_rings(sk, shape, ring):  # noqa: F811
    T, d_in, d_out, l, k = shape
    w = W.Workload("ring_pair", T, d_in, d_out, l, k, "bf16", seed=T)
    names = _kernels_of(sk, DeviceLayer(W.generate(w), sk), ("bwd",))
    assert names[0] == ("dual_gemm_kernel<ring>" if ring else "dual_gemm_kernel"), names
    check_all(sk, w, 0, single_call=True)   # bound: the repository's bf16 bar (two roundings to 8 bits)


@pytest.mark.parametrize("tokens,d_in,d_out,R", [(4096, 768, 768, 256), (3584, 400, 2336, 32)], ids=["wide", "narrow"])
def test_two_products_on_either_side_of_a_round(sk, tokens, d_in, d_out, R):  # noqa: F811
    """One token more is one work-group too many for a round: dX of the tokens before it bit for bit, ring and staged."""
    big = DeviceLayer(W.generate(W.Workload("pair_round", tokens + 1, d_in, d_out, 1, R, "bf16", seed=R)), sk)
    small = DeviceLayer(W.generate(W.Workload("pair_round", tokens, d_in, d_out, 1, R, "bf16", seed=R)), sk)
    for n in ("x", "dY"):
        getattr(small, n).copy_(getattr(big, n)[:tokens])
    for n in ("S_cat", "U_cat"):
        getattr(small, n).copy_(getattr(big, n))
    assert _kernels_of(sk, small, ("bwd",))[0] == "dual_gemm_kernel<ring>" and _kernels_of(sk, big, ("bwd",))[0] == "dual_gemm_kernel"
    assert torch.equal(small.dX, big.dX[:tokens])
