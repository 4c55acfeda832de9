"""The fused chain on rings of loads: first contractions of fewer chunks than its ring has slots and of one more than
a turn, ending inside a chunk; sketch widths below the kernel's; runs shorter and longer than the ring of output
tiles, last tile ragged; on either side of the round past which long runs of a narrow sketch take the other kernel;
infinities beside widths below the kernel's -- against the fp64 oracle and the two-GEMM plan."""
import pytest
import torch

from paper_2601_15473_amd import workloads as W
from test_gpu_parity import DeviceLayer, _kernels_of, check_all, sk, tuning  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slices", [1, 4], ids=["long", "short"])
@pytest.mark.parametrize("R", [16, 48, 64, 80, 128])
@pytest.mark.parametrize("d_in,d_out", [(16, 1040), (208, 1168), (272, 48), (336, 912)])
def test_ring_edges(sk, tuning, d_in, d_out, R, slices):  # noqa: F811
    # bound: the repository's bf16 bar (the intermediate and the result rounded to 8 bits once each)
    tuning(sk.SK_TUNE_BM, 64)
    tuning(sk.SK_TUNE_SLICES, slices)
    check_all(sk, W.Workload("chain_ring", 131, d_in, d_out, 1, R, "bf16", seed=R + d_in), 1)


@pytest.mark.parametrize("tokens,ring", [(64 * 256, True), (64 * 256 + 1, False)])
def test_long_runs_of_a_narrow_sketch(sk, tuning, tokens, ring):  # noqa: F811
    tuning(sk.SK_TUNE_BM, 64)
    tuning(sk.SK_TUNE_SLICES, 1)
    w = W.Workload("chain_round", tokens, 80, 592, 1, 32, "bf16", seed=3)
    check_all(sk, w, 1)
    sk.sk_set_plan(1)
    try:
        name, = _kernels_of(sk, DeviceLayer(W.generate(w), sk), ("fwd",))
    finally:
        sk.sk_set_plan(0)
    assert name.startswith("chain_small_kernel<64, 64,") and name.endswith("true>") == ring, name


@pytest.mark.parametrize("tokens,R,ring", [(64 * 256, 32, True), (64 * 256 + 1, 32, False), (64 * 256 + 1, 80, True)])
def test_short_runs_past_a_round(sk, tuning, tokens, R, ring):  # noqa: F811
    """Three output tiles, the last one ragged: a narrow sketch leaves the rings with the first work-group past a round."""
    # bound of check_all: the repository's bf16 bar (the intermediate and the result rounded to 8 bits once each)
    w = W.Workload("chain_short_round", tokens, 208, 272, 1, R, "bf16", seed=4)
    check_all(sk, w, 1)
    sk.sk_set_plan(1)
    try:
        for call in ("fwd", "bwd_input"):
            name, = _kernels_of(sk, DeviceLayer(W.generate(w), sk), (call,))
            assert name.startswith("chain_short_kernel<64, ") and (name.count(",") == 5) == ring, name
    finally:
        sk.sk_set_plan(0)


@pytest.mark.parametrize("R", [16, 48, 80])
def test_infinities_stay_in_their_rows(sk, tuning, R):  # noqa: F811
    """As in the plan of two GEMMs: sketch columns the kernel pads with meet no infinity of x."""
    t = W.generate(W.Workload("chain_inf", 100, 208, 336, 1, R, "bf16", seed=R))
    got = []
    for plan in (1, 2):
        dev = DeviceLayer(t, sk)
        dev.x[7, 3] = float("inf")
        dev.x[40] = 3e38
        sk.sk_set_plan(plan)
        try:
            sk.check(dev.fwd())
        finally:
            sk.sk_set_plan(0)
        torch.cuda.synchronize()
        got.append(dev.y.float())
    a, b = got
    finite = torch.isfinite(b)
    assert torch.equal(finite, torch.isfinite(a)) and torch.equal(torch.isnan(a), torch.isnan(b))
    assert finite[:7].all() and finite[8:40].all() and not finite[7].any()
    assert torch.equal(a[finite], b[finite])   # the same sums in the same order
