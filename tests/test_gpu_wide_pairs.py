"""The backward pass of a wide sketch in shared launches, over the pairs of products it is made of: dY . U^T and x . S whole or in
ranges on either tile, dX on each of its tiles, one range of tokens and several, all sizes ragged -- against the fp64 oracle, dU and
db bit for bit those of the separate call, run to run the same."""
import pytest

from paper_2601_15473_amd import libsk
from paper_2601_15473_amd import workloads as W


def _pair(T, d_in, d_out, R):
    """-> (tile, ranges of dY . U^T, ranges of x . S, on the ring) of the first shared launch, from a host trace."""
    P = [i << 44 for i in range(1, 9)]
    args = (T, d_in, d_out, 1, R, libsk.SK_BF16)
    libsk.sk_trace_begin()
    try:
        libsk.check(libsk.sk_linear_bwd(*P[:7], *args, P[7], libsk.sk_linear_workspace_bytes(libsk.SK_OP_BWD, *args)))
        names = libsk.sk_trace_kernels()
    finally:
        accesses, _ = libsk.sk_trace_end()
    assert T % 8 != 0 and names[0][0].startswith("dual_gemm_kernel"), names
    ranges = {"g": 1, "z": 1}
    if "to_bf16" in names[1][0]:
        sums = [(b, w) for _, b, w, launch in accesses if launch == 1]
        for (slabs, _), (result, written) in zip(sums[::2], sums[1::2]):
            assert written
            ranges["g" if result == 2 * T * R else "z"] = slabs // (2 * result)   # (the rows of Z^T are padded)
    both = ranges["g"] + ranges["z"]
    tiles = [side for side in (64, 128) if -(-T // side) * -(-R // side) * both == names[0][1]]
    return (*tiles, ranges["g"], ranges["z"], names[0][0].endswith("<ring>"))


@pytest.mark.parametrize("shape,want", [
    # one range a walk on 64 x 64 tiles where they make a round, long walks of a few more than that in ranges on 128 x 128 ones: 330 walks of 94 chunks on 256 CUs
    # 104 us, 165 of 47 and their sums 86 (7024 tokens, 6000 outputs, R = 192, the whole call); 297 of 68 65.7 : 53.3 (1668, 4336, 704)
    ((4059, 144, 2000, 256), (64, 1, 1, True)), ((7023, 256, 6000, 192), (128, 2, 1, False)), ((1667, 144, 4336, 704), (128, 3, 1, False)),
    ((1383, 96, 7408, 992), (128, 2, 1, False)),
    # ... and 450 walks of 38 chunks ahead of 300 of 57 (136.7 : 127)
    ((6279, 240, 7232, 304), (128, 3, 1, False)),
    # short walks, and those of x . S in ranges, stay on 64 x 64 tiles past two work-groups a CU
    ((8645, 816, 176, 192), (64, 1, 1, False)), ((1587, 3936, 80, 160), (64, 1, 6, False)),
], ids=lambda v: "x".join(map(str, v)))
def test_which_pair_a_layer_takes(shape, want):
    assert _pair(*shape) == want


@pytest.mark.gpu
@pytest.mark.parametrize("shape,launches,pair", [
    # both whole: 64 x 64 tiles on the ring and past it, 128 x 128 tiles, one range of tokens, dX on 64 x 64 tiles
    ((735, 560, 592, 2, 216), 3, (64, 1, 1, True)), ((1482, 176, 208, 2, 400), 3, (64, 1, 1, False)), ((3642, 1360, 784, 1, 496), 3, (128, 1, 1, False)),
    ((556, 1136, 1232, 1, 176), 2, (64, 1, 1, True)), ((281, 80, 80, 1, 784), 2, (64, 1, 1, True)),
    # dY . U^T in ranges
    ((339, 1200, 3824, 1, 464), 3, (64, 4, 1, True)), ((597, 640, 3696, 1, 800), 3, (128, 6, 1, False)),
    # x . S in ranges
    ((597, 2288, 112, 1, 272), 4, (64, 1, 5, True)), ((1212, 3920, 608, 1, 272), 4, (64, 1, 5, False)), ((578, 3584, 96, 1, 800), 4, (128, 1, 7, False)),
    ((3155, 2576, 640, 1, 368), 4, (128, 1, 3, False)),
    # both
    ((861, 2240, 3568, 1, 144), 3, (64, 5, 4, True)), ((349, 2272, 3920, 1, 624), 3, (64, 4, 5, False)), ((2803, 1792, 3888, 2, 176), 4, (128, 3, 3, False)),
], ids=lambda v: "T%d_%dx%d_l%dk%d" % v if isinstance(v, tuple) and len(v) == 5 else "")
def test_against_the_oracle_and_the_separate_call(shape, launches, pair):
    import torch
    from test_gpu_parity import DeviceLayer, _kernels_of, check_all
    sk = libsk
    T, d_in, d_out, l, k = shape
    w = W.Workload("wide_pairs", T, d_in, d_out, l, k, "bf16", seed=T)
    check_all(sk, w, 0, single_call=True)   # bound: the repository's bf16 bar (two roundings to 8 bits)
    t = W.generate(w)
    names = _kernels_of(sk, DeviceLayer(t, sk), ("bwd",))
    assert len(names) == launches and sum(n.startswith("dual_gemm_kernel") for n in names) == 2, names
    assert _pair(T, d_in, d_out, l * k) == pair
    one, again, sep = DeviceLayer(t, sk), DeviceLayer(t, sk), DeviceLayer(t, sk)
    again.ws.fill_(255)
    sk.check(one.bwd())
    sk.check(again.bwd())
    sk.check(sep.bwd_weight())
    torch.cuda.synchronize()
    bits = lambda x: x.view(torch.int16 if x.element_size() == 2 else torch.int32)
    for n in ("dU", "db"):
        assert torch.equal(bits(getattr(one, n)), bits(getattr(sep, n))), n
    for n in ("dX", "dU", "db"):
        assert torch.equal(bits(getattr(one, n)), bits(getattr(again, n))), n
