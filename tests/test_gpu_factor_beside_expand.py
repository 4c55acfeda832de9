"""The factor gradient of a narrow sketch beside the expansion of dX, in one launch: ragged tokens, widths and sketches,
runs of one to three output tiles, one range of tokens and several, x . S in ranges, on either side of two work-groups a CU --
against the fp64 oracle, dU and db bit for bit those of the separate call, run to run the same."""
import pytest

from paper_2601_15473_amd import libsk
from paper_2601_15473_amd import workloads as W

KERNEL = "factor_beside_expand_kernel"


@pytest.mark.gpu
@pytest.mark.parametrize("runs,shape,launches", [(runs, *c) for runs, cases in (("short", [
    ((515, 400, 1040, 1, 16), 2), ((130, 64, 2064, 1, 48), 2), ((513, 80, 528, 1, 112), 3), ((1030, 272, 2320, 2, 32), 3), ((700, 1040, 1296, 1, 80), 3),
    ((2100, 784, 1040, 1, 128), 3), ((1111, 400, 2064, 1, 64), 3), ((4033, 384, 784, 1, 64), 3), ((1500, 2576, 1296, 1, 96), 4), ((900, 3600, 1040, 1, 32), 4), ((418, 3616, 272, 1, 80), 3),
    # instead of one pass over x and dY
    ((255, 304, 752, 1, 16), 2), ((2411, 768, 992, 1, 16), 3), ((4095, 848, 880, 2, 16), 3),
    # x . S in ranges for a few tokens
    ((9, 4000, 480, 1, 96), 3), ((143, 6000, 1808, 1, 64), 3), ((300, 4112, 1040, 1, 16), 3),
    # an expansion of fewer work-groups, to leave room
    ((1198, 3248, 752, 1, 64), 4),
]), ("long", [   # x . S whole and in ranges
    ((8200, 784, 528, 1, 48), 3), ((9295, 976, 1104, 1, 16), 3), ((2100, 4112, 2064, 1, 16), 4),
])) for c in cases], ids=lambda v: "T%d_%dx%d_l%dk%d" % v if isinstance(v, tuple) else v if isinstance(v, str) else "")
def test_against_the_oracle_and_the_separate_call(runs, shape, launches):
    import torch
    from test_gpu_parity import DeviceLayer, _kernels_of, check_all
    T, d_in, d_out, l, k = shape
    w = W.Workload("beside", T, d_in, d_out, l, k, "bf16", seed=T)
    check_all(libsk, w, 0, single_call=True)   # bound: the repository's bf16 bar (two roundings to 8 bits)
    t = W.generate(w)
    names = _kernels_of(libsk, DeviceLayer(t, libsk), ("bwd",))
    assert len(names) == launches and any(n.startswith(KERNEL) for n in names[-2:]), names
    assert [n.endswith("true>") for n in names if n.startswith(KERNEL)] == [runs == "short"], names   # (results straight from registers, or through LDS)
    one, again, sep = DeviceLayer(t, libsk), DeviceLayer(t, libsk), DeviceLayer(t, libsk)
    again.ws.fill_(255)
    libsk.check(one.bwd())
    libsk.check(again.bwd())
    libsk.check(sep.bwd_weight())
    torch.cuda.synchronize()
    bits = lambda x: x.view(torch.int16 if x.element_size() == 2 else torch.int32)
    for n in ("dU", "db"):
        assert torch.equal(bits(getattr(one, n)), bits(getattr(sep, n))), n
    for n in ("dX", "dU", "db"):
        assert torch.equal(bits(getattr(one, n)), bits(getattr(again, n))), n


def _names(T, d_in, d_out, R):
    P = [i << 44 for i in range(1, 9)]
    args = (T, d_in, d_out, 1, R, libsk.SK_BF16)
    libsk.sk_trace_begin()
    try:
        libsk.check(libsk.sk_linear_bwd(*P[:7], *args, P[7], libsk.sk_linear_workspace_bytes(libsk.SK_OP_BWD, *args)))
        return libsk.sk_trace_kernels()
    finally:
        libsk.sk_trace_end()


@pytest.mark.parametrize("shape,beside", [
    # up to two work-groups a CU
    ((16000, 128, 1024, 64), True), ((16384, 128, 1024, 64), True), ((16385, 128, 1024, 64), False),
    # runs of up to three output tiles of 128 columns, any up to R = 64
    ((2048, 1536, 3072, 80), True), ((4096, 1664, 3072, 80), False), ((4096, 1664, 3072, 64), True),
    # an expansion of one work-group a CU instead of two: dX up to twice dY, or 2048 tokens
    ((5505, 3600, 1808, 48), True), ((5505, 3600, 272, 48), False), ((2048, 3600, 272, 48), True),
    # one range of tokens, also where x . S comes in ranges
    ((300, 320, 1808, 32), True), ((320, 3616, 272, 80), True), ((9, 4000, 480, 96), True), ((34, 3696, 1248, 112), True),
    # instead of one pass over x and dY up to 4095 tokens, where there is a launch to share
    ((4095, 768, 768, 32), True), ((4096, 768, 768, 32), False), ((4095, 768, 768, 16), True), ((4096, 768, 768, 16), False), ((4095, 768, 368, 16), True),
    ((4096, 304, 784, 32), False),
    ((2000, 768, 240, 32), False),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_which_layers_take_it(shape, beside):
    names = _names(*shape)
    assert any(n.startswith(KERNEL) for n, _ in names) == beside, names
    if beside:
        assert all(g <= 512 for n, g in names if n.startswith(KERNEL)), names
