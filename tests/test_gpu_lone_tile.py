"""Products of 128 x 64 or 64 x 128 tiles in more than a round that take 128 x 128 ones in one: first contractions and expansions, ragged rows, columns
and contractions, on either side of a round -- against the fp64 oracle, and bit for bit the smaller tiles'."""
import pytest

from paper_2601_15473_amd import libsk
from paper_2601_15473_amd import workloads as W
from test_gpu_expansion_tile import _kernels

RING = "gemm_bf16_kernel<128, 128, true, false, bf16, false, true>"


@pytest.mark.parametrize("shape,which,taken", [
    # (tokens, in, out, R): 128 work-groups of 128 x 128 and 256, a tile less and a row more; a contraction of 128; 64 x 64 tiles
    ((4096, 320, 64, 512), 0, True), ((3968, 320, 64, 512), 0, False), ((8192, 320, 64, 512), 0, True), ((8193, 320, 64, 512), 0, False),
    ((4096, 128, 64, 512), 0, False), ((2048, 64, 1024, 160), 1, True), ((1920, 64, 1024, 160), 1, False),
    ((2048, 64, 2048, 160), 1, True), ((2049, 64, 2048, 160), 1, False), ((1000, 64, 1024, 160), 1, False),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_which_products_take_it(shape, which, taken):
    names = _kernels("fwd", *shape)
    assert len(names) == 2 and (names[which] == RING) == taken, names


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(3146, 272, 1168, 2, 384), (2425, 144, 1296, 1, 848), (4119, 336, 368, 2, 400), (863, 1040, 3664, 1, 544)],
                         ids=lambda v: "T%d_%dx%d_l%dk%d" % v)
def test_against_the_oracle_and_the_small_tiles(shape):
    import torch
    from test_gpu_parity import DeviceLayer, _kernels_of, check_all
    T, d_in, d_out, l, k = shape
    w = W.Workload("lone_tile", T, d_in, d_out, l, k, "bf16", seed=T)
    check_all(libsk, w, 0)                    # bound: the repository's bf16 bar (two roundings to 8 bits)
    t = W.generate(w)
    big, small = DeviceLayer(t, libsk), None
    names = _kernels_of(libsk, big, ("fwd", "bwd_input", "bwd_weight"))
    assert any(n.startswith("gemm_bf16_kernel<128, 128,") and n.endswith("true>") for n in names), names
    for call in ("fwd", "bwd_input"):
        libsk.check(getattr(big, call)())
    libsk.sk_set_tuning(libsk.SK_TUNE_TILE, 2)
    try:
        small = DeviceLayer(t, libsk)   # (its workspace for that plan)
        for call in ("fwd", "bwd_input"):
            libsk.check(getattr(small, call)())
    finally:
        libsk.sk_set_tuning(libsk.SK_TUNE_TILE, -1)
    torch.cuda.synchronize()
    for n in ("y", "dX")[:1 if d_out > 2048 else 2]:   # (over 3664 dY . U^T comes in ranges by itself, other sums)
        assert torch.equal(getattr(big, n).view(torch.int16), getattr(small, n).view(torch.int16)), n
