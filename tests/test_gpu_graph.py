"""The library's calls only launch kernels on the caller's stream (no allocation, no
synchronisation, no memset), so they can be recorded into a HIP graph.  Each replay is
checked against the eager result, with eager work and synchronisations between replays."""
import numpy as np
import pytest
import torch

from paper_2601_15473_amd import workloads as W
from paper_2601_15473_amd.device import DeviceLayer
from test_gpu_parity import _kernels_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sk():
    from paper_2601_15473_amd import libsk
    yield libsk
    libsk.sk_set_plan(0)


CASES = [
    W.scaled(W.BERT_BASE_FFN_UP, tokens=1000),      # fused forward, split + expand input gradient
    W.scaled(W.BERT_LARGE_FFN_UP, tokens=600),      # two GEMMs per call
    W.scaled(W.BY_NAME["grid8192_l1_k16"], tokens=300),   # split first contractions, sum-to-bf16 kernel
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: f"{w.name}_T{w.tokens}")
def test_calls_replay_from_a_graph(sk, w):
    sk.sk_set_plan(0)
    t = W.generate(w)
    eager = DeviceLayer(t, sk)
    eager.run_all()
    ref = {n: getattr(eager, n).clone() for n in ("y", "dX", "dU", "db")}

    dev = DeviceLayer(t, sk, poison=False)
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        # one eager pass on the capture stream first (nothing in the library is lazily set up,
        # but the first launch of a kernel loads its code object)
        for st in (dev.fwd(stream), dev.bwd_input(stream), dev.bwd_weight(stream)):
            sk.check(st)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        cap = torch.cuda.current_stream()
        for st in (dev.fwd(cap), dev.bwd_input(cap), dev.bwd_weight(cap)):
            sk.check(st)
    for rep in range(3):
        for n in ("y", "dX", "dU", "db"):
            getattr(dev, n).fill_(float("nan"))     # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n in ("y", "dX", "dU", "db"):
            got, want = getattr(dev, n), ref[n]
            assert torch.equal(got.view(torch.int16 if got.dtype == torch.bfloat16 else torch.int32),
                               want.view(torch.int16 if want.dtype == torch.bfloat16 else torch.int32)), (rep, n)


STEP_CASES = [   # the layer, and the kernels of its backward pass
    (W.scaled(W.BERT_BASE_FFN_UP, tokens=1000), ["dual_gemm_kernel", "factor_beside_expand_kernel<128, 128, true>", "reduce_splits_kernel"]),
    # sums carried by the expansion
    (W.Workload("expansion_behind", 4096, 1664, 3072, 1, 80, "bf16"), ["dual_gemm_kernel", "gemm_bf16_kernel<128, 64, true, false, float, true, true>", "chain_small_kernel<64, 128, true, false, true>"]),
    (W.scaled(W.BERT_LARGE_FFN_UP, tokens=5000), ["dual_gemm_kernel", "dual_gemm_kernel", "reduce_splits_kernel"]),
    # both products of the first launch in ranges
    (W.Workload("wide_in_ranges", 861, 2240, 3568, 1, 144, "bf16"), ["dual_gemm_kernel<ring>", "reduce_two_to_bf16_kernel", "dual_gemm_kernel"]),
    (W.scaled(W.BERT_BASE_PROJ[0], tokens=700), ["dual_gemm_kernel<ring>", "factor_beside_expand_kernel<64, 64, true>", "reduce_splits_kernel"]),
    # one pass over x and dY and the sum of the tiles' slabs, tiles of 32 tokens and of 64
    (W.Workload("one_pass", 700, 768, 208, 2, 16, "bf16"), ["bwd_narrow_kernel<1>", "reduce_tiles_kernel"]),
    (W.scaled(W.BERT_BASE_PROJ[0], tokens=9000), ["bwd_narrow_kernel<2>", "reduce_tiles_kernel"]),
]


@pytest.mark.parametrize("w,kernels", STEP_CASES, ids=lambda v: f"{v.name}_T{v.tokens}" if isinstance(v, W.Workload) else "")
def test_timed_step_replays_from_a_graph(sk, w, kernels):
    """The benchmark's step (sk_linear_fwd + sk_linear_bwd) recorded once and replayed."""
    sk.sk_set_plan(0)
    t = W.generate(w)
    eager = DeviceLayer(t, sk)
    sk.check(eager.fwd())
    assert _kernels_of(sk, eager, ("bwd",)) == kernels
    ref = {n: getattr(eager, n).clone() for n in ("y", "dX", "dU", "db")}

    dev = DeviceLayer(t, sk, poison=False)
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        for st in (dev.fwd(stream), dev.bwd(stream)):
            sk.check(st)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        cap = torch.cuda.current_stream()
        for st in (dev.fwd(cap), dev.bwd(cap)):
            sk.check(st)
    for rep in range(3):
        for n in ("y", "dX", "dU", "db"):
            getattr(dev, n).fill_(float("nan"))     # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n in ("y", "dX", "dU", "db"):
            got, want = getattr(dev, n), ref[n]
            assert torch.equal(got.view(torch.int16 if got.dtype == torch.bfloat16 else torch.int32),
                               want.view(torch.int16 if want.dtype == torch.bfloat16 else torch.int32)), (rep, n)
