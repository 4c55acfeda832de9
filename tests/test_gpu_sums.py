"""Sums of split products, over every remainder of the batches that a piece's slabs are fetched in: inputs of whole numbers small
enough that every product and sum is exact, so a slab left out, taken twice or taken from elsewhere shows."""
import pytest
import torch

from paper_2601_15473_amd import libsk
from test_gpu_parity import sk, tuning  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d_out,R", [(1024, 64), (3072, 128)], ids=["one piece a thread", "four pieces a thread"])
@pytest.mark.parametrize("splits", [1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 14, 15, 16, 23, 31, 32])
def test_every_slab_once(sk, tuning, splits, d_out, R, dtype):  # noqa: F811
    tuning(sk.SK_TUNE_WSPLITS, splits)
    T, d_in, td = 8192, 768, torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(splits)
    whole = lambda *s: torch.randint(-1, 2, s, generator=g, device="cuda").to(td)
    x, dY, S, U = whole(T, d_in), whole(T, d_out), whole(d_in, R), whole(R, d_out)
    S[64:] = 0     # |x . S| <= 64: exact in bf16
    want = (x.double() @ S.double()).T @ dY.double()
    shape = (T, d_in, d_out, 1, R, libsk.DTYPES[dtype])
    for both in (False, True):
        need = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD if both else sk.SK_OP_BWD_WEIGHT, *shape)
        ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
        dX, dU, db = torch.empty(T, d_in, dtype=td, device="cuda"), torch.empty(R, d_out, device="cuda"), torch.empty(d_out, device="cuda")
        if both:
            sk.check(sk.sk_linear_bwd(x, dY, S, U, dX, dU, db, *shape, ws, need))
        else:
            sk.check(sk.sk_linear_bwd_weight(x, S, dY, dU, db, *shape, ws, need))
        torch.cuda.synchronize()
        assert torch.equal(dU.double(), want) and torch.equal(db.double(), dY.double().sum(0)), both


@pytest.mark.parametrize("T", [1, 5, 63, 65, 700, 4001])
def test_column_sums_of_their_own(sk, tuning, T):  # noqa: F811
    """The column sums beside the 256 x 256 tile: runs of less than a batch of rows, of one and of several with a rest."""
    tuning(sk.SK_TUNE_WTILE, 0)
    d_in, d_out, R = 64, 1040, 256
    g = torch.Generator(device="cuda").manual_seed(T)
    dY = torch.randint(-8, 9, (T, d_out), generator=g, device="cuda").bfloat16()
    x, S = torch.zeros(T, d_in, device="cuda").bfloat16(), torch.zeros(d_in, R, device="cuda").bfloat16()
    shape = (T, d_in, d_out, 1, R, libsk.DTYPES["bf16"])
    need = sk.sk_linear_workspace_bytes(sk.SK_OP_BWD_WEIGHT, *shape)
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    dU, db = torch.empty(R, d_out, device="cuda"), torch.empty(d_out, device="cuda")
    sk.check(sk.sk_linear_bwd_weight(x, S, dY, dU, db, *shape, ws, need))
    torch.cuda.synchronize()
    assert torch.equal(db.double(), dY.double().sum(0)) and not dU.any()
