"""Batched dense products of few rows (a short contraction) and many columns."""
import pytest

import oracle
from paper_2507_13204_amd import inputs
from _helpers import TOL_F64_F, TOL_F64_G, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# Contractions shorter than a k-step of 16 or 32, of one, and with a remainder;
# columns that end within a wave's 32, a tile's 256 and a tile; both sides of the
# rows and of the entries from which FP32 operands are split.
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,n", [(1, 20_001), (3, 8_192), (15, 30_017), (16, 30_000), (16, 70_031), (17, 61_700),
                                 (31, 33_833), (31, 20_256), (33, 40_000), (47, 22_500), (100, 20_003),
                                 (255, 4_113), (256, 4_095), (256, 4_096), (257, 8_192)])
def test_few_rows_and_many_columns(m, n, dtype):
    from paper_2507_13204_amd import BatchedDense
    b = inputs.batched_dense(m, n, seed=m)
    A, X, W = (to_dev(t, dtype) for t in (b.A, b.X, b.W))
    f_ref, G_ref = oracle.bdense_gradient_fast(*(t.double().cpu().numpy() for t in (A, X, W)))
    tf, tg = (TOL_F64_F, TOL_F64_G) if dtype == torch.float64 else (1e-7, 3e-7)
    obj = BatchedDense(A, W, ckpt="recompute")
    f, G = obj.gradient(X)
    assert srel(f.item(), f_ref) <= tf and rel(G.cpu().numpy(), G_ref) <= tg
    assert srel(obj.objective(X).item(), f_ref) <= tf
    Xo = torch.empty(m * n + 1, dtype=dtype, device="cuda")[1:].view(m, n)  # off the 16-byte grid
    Xo.copy_(X)
    G2 = G.clone()
    f2, _ = BatchedDense(A, W, accumulate=True).gradient(Xo, out=G2)
    assert torch.equal(f, f2) and rel(G2.cpu().numpy(), 2 * G_ref) <= tg
