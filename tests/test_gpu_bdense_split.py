"""FP32 batched products of 2^20 entries and more (operands split in bfloat16
parts): tiles whose waves share the split and others, at every kind of edge."""
import numpy as np
import pytest

import oracle
from paper_2507_13204_amd import inputs
from _helpers import rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# V and G are rounded to FP32 (2^-24 each), the products behind them carry
# about 2^-24 of a term.
F32_F, F32_G = 1e-7, 3e-7


# (rows and contraction, columns): steps of 32 even and odd in number, with no,
# one and 31 terms left; columns that end within a wave's block, a wave's tile
# and a tile; tiles of 128 x 128 (4065), 64 x 128, 48 x 128 (3000, 2999) and 32 x 32 (2048 x 520).
@pytest.mark.parametrize("m,n", [(1024, 1024), (1056, 1000), (1087, 970), (1181, 900), (1345, 801),
                                 (2048, 520), (3000, 500), (2999, 497), (4065, 1000)])
def test_bdense_split_edges(m, n):
    from paper_2507_13204_amd import BatchedDense
    b = inputs.batched_dense(m, n, seed=m)
    A, X, W = (t.astype(np.float32) for t in (b.A, b.X, b.W))
    f_ref, G_ref = oracle.bdense_gradient_fast(*(t.astype(np.float64) for t in (A, X, W)))
    obj = BatchedDense(to_dev(A), to_dev(W), ckpt="recompute")
    f, G = obj.gradient(to_dev(X))
    assert srel(f.item(), f_ref) <= F32_F and rel(G.cpu().numpy(), G_ref) <= F32_G
    f2, G2 = obj.gradient(to_dev(X))
    assert torch.equal(f, f2) and torch.equal(G, G2)
    Xo = torch.empty(m * n + 1, dtype=torch.float32, device="cuda")[1:].view(m, n)  # off the 16-byte grid
    Xo.copy_(to_dev(X))
    f3, G3 = obj.gradient(Xo)
    assert torch.equal(f, f3) and torch.equal(G, G3)


@pytest.mark.parametrize("m,n", [(1100, 1000), (2048, 520)])
@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** 30])
def test_bdense_split_small_and_large_operands(m, n, scale):
    """A at 2^-120 (its low parts below bfloat16's range) against X at 2^120,
    and large ones."""
    from paper_2507_13204_amd import BatchedDense
    b = inputs.batched_dense(m, n, seed=9)
    a_scale = scale * scale if scale < 1 else scale
    A, X = (b.A * a_scale).astype(np.float32), (b.X / a_scale).astype(np.float32)
    W = b.W.astype(np.float32)
    f_ref, _ = oracle.bdense_gradient_fast(*(t.astype(np.float64) for t in (A, X, W)))
    f, _ = BatchedDense(to_dev(A), to_dev(W)).gradient(to_dev(X))
    # subnormal entries of A carry their own rounding, which the oracle sees too
    assert srel(f.item(), f_ref) <= 1e-6


@pytest.mark.parametrize("m,n", [(1100, 1000), (2048, 520)])
@pytest.mark.parametrize("bad", [float("inf"), float("nan"), 3.4e38])
def test_bdense_split_not_finite(m, n, bad):
    """A value past the largest bfloat16, an infinity or a NaN in one entry
    reaches the rows and columns it reaches in plain arithmetic."""
    from paper_2507_13204_amd import BatchedDense
    b = inputs.batched_dense(m, n, seed=12)
    A, X, W = (t.astype(np.float32) for t in (b.A, b.X, b.W))
    A[5, :] = 0.0
    A[5, 7] = 1.0
    X[7, 3] = bad
    obj = BatchedDense(to_dev(A), to_dev(W), ckpt="store")
    tape = obj.new_tape("cuda")
    obj.objective_tape(to_dev(X), tape)
    V = tape.view(torch.float32)[:m * n].view(m, n).cpu().numpy()
    with np.errstate(all="ignore"):
        Y = A.astype(np.float64) @ X.astype(np.float64)
        want = (W * (Y + Y / (1 + Y * Y))).astype(np.float32)
    cols = np.arange(n) != 3
    assert np.isfinite(V[:, cols]).all() and rel(V[:, cols], want[:, cols]) <= F32_G
    assert np.array_equal(np.isnan(V[:, 3]), np.isnan(want[:, 3]))
    ok = np.isfinite(want[:, 3]) & (np.abs(want[:, 3]) < 1e37)
    assert rel(V[ok, 3], want[ok, 3]) <= F32_G
