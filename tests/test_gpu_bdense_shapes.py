"""Batched dense products at the edges of the tile shapes, and the values that
the split of FP32 operands has to carry."""
import numpy as np
import pytest

import oracle
from paper_2507_13204_amd import inputs
from _helpers import TOL_F64_F, TOL_F64_G, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# FP32 storage: V and G are rounded to FP32 (2^-24 each), the products behind
# them carry about 2^-24 of a term.
F32_F, F32_G = 1e-7, 3e-7

# Below, on and above the blocks of 16 and 32 and the tiles of 64 and 128;
# contractions shorter than a k-step, whole steps and every kind of remainder;
# one row or column; few tiles, one round of them, several.
SIZES = [(1, 1), (1, 40), (15, 17), (16, 16), (17, 15), (31, 33), (32, 15), (33, 32), (40, 1),
         (63, 65), (64, 64), (65, 31), (100, 300), (127, 129), (128, 512), (129, 31), (255, 70),
         (300, 200), (513, 250), (640, 1030), (1100, 530), (2100, 40)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,n", SIZES)
def test_bdense_tile_edges(m, n, dtype):
    from paper_2507_13204_amd import BatchedDense
    b = inputs.batched_dense(m, n, seed=400 + m)
    A, X, W = (to_dev(t, dtype) for t in (b.A, b.X, b.W))
    h = [t.double().cpu().numpy() for t in (A, X, W)]
    f_ref, G_ref = oracle.bdense_gradient_fast(*h)
    tf, tg = (TOL_F64_F, TOL_F64_G) if dtype == torch.float64 else (F32_F, F32_G)
    obj = BatchedDense(A, W, ckpt="recompute")
    f, G = obj.gradient(X)
    assert srel(f.item(), f_ref) <= tf and rel(G.cpu().numpy(), G_ref) <= tg
    assert srel(obj.objective(X).item(), f_ref) <= tf
    # an operand off the 16-byte grid, the result added to what is there, the
    # same bits again
    Xo = torch.empty(m * n + 1, dtype=dtype, device="cuda")[1:].view(m, n)
    Xo.copy_(X)
    add = BatchedDense(A, W, accumulate=True)
    G2 = G.clone()
    f2, _ = add.gradient(Xo, out=G2)
    assert torch.equal(f, f2) and rel(G2.cpu().numpy(), 2 * G_ref) <= tg
    f3, G3 = obj.gradient(X)
    assert torch.equal(f, f3) and torch.equal(G, G3)


@pytest.mark.parametrize("m,n", [(48, 20), (130, 64), (600, 500)])
@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** -30, 2.0 ** 30])
def test_bdense_f32_small_and_large_operands(m, n, scale):
    """Operands whose low parts are below the normal range of bfloat16 (A at
    2^-126 and less against X at 2^60 and more), and large ones."""
    from paper_2507_13204_amd import BatchedDense
    b = inputs.batched_dense(m, n, seed=9)
    a_scale = scale * scale if scale < 1 else scale  # 2^-120, 2^-60, 2^30
    A = (b.A * a_scale).astype(np.float32)
    X = (b.X / a_scale).astype(np.float32)
    W = b.W.astype(np.float32)
    f_ref, _ = oracle.bdense_gradient_fast(*(t.astype(np.float64) for t in (A, X, W)))
    f, _ = BatchedDense(to_dev(A), to_dev(W)).gradient(to_dev(X))
    # subnormal entries of A carry their own rounding, which the oracle sees too
    assert srel(f.item(), f_ref) <= 1e-6


@pytest.mark.parametrize("bad", [float("inf"), -float("inf"), float("nan"), 3.4e38])
def test_bdense_f32_not_finite(bad):
    """A value past the largest bfloat16, an infinity or a NaN in one entry
    reaches the rows and columns it reaches in plain arithmetic."""
    from paper_2507_13204_amd import BatchedDense
    b = inputs.batched_dense(200, 70, seed=12)
    A, X, W = (t.astype(np.float32) for t in (b.A, b.X, b.W))
    A[5, :] = 0.0
    A[5, 7] = 1.0
    X[7, 3] = bad
    obj = BatchedDense(to_dev(A), to_dev(W), ckpt="store")
    tape = obj.new_tape("cuda")
    f = obj.objective_tape(to_dev(X), tape)
    V = tape.view(torch.float32)[:200 * 70].view(200, 70).cpu().numpy()
    Y = A.astype(np.float64) @ X.astype(np.float64)
    with np.errstate(all="ignore"):
        want = (W * (Y + Y / (1 + Y * Y))).astype(np.float32)
        assert np.isfinite(f.item()) == np.isfinite((W * (0.5 * Y * Y + 0.5 * np.log1p(Y * Y))).sum())
    cols = np.arange(70) != 3
    assert np.isfinite(V[:, cols]).all() and rel(V[:, cols], want[:, cols]) <= F32_G
    assert np.array_equal(np.isnan(V[:, 3]), np.isnan(want[:, 3]))
    ok = np.isfinite(want[:, 3]) & (np.abs(want[:, 3]) < 1e37)
    assert rel(V[ok, 3], want[ok, 3]) <= F32_G
