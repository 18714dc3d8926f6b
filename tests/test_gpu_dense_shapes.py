"""Row reductions at the edges of the row-length classes: lanes to a row, waves
to a team, slices to a thread, one pass or two, whole and partial bands."""
import numpy as np
import pytest

import oracle
from paper_2507_13204_amd import inputs
from _helpers import TOL_F32, TOL_F64_F, TOL_F64_G, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# Row lengths on both sides of every class boundary, with and without whole
# 16-byte slices.
COLS = [1, 3, 8, 9, 16, 17, 32, 33, 34, 64, 65, 66, 128, 130, 192, 256, 257, 320, 384, 511, 512,
        513, 514, 1024, 1536, 1537, 2047, 2048, 2049, 2050, 3072, 4100, 5121, 6146, 8193, 10242,
        12288, 12289, 12292, 16383, 16384, 16385]
# One row, fewer rows than a team takes at once, a ragged number of them.
ROWS = [1, 5, 77]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("cols", COLS)
def test_dense_row_classes(cols, dtype):
    from paper_2507_13204_amd import DenseObjective
    for rows in ROWS:
        d = inputs.dense(cols, seed=300 + rows, rows=rows)
        A, x, w = to_dev(d.A, dtype), to_dev(d.x, dtype), to_dev(d.w, dtype)
        h = [t.double().cpu().numpy() for t in (A, x, w)]
        f_ref, g_ref = oracle.dense_gradient(*h)
        tf, tg = (TOL_F64_F, TOL_F64_G) if dtype == torch.float64 else (TOL_F32, TOL_F32)
        obj = DenseObjective(A, w)
        f, g = obj.gradient(x)
        assert srel(f.item(), f_ref) <= tf and rel(g.cpu().numpy(), g_ref) <= tg, (rows, cols)
        assert srel(obj.objective(x).item(), f_ref) <= tf, (rows, cols)
        fbar = torch.tensor([-2.5], dtype=torch.float64, device="cuda")
        assert rel(obj.adjoint(x, fbar).cpu().numpy(), -2.5 * g_ref) <= tg, (rows, cols)
        # x off the 16-byte grid, and the gradient added to what is there
        xo = torch.empty(cols + 1, dtype=dtype, device="cuda")[1:]
        xo.copy_(x)
        add = DenseObjective(A, w, accumulate=True)
        g2 = g.clone()
        f2, _ = add.gradient(xo, out=g2)
        assert srel(f2.item(), f_ref) <= tf and rel(g2.cpu().numpy(), 2 * g_ref) <= tg, (rows, cols)


@pytest.mark.parametrize("rows,cols", [(5000, 20), (3001, 301), (9000, 130), (4000, 1000), (1500, 2500)])
def test_dense_many_rows_repeatable(rows, cols):
    """Bands of many steps: parity, and the same bits on every call."""
    from paper_2507_13204_amd import DenseObjective
    d = inputs.dense(cols, seed=17, rows=rows)
    obj = DenseObjective(to_dev(d.A), to_dev(d.w))
    x = to_dev(d.x)
    f, g = obj.gradient(x)
    f_ref, g_ref = oracle.dense_gradient(d.A, d.x, d.w)
    assert srel(f.item(), f_ref) <= TOL_F64_F and rel(g.cpu().numpy(), g_ref) <= TOL_F64_G
    for _ in range(3):
        f2, g2 = obj.gradient(x)
        assert torch.equal(f, f2) and torch.equal(g, g2)


@pytest.mark.parametrize("rows,cols", [(77, 20), (77, 301), (78, 1000), (77, 5001), (77, 16500)])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_dense_not_finite(rows, cols, bad):
    """A value that is not finite reaches the entries it reaches in plain
    arithmetic and no others (the lanes past a row and the rows past a band
    add nothing)."""
    from paper_2507_13204_amd import DenseObjective
    d = inputs.dense(cols, seed=5, rows=rows)
    A = d.A.copy()
    A[rows - 1, :] = 0.0
    A[rows - 1, cols - 1] = bad
    x = np.abs(d.x) + 0.5
    obj = DenseObjective(to_dev(A), to_dev(d.w))
    f, g = obj.gradient(to_dev(x))
    # the last row's sum is not finite: f is, and v A is NaN or not finite in
    # every column (0 * v in all but the last)
    assert not np.isfinite(f.item()) and not torch.isfinite(g).any()
    x[cols - 1] = 0.0
    A[rows - 1, cols - 1] = 1.0
    x[0] = bad
    A[:, 0] = 0.0
    A[0, 0] = 2.0
    A[1:, 0] = 1e-3
    f, g = DenseObjective(to_dev(A), to_dev(d.w)).gradient(to_dev(x))
    r = A @ x
    want = (d.w * (r + r / (1 + r * r))) @ A
    assert np.array_equal(np.isnan(g.cpu().numpy()), np.isnan(want))
    assert np.isnan(f.item()) == np.isnan((d.w * (0.5 * r * r + 0.5 * np.log1p(r * r))).sum())
