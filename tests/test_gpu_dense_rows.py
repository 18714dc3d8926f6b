"""The dense row pass on both sides of its rules: rows at a time, threads, and
x on and off the 16-byte grid."""
import pytest

import oracle
from paper_2507_13204_amd import inputs
from _helpers import TOL_F32, TOL_F64_F, TOL_F64_G, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("rows,cols", [(1, 700), (1, 40_001), (3, 24_576), (5, 24_580), (128, 12_289), (128, 49_156), (129, 33_000),
                                       (300, 17_000), (1023, 516), (1023, 2050), (1024, 516), (1026, 5000),
                                       (1031, 16_388), (2101, 1031)])
def test_row_pass(rows, cols, dtype):
    from paper_2507_13204_amd import DenseObjective
    d = inputs.dense(cols, seed=rows, rows=rows)
    A, w, x = (to_dev(t, dtype) for t in (d.A, d.w, d.x))
    f_ref, g_ref = oracle.dense_gradient(*(t.double().cpu().numpy() for t in (A, x, w)))
    tf, tg = (TOL_F64_F, TOL_F64_G) if dtype == torch.float64 else (TOL_F32, TOL_F32)
    off = torch.empty(cols + 1, dtype=dtype, device="cuda")[1:]
    off.copy_(x)
    obj = DenseObjective(A, w)
    fbar = torch.tensor([0.5], dtype=torch.float64, device="cuda")
    for v in (x, off):
        assert srel(obj.objective(v).item(), f_ref) <= tf
        f, g = obj.gradient(v)
        assert srel(f.item(), f_ref) <= tf and rel(g.cpu().numpy(), g_ref) <= tg
        assert rel(obj.adjoint(v, fbar).cpu().numpy(), 0.5 * g_ref) <= tg
