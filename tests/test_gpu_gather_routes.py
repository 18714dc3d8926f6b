"""Gathers whose reverse may go through the transposed connectivity: which of
them do, what is reserved for it, and what a changed connectivity costs."""
import numpy as np
import pytest

from oracle import program as OP
from _helpers import TOL_F64_F, TOL_F64_G, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _gather(n, E, k, seed):
    """Input of n entries, and the spec of sum w psi(gather of E random rows)."""
    rng = np.random.default_rng(seed)
    x = rng.uniform(-1.0, 1.0, n)
    conn = rng.integers(0, n, size=(E, k)).astype(np.int32)
    B, w = rng.standard_normal((E, k)) / np.sqrt(k), rng.uniform(0.5, 1.5, E)
    return x, [("input", n), ("gather", 0, conn, B), ("map", 1, "psi"), ("const", w),
               ("mul", 2, 3), ("sum", 4)]


def _check(prog, spec, x):
    f, (g,) = prog.run([to_dev(x)])
    f_ref, (g_ref,) = OP.gradient(spec, [x])
    assert srel(f.item(), f_ref) < TOL_F64_F and rel(g.cpu().numpy(), g_ref) < TOL_F64_G


@pytest.mark.parametrize("times,atomics", [(8, 0), (9, 1), (40, 1)])
def test_operands_far_longer_than_the_gather(times, atomics):
    """A pass over every entry does not replace a few atomics, nor is room kept
    for it."""
    from paper_2507_13204_amd import Program
    E, k = 16_400, 4
    n = E * k * times
    x, spec = _gather(n, E, k, times)
    prog = Program.from_spec(spec).plan("cuda")
    assert prog.info()["atomic_ops"] == atomics
    assert (prog.workspace_bytes < 8 * n + (1 << 20)) == bool(atomics)
    _check(prog, spec, x)
