"""Reverse of large scattered gathers through the transposed connectivity:
both sides of the rule, each row length, first and later deliveries, and a
connectivity changed after the plan was bound."""
import numpy as np
import pytest

from oracle import program as OP
from paper_2507_13204_amd import inputs
from _helpers import TOL_F64_F, TOL_F64_G, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _spec(n, conn, B, w, twice=False, hot=False):
    """sum w psi(gather(x)); twice: x is read by a later construct too, so the
    gather's delivery is not the first into its shadow."""
    E = conn.shape[0]
    if not twice:
        return [("input", n), ("gather", 0, conn, B), ("map", 1, "psi"), ("const", w),
                ("mul", 2, 3), ("sum", 4)]
    # views 5.. read x again through a stencil of the gather's own length
    assert n == E
    return [("input", n), ("gather", 0, conn, B), ("map", 1, "psi"), ("const", w), ("mul", 2, 3),
            ("stencil", 0, [-1, 0, 2], [0.5, -1.0, 0.25]), ("map", 5, "square"),
            ("add", 4, 1.0, 6, 0.3), ("sum", 7)]


def _case(n, E, k, seed, span=None):
    rng = np.random.default_rng(seed)
    x = rng.uniform(-1.0, 1.0, n)
    conn = rng.integers(0, n if span is None else span, size=(E, k)).astype(np.int32)
    return x, conn, rng.standard_normal((E, k)) / np.sqrt(k), rng.uniform(0.5, 1.5, E)


def _run(spec, x, fusion):
    from paper_2507_13204_amd import Program
    prog = Program.from_spec(spec, fusion=fusion).plan("cuda")
    return prog, prog.run([to_dev(x)])


@pytest.mark.parametrize("fusion", [0, 1])
@pytest.mark.parametrize("twice", [False, True])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 11])
def test_scattered_gather(k, twice, fusion):
    n = E = max(40_011, (1 << 16) // k + 7)  # past the size the rule asks for, ragged
    x, conn, B, w = _case(n, E, k, 70 + k)
    spec = _spec(n, conn, B, w, twice)
    prog, (f, (g,)) = _run(spec, x, fusion)
    assert prog.info()["atomic_ops"] == 0 and prog.info()["rescheduled_ops"] == 1 + twice
    f_ref, (g_ref,) = OP.gradient(spec, [x])
    assert srel(f.item(), f_ref) < TOL_F64_F and rel(g.cpu().numpy(), g_ref) < TOL_F64_G
    f2, (g2,) = prog.run([to_dev(x)])
    assert torch.equal(f, f2) and torch.equal(g, g2)  # no atomics: the same bits
    fbar = torch.tensor([-0.5], dtype=torch.float64, device="cuda")
    _, (g3,) = prog.run([to_dev(x)], fbar=fbar)
    assert rel(g3.cpu().numpy(), -0.5 * g_ref) < TOL_F64_G


@pytest.mark.parametrize("what", ["small", "local", "hot"])
def test_other_gathers_keep_the_atomics(what):
    """Below the size, with entries that share cache lines, and with an entry
    of many incidences."""
    n, E, k = (5000, 8191, 8) if what == "small" else (40_000, 40_000, 4)
    x, conn, B, w = _case(n, E, k, 91)
    if what == "local":
        conn = ((np.arange(E)[:, None] + np.arange(k)) % n).astype(np.int32)
    if what == "hot":
        conn[::100, 0] = 7
    spec = _spec(n, conn, B, w)
    prog, (f, (g,)) = _run(spec, x, 1)
    assert prog.info()["atomic_ops"] == 1
    f_ref, (g_ref,) = OP.gradient(spec, [x])
    assert srel(f.item(), f_ref) < TOL_F64_F and rel(g.cpu().numpy(), g_ref) < TOL_F64_G


@pytest.mark.parametrize("fusion", [0, 1])
@pytest.mark.parametrize("twice", [False, True])
@pytest.mark.parametrize("k", [5, 8])
def test_changed_connectivity_and_coefficients(k, twice, fusion):
    """conn and B are read on every run: written to in place after the plan was
    bound, the results are those of what they now hold."""
    from paper_2507_13204_amd import Program
    n = E = 40_011
    x, conn, B, w = _case(n, E, k, 55)
    cd, Bd = to_dev(conn), to_dev(B)
    prog = Program.from_spec(_spec(n, cd, Bd, w, twice), fusion=fusion).plan("cuda")
    assert prog.info()["atomic_ops"] == 0
    prog.run([to_dev(x)])
    for step in range(3):
        if step == 0:
            Bd.mul_(1.25)
        elif step == 1:
            cd[E - 1, k - 1] = (int(cd[E - 1, k - 1]) + 17) % n  # one entry
        else:
            cd.copy_(to_dev(np.roll(conn, 3, axis=0)))
        f, (g,) = prog.run([to_dev(x)])
        f_ref, (g_ref,) = OP.gradient(_spec(n, cd.cpu().numpy(), Bd.cpu().numpy(), w, twice), [x])
        assert srel(f.item(), f_ref) < TOL_F64_F and rel(g.cpu().numpy(), g_ref) < TOL_F64_G, step


@pytest.mark.parametrize("n,E,k", [
    (700_001, 100_003, 8),  # one list: operand and products past the caches
    (300_007, 30_011, 8),   # one list: fewer incidences than entries
    (66_001, 8_300, 8),     # a part per XCD, 33 workgroups: one part longer
    (30_011, 210_000, 5),   # some 35 incidences per entry: runs past the first reads
])
def test_parts_of_the_products(n, E, k):
    """The products in one list and in one part per XCD (the same fixed order)."""
    x, conn, B, w = _case(n, E, k, 33)
    spec = _spec(n, conn, B, w)
    prog, (f, (g,)) = _run(spec, x, 1)
    assert prog.info()["atomic_ops"] == 0
    f_ref, (g_ref,) = OP.gradient(spec, [x])
    assert srel(f.item(), f_ref) < TOL_F64_F and rel(g.cpu().numpy(), g_ref) < TOL_F64_G
    f2, (g2,) = prog.run([to_dev(x)])
    assert torch.equal(f, f2) and torch.equal(g, g2)
