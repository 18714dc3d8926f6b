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


def test_changed_connectivity_takes_its_gather_alone_to_the_atomics():
    """Two transposed gathers, conn of one written to in place: its run and all
    later ones are right, later ones with atomics again (as info says once the
    run has ended), the other gather keeps its order; a graph captured before
    the change stays right; binding again starts afresh."""
    from paper_2507_13204_amd import Program
    n, E, k = 40_011, 40_011, 4
    rng = np.random.default_rng(3)
    x = rng.uniform(-1.0, 1.0, n)
    conn = [rng.integers(0, n, size=(E, k)).astype(np.int32) for _ in range(2)]
    B = [rng.standard_normal((E, k)) for _ in range(2)]
    cd, Bd = [to_dev(c) for c in conn], [to_dev(b) for b in B]

    def spec(c, b):
        return [("input", n), ("gather", 0, c[0], b[0]), ("map", 1, "psi"), ("gather", 0, c[1], b[1]),
                ("map", 3, "square"), ("add", 2, 1.0, 4, 0.5), ("sum", 5)]

    def check(f, g):
        f_ref, (g_ref,) = OP.gradient(spec([c.cpu().numpy() for c in cd], B), [x])
        assert srel(f.item(), f_ref) < TOL_F64_F and rel(g.cpu().numpy(), g_ref) < TOL_F64_G

    prog = Program.from_spec(spec(cd, Bd)).plan("cuda")
    xd, gc = to_dev(x), torch.empty(n, dtype=torch.float64, device="cuda")
    fc = torch.empty((), dtype=torch.float64, device="cuda")
    before = prog.info()
    assert before["atomic_ops"] == 0 and before["rescheduled_ops"] == 2
    f, (g,) = prog.run([xd])
    check(f, g)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        prog.run([xd], grads=[gc], f_out=fc)
    for step in range(3):
        cd[1].copy_(to_dev(np.roll(conn[1], 1 + step, axis=0)))
        for _ in range(2):
            f, (g,) = prog.run([xd])
            check(f, g)
        now = prog.info()
        assert now["atomic_ops"] == 1 and now["rescheduled_ops"] == 1
        assert now["rev_kernels"] == before["rev_kernels"] - 2
        graph.replay()
        check(fc, gc)
        xd.mul_(1.0)  # eager work between the replays
        graph.replay()
        check(fc, gc)
    prog.plan("cuda")
    assert prog.info() == before
    f, (g,) = prog.run([xd])
    check(f, g)


def test_room_is_kept_only_where_it_is_used():
    """A structured connectivity reserves nothing for the transposed order;
    two gathers share what one of them uses at a time."""
    from paper_2507_13204_amd import Program
    n, E, k = 40_011, 40_011, 4
    x, spec = _gather(n, E, k, 5)
    one = Program.from_spec(spec).plan("cuda")
    local = list(spec)
    local[1] = ("gather", 0, ((np.arange(E)[:, None] + np.arange(k)) % n).astype(np.int32), spec[1][3])
    prog = Program.from_spec(local).plan("cuda")
    assert prog.workspace_bytes < 8 * n + (1 << 16) < one.workspace_bytes
    _check(prog, local, x)
    two = spec[:4] + [("mul", 2, 3), ("gather", 0, np.roll(spec[1][2], 1, axis=1), spec[1][3]),
                      ("map", 5, "square"), ("add", 4, 1.0, 6, 0.5), ("sum", 7)]
    prog = Program.from_spec(two).plan("cuda")
    assert prog.info()["atomic_ops"] == 0
    # of its own: places, rows and (in eight parts) offsets; the group that adds
    # the two keeps one gathered value and its shadow
    assert prog.workspace_bytes - one.workspace_bytes <= 8 * E * k + 32 * (n + 1) + 16 * E + 4096
    _check(prog, two, x)
