"""The counter by which the last workgroup of a small launch sums f."""
import numpy as np
import pytest

import oracle
from oracle import program as OP
from paper_2507_13204_amd import inputs
from _helpers import TOL_F64_F, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _mesh():
    from paper_2507_13204_amd import MeshObjective
    m = inputs.hex_mesh(30, seed=2)
    obj = MeshObjective(to_dev(m.conn), to_dev(m.B), to_dev(m.w), m.n_nodes)
    x = to_dev(m.x)
    return (lambda s, g, f: obj.gradient(x, out=g, f_out=f, stream=s)), m.n_nodes, \
        oracle.mesh_gradient(m.n_nodes, m.conn, m.B, m.w, m.x)[0]


def _paper():
    from paper_2507_13204_amd import Laplace1D
    n = 9_001
    rng = np.random.default_rng(4)
    x, b = rng.uniform(-1, 1, n), rng.uniform(-1, 1, n)
    obj = Laplace1D(n)
    xd, bd, gb = to_dev(x), to_dev(b), torch.empty(n, dtype=torch.float64, device="cuda")
    return (lambda s, g, f: obj.gradient(xd, bd, gx=g, gb=gb, f_out=f, stream=s)), n, \
        oracle.laplace1d_gradient(x, b)[0]


def _program():
    from paper_2507_13204_amd import Program
    n = 9_001
    x = np.random.default_rng(5).uniform(-1, 1, n)
    spec = [("input", n), ("map", 0, "psi"), ("mul", 0, 1), ("sum", 2)]
    prog, xd = Program.from_spec(spec).plan("cuda"), to_dev(x)
    return (lambda s, g, f: prog.run([xd], grads=[g], f_out=f, stream=s)), n, OP.objective(spec, [x])


@pytest.mark.parametrize("make", [_mesh, _paper, _program])
def test_calls_that_overlapped_leave_the_counter_ready(make):
    """Calls of one plan on two streams at once, which the plan's rules forbid,
    give no promise for their own f, but every later one is right."""
    call, n, want = make()
    g = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2)]
    f = [torch.empty((), dtype=torch.float64, device="cuda") for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(100):
        for q in range(2):
            call(streams[q], g[q], f[q])
    torch.cuda.synchronize()
    for _ in range(3):
        f[0].fill_(float("nan"))
        torch.cuda.synchronize()
        call(streams[0], g[0], f[0])
        torch.cuda.synchronize()
        assert srel(f[0].item(), want) <= TOL_F64_F


@pytest.mark.parametrize("n", [33, 34, 35, 41, 42, 44, 45])
def test_both_sides_of_the_lines(n):
    """Grids just below and above those up to which a gradient (72 workgroups),
    an objective (128) and a JVP (160) sum f themselves, repeated and with f
    written in place."""
    from paper_2507_13204_amd import MeshObjective
    m = inputs.hex_mesh(n, seed=n)
    f_ref, g_ref = oracle.mesh_gradient(m.n_nodes, m.conn, m.B, m.w, m.x)
    obj, x = MeshObjective(to_dev(m.conn), to_dev(m.B), to_dev(m.w), m.n_nodes), to_dev(m.x)
    d = torch.linspace(-1, 1, m.n_nodes, dtype=torch.float64, device="cuda")
    f = torch.empty((), dtype=torch.float64, device="cuda")
    j_ref = float(g_ref @ d.cpu().numpy())
    first = None
    for _ in range(3):
        obj.gradient(x, f_out=f)
        fg = f.clone()
        fo, j = obj.objective(x), obj.jvp(x, d)
        assert srel(fg.item(), f_ref) <= TOL_F64_F and srel(j.item(), j_ref) <= 1e-9
        assert torch.equal(fg, fo)  # the same partials in the same order, summed here or there
        assert first is None or torch.equal(first, fg)
        first = fg
