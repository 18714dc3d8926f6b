"""Fused groups on both sides of the register / LDS slot rule, up to the
largest group, forward and reverse apart and together."""
import numpy as np
import pytest

from oracle import program as OP
from _helpers import TOL_F64_F, TOL_F64_G, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _chain(n, n_in, n_const, n_ops, seed, tail):
    """n_ops pointwise constructs over n_in inputs and n_const constants, mixing
    scales, sums, products (one of a view with itself) and maps.  tail: the
    result goes through a scan, so the group exports its value and its reverse
    is a launch of its own."""
    rng = np.random.default_rng(seed)
    spec = [("input", n) for _ in range(n_in)]
    spec += [("const", rng.uniform(-1.0, 1.0, n)) for _ in range(n_const)]
    leaves = list(range(len(spec)))
    v = 0
    for j in range(n_ops):
        kind = ["mul", "add", "map", "scale", "self"][(j + seed) % 5]
        other = leaves[(j + 1) % len(leaves)]
        if kind == "mul":
            spec.append(("mul", v, other))
        elif kind == "self":
            spec.append(("mul", v, v))
        elif kind == "add":
            spec.append(("add", v, 0.7, other, -0.4))
        elif kind == "map":
            spec.append(("map", v, "psi" if j % 2 else "square"))
        else:
            spec.append(("scale", v, 0.8))
        v = len(spec) - 1
    if tail:
        spec += [("scan", v), ("scale", v + 1, 1.0 / n), ("map", v + 2, "square")]
        v = len(spec) - 1
    spec.append(("sum", v))
    return spec, [rng.uniform(-1.0, 1.0, n) for _ in range(n_in)]


@pytest.mark.parametrize("tail", [False, True])
@pytest.mark.parametrize("n_in,n_const,n_ops", [(1, 0, 1), (1, 0, 3), (2, 1, 1), (2, 1, 2), (1, 0, 4),
                                                (2, 2, 4), (3, 1, 7), (2, 2, 12), (4, 4, 8)])
def test_group_sizes(n_in, n_const, n_ops, tail):
    from paper_2507_13204_amd import Program
    for n in (1, 257, 700):
        spec, xs = _chain(n, n_in, n_const, n_ops, n_ops, tail)
        prog = Program.from_spec(spec).plan("cuda")
        f, gs = prog.run([to_dev(x) for x in xs])
        f_ref, g_ref = OP.gradient(spec, xs)
        assert srel(f.item(), f_ref) < TOL_F64_F
        assert srel(prog.run([to_dev(x) for x in xs], grads=None).item(), f_ref) < TOL_F64_F
        for g, gr in zip(gs, g_ref):
            assert rel(g.cpu().numpy(), gr) < TOL_F64_G, (n, n_in, n_const, n_ops, tail)
