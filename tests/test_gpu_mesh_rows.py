"""Rows of every length up to the registers' limit and beyond, and both sides
of the rule that leaves the combining table out."""
import numpy as np
import pytest

import oracle
from paper_2507_13204_amd import inputs
from _helpers import TOL_F32, TOL_F64_F, TOL_F64_G, mesh_to_dev, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _check(m, dtype, **kw):
    from paper_2507_13204_amd import MeshObjective
    conn, B, w, x = mesh_to_dev(m, dtype)
    h = [t.double().cpu().numpy() for t in (B, w, x)]
    f_ref, g_ref = oracle.mesh_gradient(m.n_nodes, m.conn, *h)
    tf, tg = (TOL_F64_F, TOL_F64_G) if dtype == "f64" else (TOL_F32, TOL_F32)
    obj = MeshObjective(conn, B, w, m.n_nodes, **kw)
    f, g = obj.gradient(x)
    assert srel(f.item(), f_ref) <= tf and rel(g.cpu().numpy(), g_ref) <= tg, m.name
    fbar = torch.tensor([1.5], dtype=torch.float64, device="cuda")
    assert srel(obj.objective(x).item(), f_ref) <= tf
    assert rel(obj.adjoint(x, fbar).cpu().numpy(), 1.5 * g_ref) <= tg
    v = torch.linspace(-1, 1, m.n_nodes, dtype=torch.float64, device="cuda").to(x.dtype)
    hv = oracle.mesh_hvp(m.n_nodes, m.conn, *h, v.double().cpu().numpy())
    assert rel(obj.hvp(x, v).cpu().numpy(), hv) <= tg
    assert srel(obj.jvp(x, v).item(), float(g_ref @ v.double().cpu().numpy())) <= max(tf, 1e-9)
    return obj


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("k", [1, 3, 5, 6, 7, 9, 10, 15, 16, 17, 27, 32])
def test_row_lengths(k, dtype):
    _check(inputs.ring_mesh(1537, k, seed=k), dtype)
    _check(inputs.random_mesh(800, 1025, k, seed=k), dtype, ckpt="store" if k % 2 else "recompute",
           scatter=k % 4) if k % 2 == 0 else _check(inputs.random_mesh(800, 1025, k, seed=k), dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("k,nodes,table", [(8, 3000, True), (8, 40_000, False), (4, 4500, True),
                                           (4, 60_000, False), (6, 40_000, False), (10, 40_000, False)])
def test_combining_rule(k, nodes, table, dtype):
    """Random rows that share nodes keep the table, those that do not go to
    memory directly; a size the caller fixes is kept."""
    m = inputs.random_mesh(nodes, 35_000, k, seed=3)
    assert (_check(m, dtype).info()["lds_slots"] > 0) == table
    assert _check(m, dtype, scatter=2).info()["lds_slots"] == 4096


@pytest.mark.parametrize("k", [5, 11])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_not_finite_entry(k, bad):
    """One entry that is not finite reaches its rows' nodes and no others (the
    entries past a row and the lanes past the mesh add nothing)."""
    from paper_2507_13204_amd import MeshObjective
    m = inputs.ring_mesh(700, k, seed=1)
    x = m.x.copy()
    x[699] = bad  # read by the last rows, whose lanes the idle ones repeat
    obj = MeshObjective(to_dev(m.conn), to_dev(m.B), to_dev(m.w), m.n_nodes)
    f, g = obj.gradient(to_dev(x))
    hit = np.zeros(700, bool)
    for e in range(700 - k, 700):
        hit[(e + np.arange(k)) % 700] |= 699 in (e + np.arange(k)) % 700
    assert not np.isfinite(f.item())
    assert np.array_equal(~np.isfinite(g.cpu().numpy()), hit)
