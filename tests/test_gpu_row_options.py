"""Rows of 9 to 16 entries (and shorter and longer ones) with each adjoint,
scatter and checkpoint, through one mesh and through a batch."""
import numpy as np
import pytest

import oracle
from paper_2507_13204_amd import inputs
from _helpers import TOL_F32, TOL_F64_F, TOL_F64_G, mesh_to_dev, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = {"f64": (TOL_F64_F, TOL_F64_G), "f32": (TOL_F32, TOL_F32)}


def _mesh_check(m, dtype, **kw):
    from paper_2507_13204_amd import MeshObjective
    conn, B, w, x = mesh_to_dev(m, dtype)
    h = [t.double().cpu().numpy() for t in (B, w, x)]
    f_ref, g_ref = oracle.mesh_gradient(m.n_nodes, m.conn, *h)
    tf, tg = TOL[dtype]
    obj = MeshObjective(conn, B, w, m.n_nodes, **kw)
    fbar = torch.tensor([-1.5], dtype=torch.float64, device="cuda")
    f, g = obj.gradient(x)
    assert srel(f.item(), f_ref) <= tf and rel(g.cpu().numpy(), g_ref) <= tg
    assert srel(obj.objective(x).item(), f_ref) <= tf  # what a stored tape holds for the adjoint
    assert rel(obj.adjoint(x, fbar).cpu().numpy(), -1.5 * g_ref) <= tg
    if kw.get("ckpt") == "store":
        tape = obj.new_tape("cuda")
        assert srel(obj.objective_tape(x, tape).item(), f_ref) <= tf
        obj.objective(2 * x)  # another tape in the workspace
        assert rel(obj.adjoint_tape(fbar, tape, x).cpu().numpy(), -1.5 * g_ref) <= tg


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("ckpt", ["recompute", "store"])
@pytest.mark.parametrize("k", [5, 9, 10, 15, 16, 17])
def test_mesh_scatters(k, ckpt, dtype):
    for scatter in (0, 1, 2, 3):
        _mesh_check(inputs.random_mesh(800, 1025, k, seed=k), dtype, ckpt=ckpt, scatter=scatter)
        _mesh_check(inputs.ring_mesh(1537, k, seed=k), dtype, ckpt=ckpt, scatter=scatter)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("ckpt", ["recompute", "store"])
@pytest.mark.parametrize("adjoint", ["gather", "colour", "tiled"])
@pytest.mark.parametrize("k", [5, 9, 10, 15, 16, 17])
def test_mesh_adjoints(k, adjoint, ckpt, dtype):
    _mesh_check(inputs.ring_mesh(1537, k, seed=k), dtype, ckpt=ckpt, adjoint=adjoint)
    if adjoint != "colour":  # random rows need more colours than there are
        _mesh_check(inputs.random_mesh(800, 1025, k, seed=k), dtype, ckpt=ckpt, adjoint=adjoint)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("ckpt", ["recompute", "store"])
@pytest.mark.parametrize("k", [3, 7, 9, 16, 17])
def test_batches(k, ckpt, dtype):
    from paper_2507_13204_amd import MeshBatch
    sizes = [(40, 70), (7, 3), (300, 999), (1, 2), (64, 0), (500, 257)]
    meshes = [inputs.random_mesh(nn, ne, k, 90 + i) for i, (nn, ne) in enumerate(sizes)]
    offs = np.cumsum([(0, 0)] + sizes, axis=0)
    inst = [(nn, ne, no, eo) for (nn, ne), (no, eo) in zip(sizes, offs)]
    cat = [np.concatenate([getattr(m, a) for m in meshes]) for a in ("conn", "B", "w", "x")]
    dt = {"f64": torch.float64, "f32": torch.float32}[dtype]
    conn, (B, w, x) = to_dev(cat[0]), (to_dev(a, dt) for a in cat[1:])
    h = [t.double().cpu().numpy() for t in (B, w, x)]
    seeds = np.linspace(-1.0, 2.0, len(sizes))
    f_ref, g_ref, a_ref = [], np.zeros(offs[-1][0]), np.zeros(offs[-1][0])
    for s, (nn, ne, no, eo) in zip(seeds, inst):
        f, g = oracle.mesh_gradient(nn, cat[0][eo:eo + ne], h[0][eo:eo + ne], h[1][eo:eo + ne], h[2][no:no + nn])
        f_ref.append(f)
        g_ref[no:no + nn], a_ref[no:no + nn] = g, s * g
    tf, tg = TOL[dtype]
    fbar = to_dev(seeds)
    for scatter in (0, 1):
        obj = MeshBatch(inst, conn, B, w, block=128, ckpt=ckpt, scatter=scatter)

        def same(f):
            assert all(srel(p, q) <= tf for p, q in zip(f.cpu().numpy(), f_ref))

        f, g = obj.gradient(x)
        same(f)
        assert rel(g.cpu().numpy(), g_ref) <= tg
        same(obj.objective(x))
        assert rel(obj.adjoint(x, fbar).cpu().numpy(), a_ref) <= tg
        tape = obj.new_tape("cuda")
        same(obj.objective_tape(x, tape, f_shape=(len(sizes),)))
        obj.objective(2 * x)
        assert rel(obj.adjoint_tape(fbar, tape, x).cpu().numpy(), a_ref) <= tg


@pytest.mark.parametrize("k,nodes,elems,table", [(1, 6000, 6000, False), (1, 400, 6000, True), (3, 6000, 6000, True),
                                                 (16, 30_000, 30_000, False), (10, 900, 20_000, True)])
def test_combining_rule(k, nodes, elems, table):
    """Rows that share too few nodes go to memory directly, in one mesh and in
    a batch; a size the caller fixes is kept."""
    from paper_2507_13204_amd import MeshBatch, MeshObjective
    ring = nodes == elems and k < 10
    m = inputs.ring_mesh(elems, k, seed=2) if ring else inputs.random_mesh(nodes, elems, k, seed=2)
    conn, B, w, x = mesh_to_dev(m, "f64")
    f_ref, g_ref = oracle.mesh_gradient(m.n_nodes, m.conn, m.B, m.w, m.x)
    inst = [(m.n_nodes, m.n_elems, 0, 0)]
    for scatter in (0, 2):
        for obj in (MeshObjective(conn, B, w, m.n_nodes, scatter=scatter), MeshBatch(inst, conn, B, w, scatter=scatter)):
            assert (obj.info()["lds_slots"] > 0) == (table or scatter == 2)
            f, g = obj.gradient(x)
            assert srel(f.reshape(-1)[0].item(), f_ref) <= TOL_F64_F and rel(g.cpu().numpy(), g_ref) <= TOL_F64_G
