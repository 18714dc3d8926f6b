"""The native autograd node against the Python Function it stands for: values,
gradients, saved tensors, errors, and the inputs that are left to the Function."""
import gc
import weakref

import numpy as np
import pytest

import oracle
from paper_2507_13204_amd import inputs
from _helpers import TOL_F32, TOL_F64_F, TOL_F64_G, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _mesh(dtype=torch.float64, policy="gradient", n=12):
    from paper_2507_13204_amd import MeshObjective
    m = inputs.hex_mesh(n, seed=7)
    obj = MeshObjective(to_dev(m.conn), to_dev(m.B, dtype), to_dev(m.w, dtype), m.n_nodes, autograd=policy)
    return m, obj, to_dev(m.x, dtype)


def test_plain_inputs_take_the_node():
    from paper_2507_13204_amd import MeshFn, pgrad
    _, obj, x = _mesh()
    f = MeshFn.apply(x.requires_grad_(True), obj)
    assert f.grad_fn.name() == "MeshFnBackward"
    assert type(f.grad_fn).__module__ != "torch.autograd.function"  # no Python Function
    assert pgrad._node().__file__.endswith("_pgrad_torch.so")


def _python(cls, x, obj):
    """The same step through the Python Function."""
    class Sub(cls):  # a subclass is not taken by the node
        pass
    return Sub.apply(x, obj)


@pytest.mark.parametrize("policy", ["gradient", "store", "recompute"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_matches_the_python_function(policy, dtype):
    from paper_2507_13204_amd import MeshFn
    m, obj, x = _mesh(dtype, policy)
    got = []
    for fn in (MeshFn.apply, lambda a, o: _python(MeshFn, a, o)):
        a = x.clone().requires_grad_(True)
        f = fn(a * 2.0, obj)
        (3.0 * f).backward()
        got.append((f.detach(), a.grad))
    (f1, g1), (f2, g2) = got
    assert f1.dtype == f2.dtype and f1.shape == f2.shape == () and g1.dtype == dtype
    assert srel(f1.item(), f2.item()) <= TOL_F64_F and rel(g1.cpu().numpy(), g2.cpu().numpy()) <= TOL_F64_G * 1e3
    h = [t.double().cpu().numpy() for t in (obj.B, obj.w, x * 2.0)]
    f_ref, g_ref = oracle.mesh_gradient(m.n_nodes, m.conn, *h, fbar=3.0)
    tol = TOL_F64_G if dtype == torch.float64 else TOL_F32
    assert rel(g1.cpu().numpy(), 2.0 * g_ref) <= tol


def test_other_objectives_and_a_strided_input():
    from paper_2507_13204_amd import (BatchedDense, BatchedDenseFn, DenseFn, DenseObjective, MeshBatch,
                                      MeshBatchFn)
    d = inputs.dense(60, seed=1, rows=40)
    obj = DenseObjective(to_dev(d.A), to_dev(d.w))
    wide = torch.stack([to_dev(d.x), to_dev(d.x)], 1).requires_grad_(True)
    DenseFn.apply(wide[:, 1], obj).backward()
    _, g_ref = oracle.dense_gradient(d.A, d.x, d.w)
    assert rel(wide.grad[:, 1].cpu().numpy(), g_ref) <= TOL_F64_G and not wide.grad[:, 0].any()
    b = inputs.batched_dense(70, 20, seed=2)
    ob, X = BatchedDense(to_dev(b.A), to_dev(b.W)), to_dev(b.X).requires_grad_(True)
    (BatchedDenseFn.apply(X, ob) * 0.5).backward()
    assert rel(X.grad.cpu().numpy(), 0.5 * oracle.bdense_gradient_fast(b.A, b.X, b.W)[1]) <= TOL_F64_G
    bt = inputs.uneven_batch(4, seed=3, lo=3, hi=6)
    om = MeshBatch(bt.inst, to_dev(bt.conn), to_dev(bt.B), to_dev(bt.w))
    xb = to_dev(bt.x).requires_grad_(True)
    f = MeshBatchFn.apply(xb, om)
    wts = torch.tensor([1.0, -2.0, 0.5, 3.0], dtype=torch.float64, device="cuda")
    (f * wts).sum().backward()
    for i in range(4):
        m = bt.instance(i)
        _, no = m.n_nodes, int(bt.inst[i][2])
        _, g = oracle.mesh_gradient(m.n_nodes, m.conn, m.B, m.w, m.x, fbar=float(wts[i]))
        assert rel(xb.grad[no:no + m.n_nodes].cpu().numpy(), g) <= TOL_F64_G


def test_graph_rules_are_kept():
    """Retained and second backwards, accumulation, saved-tensor hooks, an
    input changed in place before a store-policy backward, no_grad."""
    from paper_2507_13204_amd import MeshFn
    _, obj, x = _mesh()

    def near(p, q):  # two gradients of one x differ in the order of the atomics
        return rel(p.cpu().numpy(), q.cpu().numpy()) <= TOL_F64_G

    a = x.clone().requires_grad_(True)
    f = MeshFn.apply(a, obj)
    f.backward(retain_graph=True)
    once = a.grad.clone()
    f.backward()
    assert torch.equal(a.grad, 2 * once)  # the saved gradient, twice
    with pytest.raises(RuntimeError, match="second time"):
        f.backward()
    packed = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: (packed.append(t.shape), t.cpu())[1],
                                                  lambda t: t.cuda()):
        b = x.clone().requires_grad_(True)
        f = MeshFn.apply(b, obj)
    f.backward()
    assert packed == [x.shape] and near(b.grad, once)
    _, ob, _ = _mesh(policy="store")
    c = x.clone().requires_grad_(True)
    y = c * 1.0
    f = MeshFn.apply(y, ob)
    with torch.no_grad():
        y.add_(1.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        f.backward()
    with torch.no_grad():
        assert not MeshFn.apply(a, obj).requires_grad
    (g,) = torch.autograd.grad(MeshFn.apply(a, obj), a, create_graph=True)
    assert not g.requires_grad and near(g, once)


def test_left_to_the_function():
    """Subclasses, transforms, forward mode and CPU tensors behave as with the
    Python Function: the same results or the same kind of error."""
    from paper_2507_13204_amd import MeshFn
    from paper_2507_13204_amd.pgrad import PgError
    m, obj, x = _mesh()

    class Tagged(torch.Tensor):
        pass

    a = x.clone().as_subclass(Tagged).requires_grad_(True)
    f = MeshFn.apply(a, obj)
    f.backward()
    _, g_ref = oracle.mesh_gradient(m.n_nodes, m.conn, m.B, m.w, m.x)
    assert rel(a.grad.as_subclass(torch.Tensor).cpu().numpy(), g_ref) <= TOL_F64_G
    with pytest.raises(PgError):
        MeshFn.apply(x.cpu().requires_grad_(True), obj)
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda t: MeshFn.apply(t, obj))(x)
    import torch.autograd.forward_ad as fw
    with fw.dual_level(), pytest.raises(RuntimeError):
        MeshFn.apply(fw.make_dual(x.clone().requires_grad_(True), torch.ones_like(x)), obj)


def test_plan_lives_as_long_as_the_graph():
    from paper_2507_13204_amd import MeshFn
    _, obj, x = _mesh(policy="store")
    a = x.clone().requires_grad_(True)
    f = MeshFn.apply(a, obj)
    ref = weakref.ref(obj)
    del obj
    gc.collect()
    assert ref() is not None
    f.backward()
    assert torch.isfinite(a.grad).all()
    del f
    gc.collect()
    assert ref() is None


def test_a_closed_plan_raises():
    from paper_2507_13204_amd import MeshFn
    from paper_2507_13204_amd.pgrad import PgError
    _, obj, x = _mesh(policy="store")
    a = x.clone().requires_grad_(True)
    f = MeshFn.apply(a, obj)
    obj.close()
    with pytest.raises(PgError):
        f.backward()
    with pytest.raises(PgError):
        MeshFn.apply(a, obj)


def test_side_stream():
    from paper_2507_13204_amd import MeshFn
    m, obj, x = _mesh()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        a = x.clone().requires_grad_(True)
        f = MeshFn.apply(a, obj)
        f.backward()
    torch.cuda.current_stream().wait_stream(s)
    _, g_ref = oracle.mesh_gradient(m.n_nodes, m.conn, m.B, m.w, m.x)
    assert rel(a.grad.cpu().numpy(), g_ref) <= TOL_F64_G and np.isfinite(f.item())
