"""Hooks that hand the native autograd node other tensors than it saved or was
sent: refused, or taken, as the Python Function does."""
import pytest

from paper_2507_13204_amd import inputs
from _helpers import TOL_F64_G, rel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _mesh(policy):
    from paper_2507_13204_amd import MeshObjective
    m = inputs.hex_mesh(9, seed=7)
    obj = MeshObjective(to_dev(m.conn), to_dev(m.B), to_dev(m.w), m.n_nodes, autograd=policy)
    return obj, to_dev(m.x).requires_grad_(True)


def _fns():
    from paper_2507_13204_amd import MeshFn

    class Sub(MeshFn):  # a subclass goes through the Python Function
        pass
    return MeshFn, Sub


# What unpacking returns of each saved tensor: the gradient, or the tape and x.
UNPACK = {"host": lambda t: t.cpu(), "half": lambda t: t.half(),
          "strided": lambda t: torch.stack([t, t], -1)[..., 0], "short": lambda t: t[:t.numel() // 2]}


@pytest.mark.parametrize("policy,what", [("gradient", "host"), ("gradient", "half"), ("gradient", "strided"),
                                         ("store", "host"), ("store", "strided")])
def test_unpacked_tensors_are_checked(policy, what):
    from paper_2507_13204_amd.pgrad import PgError
    obj, x = _mesh(policy)
    for fn in _fns():
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t, UNPACK[what]):
            f = fn.apply(x, obj)
        with pytest.raises(PgError):
            f.backward()
        assert x.grad is None


def test_a_tape_too_short_is_refused():
    from paper_2507_13204_amd.pgrad import PgError
    obj, x = _mesh("store")
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, UNPACK["short"]):
        f = _fns()[0].apply(x, obj)
    with pytest.raises(PgError):
        f.backward()


@pytest.mark.parametrize("policy", ["gradient", "store"])
def test_a_seed_from_a_hook_is_checked(policy):
    from paper_2507_13204_amd.pgrad import PgError
    obj, x = _mesh(policy)
    for fn in _fns():
        f = fn.apply(x, obj)
        f.register_hook(lambda g: g.cpu())
        with pytest.raises((PgError, RuntimeError)):
            f.backward()
        assert x.grad is None


def test_copies_are_taken():
    """Tensors of the right kind serve as well as those that were saved; of x
    only the shape is needed."""
    for policy in ("gradient", "store"):
        obj, x = _mesh(policy)
        _fns()[0].apply(x, obj).backward()
        want, x.grad = x.grad, None
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), lambda t: t.cuda()):
            f = _fns()[0].apply(x, obj)
        f.backward()
        assert rel(x.grad.cpu().numpy(), want.cpu().numpy()) <= TOL_F64_G
    x.grad = None
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: t.cpu() if t.numel() == x.numel() else t):
        f = _fns()[0].apply(x, obj)
    f.backward()
    assert rel(x.grad.cpu().numpy(), want.cpu().numpy()) <= TOL_F64_G


@pytest.mark.parametrize("policy", ["gradient", "store"])
def test_an_error_of_the_forward_is_the_bindings(policy):
    from paper_2507_13204_amd.pgrad import PgError
    obj, x = _mesh(policy)
    empty = torch.empty(0, dtype=torch.float64, device="cuda", requires_grad=True)  # a NULL pointer
    for fn in _fns():
        with pytest.raises(PgError):
            fn.apply(empty, obj)
    _fns()[0].apply(x, obj).backward()
    assert torch.isfinite(x.grad).all()


def test_grad_fn_has_the_contexts_attributes():
    """What a caller could read of the Function's context through f.grad_fn."""
    import gc
    import weakref
    from paper_2507_13204_amd import DenseFn, DenseObjective
    for policy in ("gradient", "store"):
        obj, x = _mesh(policy)
        for fn in _fns():
            f = fn.apply(x, obj)
            ctx = f.grad_fn
            assert ctx.obj is obj and ctx.policy == policy and ctx.needs_input_grad == (True, False, False)
            saved = ctx.saved_tensors
            assert [t.shape for t in saved][-1] == x.shape and len(saved) == (2 if policy == "store" else 1)
            assert ctx.next_functions[0][0].name() == "torch::autograd::AccumulateGrad"
            f.backward()
            if policy == "gradient":
                assert torch.equal(x.grad, saved[0])
            with pytest.raises(RuntimeError, match="second time"):
                ctx.saved_tensors
            x.grad = None
    f = _fns()[0].apply(x, obj)
    assert f.grad_fn is f.grad_fn and f.grad_fn.name() == type(f.grad_fn).__name__ == "MeshFnBackward"
    A = torch.ones(3, 4, dtype=torch.float64, device="cuda")
    d = DenseObjective(A, torch.ones(3, dtype=torch.float64, device="cuda"))
    y = torch.ones(4, dtype=torch.float64, device="cuda", requires_grad=True)
    assert type(DenseFn.apply(y, d).grad_fn).__name__ == "DenseFnBackward"
    ref = weakref.ref(obj)  # reading the attributes keeps nothing
    del f, obj, ctx, saved
    gc.collect()
    assert ref() is None
