"""Every entry of the FP32 batched products against FP64: operands whose sums
have one term, cancel, mix magnitudes or are all positive, very small or very
large, on the FP32 instruction and in every tile shape of the split."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

U = 2.0 ** -24  # rounding of one FP32 operation


def _operands(kind, m, n, dev="cuda"):
    g = torch.Generator(device=dev)
    g.manual_seed(m + n)
    uni = lambda *s: torch.rand(*s, generator=g, device=dev, dtype=torch.float64)
    nor = lambda *s: torch.randn(*s, generator=g, device=dev, dtype=torch.float64)
    if kind == "one_term":
        A = torch.zeros(m, m, device=dev, dtype=torch.float64)
        A[torch.arange(m, device=dev), torch.randperm(m, generator=g, device=dev)] = 1 + uni(m)
        X = 1 + uni(m, n)
    elif kind == "cancel":  # terms 2 i and 2 i + 1 cancel to 1e-3, by rows and by columns
        h = m // 2
        A, X = nor(m, m), 1 + uni(m, n)
        A[1:2 * h:2] = -A[0:2 * h:2] * (1 + 1e-3 * nor(h, m))
        A[:, 1:2 * h:2] = -A[:, 0:2 * h:2] * (1 + 1e-3 * nor(m, h))
        X[1:2 * h:2] = X[0:2 * h:2]
    elif kind == "mixed":  # within each run of 32 terms
        s = torch.tensor([1.0, 2.0 ** 10, 2.0 ** -10, 2.0 ** 5, 2.0 ** -20], device=dev, dtype=torch.float64)
        s = s[torch.arange(m, device=dev) % 5]
        A, X = nor(m, m) * s[None, :] * s[:, None], nor(m, n)
    elif kind == "positive":
        A, X = 1 + uni(m, m), 1 + uni(m, n)
    elif kind == "tiny":  # low parts far below the normal range of bfloat16
        A, X = nor(m, m) * 2.0 ** -122, nor(m, n)
    else:  # "huge": past what the scaled parts' products hold
        A, X = nor(m, m) * 2.0 ** 50, nor(m, n) * 2.0 ** 50
    return A.float(), X.float()


# 600 x 500: the FP32 instruction; the others split, in tiles of 48 x 128, 64 x
# 64, 128 x 128 and 64 x 128.
@pytest.mark.parametrize("m,n", [(600, 500), (1056, 1000), (1024, 1024), (4065, 1000), (5000, 300)])
@pytest.mark.parametrize("kind", ["one_term", "cancel", "mixed", "positive", "tiny", "huge"])
def test_entries(kind, m, n):
    from paper_2507_13204_amd import BatchedDense
    A, X = _operands(kind, m, n)
    W = torch.ones(m, n, device="cuda")
    obj = BatchedDense(A, W, ckpt="store", autograd="recompute")
    Ad, Xd = A.double(), X.double()
    tape = obj.new_tape("cuda")
    # The backward product of any V: G = A^T V, rounded once to FP32.  A sum of
    # 16 products rounds 16 times at most; a single term rounds in the small
    # parts' sums, 2^-8 of it, or is left to that last rounding.
    tape.zero_()
    tape.view(torch.float32)[:m * n].view(m, n).copy_(X)
    fbar = torch.ones(1, dtype=torch.float64, device="cuda")
    G = obj.adjoint_tape(fbar, tape, like=X).double()
    At = Ad.t().contiguous()
    want, S = At @ Xd, At.abs() @ Xd.abs()
    eG = (0 if kind == "one_term" else 16) * U * S + 2.0 ** -29 * S
    assert ((G - want).abs() <= eG + U * want.abs() + 2.0 ** -149).all()
    if kind in ("tiny", "huge"):
        return  # psi of these is no test of the product
    # The forward product through V = psi'(Y), whose slope is at most 2, and f.
    f = obj.objective_tape(X, tape)
    V = tape.view(torch.float32)[:m * n].view(m, n).double()
    Y, S = Ad @ Xd, Ad.abs() @ Xd.abs()
    want = Y + Y / (1 + Y * Y)
    assert ((V - want).abs() <= 2 * 16 * U * S + U * want.abs()).all()
    if kind in ("one_term", "positive"):
        # one entry's error is 2^-24 of it, of either sign, on the FP32 instruction;
        # and 2^-29 in the split's small parts, twice that in f
        fw = (0.5 * Y * Y + 0.5 * torch.log1p(Y * Y)).sum()
        assert abs((f - fw) / fw).item() <= 4e-9
