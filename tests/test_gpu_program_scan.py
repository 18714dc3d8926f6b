"""Scans by number of chunks (2,048 entries each): one, two and three launches,
stored and added reverse deliveries, both pass directions."""
import numpy as np
import pytest

from oracle import program as OP
from _helpers import TOL_F64_F, TOL_F64_G, rel, srel, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CHUNK, DIRECT = 2048, 8192


@pytest.mark.parametrize("n", [1, 7, CHUNK - 1, CHUNK, CHUNK + 1, 5 * CHUNK + 3, 257 * CHUNK + 9,
                               DIRECT * CHUNK, DIRECT * CHUNK + 1])
@pytest.mark.parametrize("twice", [False, True])
def test_scan_lengths(n, twice):
    from paper_2507_13204_amd import Program
    rng = np.random.default_rng(n)
    x = rng.uniform(0.5, 1.5, n) * rng.choice([-1.0, 1.0], n) / np.sqrt(n)
    spec = [("input", n), ("scan", 0), ("map", 1, "square"), ("sum", 2)]
    if twice:  # x is read after the scan too: the scan's reverse adds to its shadow
        spec = spec[:3] + [("map", 0, "psi"), ("add", 2, 1.0, 3, -0.5), ("sum", 4)]
    prog = Program.from_spec(spec).plan("cuda")
    chunks = -(-n // CHUNK)
    scan = 1 if chunks == 1 else 2 if chunks <= DIRECT else 3
    assert prog.info()["fwd_kernels"] == scan + (1 if n <= 16_384 else 2)
    assert prog.info()["rev_kernels"] == scan
    f, (g,) = prog.run([to_dev(x)])
    y = np.cumsum(x)  # (the program oracle's scan is a dense matrix)
    f_ref, g_ref = np.sum(y * y), np.cumsum(2.0 * y[::-1])[::-1]
    if twice:
        f_ref, g_ref = f_ref - 0.5 * np.sum(OP._phi("psi", x)), g_ref - 0.5 * OP._dphi("psi", x)
    # both sides' running sums of n terms: at most n/2 ulp each
    tol = 2 * n * 2.0 ** -53
    assert srel(f.item(), f_ref) < TOL_F64_F + tol and rel(g.cpu().numpy(), g_ref) < TOL_F64_G + tol
    f2, (g2,) = prog.run([to_dev(x)])
    assert torch.equal(f, f2) and torch.equal(g, g2)
