"""Householder QR kernels at the edges of their row blocks (64, 128, 256 and 512
rows; 1 to 64 columns), through the calls that run them: the multilinear
Nystrom recovery (pivoted QR of an (r + p) x r matrix with a rank cut and a
plain QR of the kept rows) and the exact norm (R-only QR of n x r factors for
one block; pivoted QRs and re-orthogonalisation for two).  A sum of rank at
most r is recovered exactly, so the bound is the recovery's 1e-10; the norm is
held to 1e-12 (sums of squares of O(1) terms at 1e-16 each)."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def tk():
    import paper_2608_11091_amd as tk
    tk.load()
    return tk


def _cm(M):
    return torch.from_numpy(np.ascontiguousarray(M.T)).cuda()


@pytest.mark.parametrize("r,p,rank", [(1, 0, 1), (2, 1, 1), (16, 15, 16), (17, 47, 17), (32, 32, 20), (33, 32, 33),
                                      (48, 48, 48), (48, 79, 31), (48, 80, 48), (64, 64, 64), (40, 89, 40),
                                      (64, 192, 64)])
def test_recovery_rows(tk, r, p, rank):
    rng = np.random.default_rng(1000 * r + p)
    n, rt = max(80, r + p + 5), r + p
    X = O.Tucker(rng.standard_normal((rank,) * 3), [rng.standard_normal((n, rank)) for _ in range(3)])
    Psi = [_cm(rng.standard_normal((n, rt))) for _ in range(3)]
    core, F, _ = tk.mln_sketch([(1.0, tk.Tucker.from_numpy(X.core, X.U))], Psi, r)
    got = tk.mln_recover(core, F, Psi, r)
    dist = O.exact_norm([(1.0, O.Tucker(*got.to_numpy())), (-1.0, X)]) / O.exact_norm([(1.0, X)])
    print(f"recovery {rt} x {r}, rank {rank}: ranks {got.ranks} dist {dist:.1e}", flush=True)
    assert got.ranks == (rank,) * 3
    assert dist <= 1e-10


@pytest.mark.parametrize("n,r", [(1, 1), (15, 15), (16, 5), (64, 64), (65, 33), (128, 48), (129, 2), (256, 31), (257, 64),
                                 (320, 16), (511, 48), (512, 64)])
def test_norm_rows(tk, n, r):
    rng = np.random.default_rng(n + r)
    X = [O.Tucker(rng.standard_normal((r,) * 3), [rng.standard_normal((n, r)) for _ in range(3)]) for _ in range(2)]
    for blocks in ([(1.0, X[0])], [(1.0, X[0]), (-0.5, X[1])]):
        ref = O.exact_norm(blocks)
        got = tk.norm([(c, tk.Tucker.from_numpy(x.core, x.U)) for c, x in blocks])
        print(f"norm n {n} r {r} blocks {len(blocks)}: {got / ref - 1.0:.1e}", flush=True)
        assert abs(got / ref - 1.0) <= 1e-12
