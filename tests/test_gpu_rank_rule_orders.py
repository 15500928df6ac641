"""Effective-rank rule (Sec. 3.1) over the orders of the register eigensolver:
its Gram is taken on the n-side or on the R-side (FP64, 64 < n <= 160, the
concatenation narrower than n), the reduction is compiled for orders up to
64, 112 and 160, and a threshold tau far below the zero clamp leaves one
eigenvalue and one count instead of the spectrum.  Every sum has factors in a
subspace whose dimension, below the cap, is the rule's answer; the sketch
width must equal the oracle's exactly, for a tau under the clamp (the count)
and for one above it (the spectrum and its tail)."""
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


@pytest.mark.parametrize("tau", [None, 1e-3])
@pytest.mark.parametrize("n,nb,r,dim,cap", [
    (12, 1, 1, 1, 4),       # n-side, rank 1
    (64, 2, 20, 17, 30),    # n-side, largest order of the short body
    (65, 2, 20, 17, 30),    # R-side, R = 40 of 60
    (100, 2, 32, 30, 40),   # R-side, R = 64
    (100, 2, 33, 30, 40),   # R-side, R = 66
    (113, 2, 56, 41, 56),   # R-side, R = 112
    (113, 3, 38, 35, 38),   # n-side, order 113 (R = 114 > n)
    (160, 3, 40, 33, 50),   # R-side, R = 120
    (160, 3, 53, 44, 53),   # R-side, R = 159
    (160, 4, 41, 37, 41),   # n-side, order 160
])
def test_rank_rule_orders(tk, n, nb, r, dim, cap, tau):
    rng = np.random.default_rng(1000 * n + r)
    blocks = []
    B = [np.linalg.qr(rng.standard_normal((n, dim)))[0] for _ in range(3)]
    for b in range(nb):
        U = [Bk @ rng.standard_normal((dim, r)) for Bk in B]
        blocks.append((float(rng.uniform(0.5, 1.5)), O.Tucker(rng.standard_normal((r,) * 3), U)))
    p = 4
    Om = [rng.standard_normal((n, cap + p)) for _ in range(3)]
    ref, info = O.roundsum(blocks, Om, O.RoundParams(eps=1e-10, cap=cap, p=p, tau=tau))
    got, s = tk.rhosvd([(c, tk.Tucker.from_numpy(X.core, X.U)) for c, X in blocks],
                       [torch.from_numpy(np.ascontiguousarray(o.T)).cuda() for o in Om], 1e-10, cap, p,
                       tau=-1.0 if tau is None else tau)
    print(f"n {n} blocks {nb} r {r} dim {dim} tau {tau}: oracle r~ {info['rtilde']} s {info['s']}, gpu s {s}",
          flush=True)
    assert max(info["rtilde"]) <= dim < cap + p
    assert s == info["s"] and got.ranks == tuple(info["ranks"])
