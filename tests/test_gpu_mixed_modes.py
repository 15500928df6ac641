"""RoundSum with unequal mode sizes: the products of all modes share grouped
launches with dims per group, and the effective-rank rule's modes are gathered
by the side their Gram is on (n-side by size; R-side together).  Widths and
ranks must equal the oracle's; the result is the sum to 1e-9 (exact up to
rounding at the asked 1e-10)."""
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
@pytest.mark.parametrize("ns,nb,r,dims,cap", [
    ((200, 70, 40), 2, 16, (12, 9, 15), 18),        # R-side twice (Rp = 36), n-side
    ((65, 30, 31), 1, 20, (17, 12, 20), 24),        # R-side, two n-sides of different order
    ((90, 300, 163), 3, 30, (22, 30, 11), 33),      # n-side (Rp = 99 > 90), R-side twice
    ((170, 190, 500), 4, 44, (20, 40, 31), 45),     # Rp = 180: above n, below n twice; both eigensolvers planned
    ((64, 512, 65, 20), 2, 8, (8, 5, 7, 6), 12),    # four modes
])
def test_unequal_modes(tk, ns, nb, r, dims, cap, tau):
    rng = np.random.default_rng(sum(ns) + nb)
    B = [np.linalg.qr(rng.standard_normal((n, q)))[0] for n, q in zip(ns, dims)]
    blocks = [(float(rng.uniform(0.5, 1.5)),
               O.Tucker(rng.standard_normal((r,) * len(ns)) / r,
                        [Bk @ rng.standard_normal((q, r)) for Bk, q in zip(B, dims)])) for _ in range(nb)]
    p = 4
    Om = [rng.standard_normal((n, cap + p)) for n in ns]
    ref, info = O.roundsum(blocks, Om, O.RoundParams(eps=1e-10, cap=cap, p=p, tau=tau))
    got, s = tk.rhosvd([(c, tk.Tucker.from_numpy(X.core, X.U)) for c, X in blocks],
                       [torch.from_numpy(np.ascontiguousarray(o.T)).cuda() for o in Om], 1e-10, cap, p,
                       tau=-1.0 if tau is None else tau)
    g = O.Tucker(*got.to_numpy())
    err = O.exact_norm([(1.0, g)] + [(-c, x) for c, x in blocks]) / O.exact_norm(blocks)
    print(f"{ns} blocks {nb} r {r} tau {tau}: oracle r~ {info['rtilde']} s {info['s']}, gpu s {s} ranks {got.ranks} "
          f"err {err:.1e}", flush=True)
    assert s == info["s"] and got.ranks == tuple(info["ranks"])
    assert err <= 1e-9
