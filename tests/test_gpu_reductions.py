"""Products and sums whose reduction is split over workgroups, at the edges of
the splits: unfolding Grams with one, a few and some thousand K slabs (the
RoundSum's truncation sees them through its result), operands that end inside
a tile, a strip of 16, a half slab or a k step, and squared norms just below
and above the length from which they are spread.  A RoundSum of a sum whose
rank fits is exact up to rounding: 1e-10 in FP64 (the tolerance asked of the
truncation), 2e-4 in the FP32 form."""
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


def _tensor(rng, ns, r):
    return O.Tucker(rng.standard_normal((r,) * len(ns)) / r,
                    [np.linalg.qr(rng.standard_normal((n, r)))[0] for n in ns])


# s = cap + p is the side of the projected core: 3 .. 64 in three dimensions
# (1 to 128 slabs of 32 per Gram), up to 37 in four (1600 slabs, folded)
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("ns,r,cap,p", [((9, 8, 7), 1, 2, 1), ((20, 21, 22), 4, 8, 3), ((30,) * 3, 5, 11, 4),
                                        ((40, 33, 47), 7, 14, 3), ((70, 65, 64), 15, 30, 2), ((70,) * 3, 16, 32, 1),
                                        ((90, 80, 85), 20, 44, 5), ((100,) * 3, 24, 56, 8), ((24, 23, 22, 21), 4, 8, 2),
                                        ((33,) * 4, 8, 16, 1), ((50, 48, 46, 44), 10, 24, 5), ((48,) * 4, 12, 30, 3)])
def test_roundsum_split_reductions(tk, ns, r, cap, p, form):
    rng = np.random.default_rng(len(ns) * 1000 + cap)
    X = [(1.0, _tensor(rng, ns, r)), (-0.5, _tensor(rng, ns, r))]
    om = [_cm(rng.standard_normal((n, cap + p))) for n in ns]
    w, s = tk.rhosvd([(c, tk.Tucker.from_numpy(x.core, x.U)) for c, x in X], om, 1e-4 if form else 1e-10, cap, p,
                     form=form)
    got = O.Tucker(*w.to_numpy())
    err = O.exact_norm([(1.0, got)] + [(-c, x) for c, x in X]) / O.exact_norm(X)
    print(f"split reductions {ns} s {cap + p} form {form}: ranks {w.ranks} err {err:.1e}", flush=True)
    assert err <= (2e-4 if form else 1e-10)


@pytest.mark.parametrize("n,r", [(40, 40), (41, 41), (64, 31), (64, 32), (64, 33), (80, 63)])
def test_norm_of_long_cores(tk, n, r):
    """r^3 entries around 64 K, aligned and not: orthonormal factors, so the
    norm is the core's (1e-13: a sum of positive terms)."""
    rng = np.random.default_rng(r)
    core = rng.standard_normal((r, r, r))
    U = [np.linalg.qr(rng.standard_normal((n, r)))[0] for _ in range(3)]
    got = tk.norm([(2.0, tk.Tucker.from_numpy(core, U))])
    assert abs(got / (2.0 * np.linalg.norm(core)) - 1.0) <= 1e-13
