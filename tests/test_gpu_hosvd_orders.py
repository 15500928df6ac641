"""ST-HOSVD eigensolver orders through RoundSum: the order is the sketch width
cap + p, so these cases walk it over the edges of the kernel's row blocks (8
rows a lane group), odd and even, from 1 to 64, on sums of full rank at the
cap and on sums whose rank lies well below the width (a rank-deficient Gram,
eigenvectors still a full orthonormal set).  Ranks equal the oracle's, and in
FP64 the widths (the width rule's cut at 1e-12 of the largest eigenvalue lies
below the rounding of an FP32 Gram).  Tensors: in FP64 the range basis, Gram and eigenvectors are each
orthonormal to O(s u) and the singular values decay by at most 1e4 with the
cut in a gap of 2, so the sum of a few hundred roundings amplified by the gap
stays below 1e-10; in FP32 (u = 6e-8) the same count gives 1e-4."""
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


def _tensor(rng, n, r, ratio):
    """Orthonormal factors, superdiagonal core with geometric singular values."""
    core = np.zeros((r,) * 3)
    i = np.arange(r)
    core[i, i, i] = ratio ** i
    return O.Tucker(core, [np.linalg.qr(rng.standard_normal((n, r)))[0] for _ in range(3)])


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("cap,p", [(1, 0), (1, 1), (2, 1), (5, 2), (5, 3), (6, 3), (11, 5), (12, 5), (19, 4), (20, 5),
                                   (27, 5), (35, 4), (36, 5), (48, 5), (50, 6), (51, 6), (58, 5), (60, 4)])
@pytest.mark.parametrize("deficient", [False, True])
def test_rhosvd_order(tk, cap, p, form, deficient):
    rng = np.random.default_rng(100 * cap + p)
    n = 70
    # full: twice the cap's rank, halving within the cap at most 1e4 deep and
    # halving again behind it; deficient: total rank cap / 2 (rounded up)
    if deficient:
        X = _tensor(rng, n, max(1, (cap + 1) // 2), 0.9)
    else:
        X = _tensor(rng, n, min(cap + p + 3, n), 0.5 if cap <= 12 else 1e-4 ** (1.0 / cap))
        for k in range(cap, X.core.shape[0]):
            X.core[k, k, k] *= 0.5
    Om = [rng.standard_normal((n, cap + p)) for _ in range(3)]
    eps = 1e-10 if form == 0 else 1e-5
    ref, info = O.roundsum([(1.0, X)], Om, O.RoundParams(eps=eps, cap=cap, p=p))
    got, s = tk.rhosvd([(1.0, tk.Tucker.from_numpy(X.core, X.U))],
                       [torch.from_numpy(np.ascontiguousarray(o.T)).cuda() for o in Om], eps, cap, p, form=form)
    core, U = got.to_numpy()
    dist = O.exact_norm([(1.0, O.Tucker(core, U)), (-1.0, ref)]) / O.exact_norm([(1.0, ref)])
    orth = max(np.abs(u.T @ u - np.eye(u.shape[1])).max() for u in U)
    print(f"order {cap + p} form {form} deficient {deficient}: ranks {got.ranks} s {s} dist {dist:.1e} orth {orth:.1e}",
          flush=True)
    assert got.ranks == tuple(info["ranks"])
    assert form == 1 or s == info["s"]
    assert dist <= (1e-10 if form == 0 else 1e-4)
    assert orth <= (1e-12 if form == 0 else 1e-4)
