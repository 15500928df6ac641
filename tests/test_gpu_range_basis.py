"""Shifted Cholesky-QR of the range sketches at the edges of its kernels: row
counts around the 32 rows of a workgroup, widths around the 16, 32 and 48
columns of the column groups and the panels of the factorisation, equal and
unequal mode sizes, full and deficient rank (dead columns).  The factors of a
RoundSum are the basis times an orthogonal matrix: orthonormal to 1e-13 in FP64
(working accuracy times the width), 1e-5 in the FP32 form."""
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


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("ns,cap,p,rank", [((4, 3, 5), 2, 1, 2), ((15,) * 3, 7, 8, 7), ((16,) * 3, 12, 4, 4),
                                           ((17, 31, 32), 14, 2, 14), ((33,) * 3, 16, 1, 9), ((31, 32, 33), 24, 7, 24),
                                           ((64,) * 3, 30, 2, 30), ((65, 64, 63), 31, 2, 12), ((48, 49, 96), 40, 8, 33),
                                           ((97,) * 3, 45, 4, 45), ((129, 70, 64), 56, 8, 20), ((66,) * 3, 48, 16, 48),
                                           ((9, 33, 17, 20), 8, 1, 8), ((40,) * 4, 17, 4, 6)])
def test_orthonormal_factors(tk, ns, cap, p, rank, form):
    rng = np.random.default_rng(sum(ns) + cap + rank)
    x = O.Tucker(rng.standard_normal((rank,) * len(ns)),
                 [np.linalg.qr(rng.standard_normal((n, rank)))[0] for n in ns])
    om = [_cm(rng.standard_normal((n, cap + p))) for n in ns]
    eps = 1e-5 if form else 1e-12
    # tau below the certificate's reach keeps the full width cap + p
    w, s = tk.rhosvd([(1.0, tk.Tucker.from_numpy(x.core, x.U))], om, eps, cap, p, force_s=cap + p, form=form)
    got = O.Tucker(*w.to_numpy())
    err = O.exact_norm([(1.0, got), (-1.0, x)]) / O.exact_norm([(1.0, x)])
    dev = max(np.abs(u.T @ u - np.eye(u.shape[1])).max() for u in got.U)
    print(f"basis {ns} s {s} rank {rank} form {form}: ranks {w.ranks} orth {dev:.1e} err {err:.1e}", flush=True)
    assert s == cap + p
    assert dev <= (1e-5 if form else 1e-13)
    assert err <= (5e-5 if form else 1e-11)
