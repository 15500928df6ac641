"""Effective-rank rule on Grams whose first Householder vector lies in rows 64
and beyond, which other waves clear than the one that writes it: the first row
of every factor meets the others only there.  A vector that lost those entries
gives another spectrum; the width must be the oracle's on every repetition."""
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


@pytest.mark.parametrize("form,tau", [(0, None), (0, 1e-3), (1, 1e-3)])
@pytest.mark.parametrize("n,r", [(66, 34), (100, 51), (128, 43), (160, 54)])
def test_far_rows(tk, n, r, form, tau):
    rng = np.random.default_rng(n)
    dim, cap, p, nb = r - 5, r, 4, 3 if 2 * r <= n else 2  # nb r > n: n-side Gram
    B = []
    for _ in range(3):
        b = np.zeros((n, dim))
        b[1:, 1:] = np.linalg.qr(rng.standard_normal((n - 1, dim - 1)))[0]
        b[0, 0] = 1.0
        b[64:, 0] = rng.uniform(0.5, 1.5, n - 64)
        B.append(b)
    blocks = []
    for _ in range(nb):
        U = [np.concatenate([b[:, :1], b[:, 1:] @ rng.standard_normal((dim - 1, r - 1))], axis=1) for b in B]
        blocks.append((float(rng.uniform(0.5, 1.5)), O.Tucker(rng.standard_normal((r,) * 3), U)))
    Om = [rng.standard_normal((n, cap + p)) for _ in range(3)]
    _, info = O.roundsum(blocks, Om, O.RoundParams(eps=1e-5, cap=cap, p=p, tau=tau))
    gb = [(c, tk.Tucker.from_numpy(X.core, X.U)) for c, X in blocks]
    go = [torch.from_numpy(np.ascontiguousarray(o.T)).cuda() for o in Om]
    got = [tk.rhosvd(gb, go, 1e-5, cap, p, tau=-1.0 if tau is None else tau, form=form)[1] for _ in range(20)]
    print(f"n {n} r {r} form {form} tau {tau}: oracle r~ {info['rtilde']} s {info['s']}, gpu {set(got)}", flush=True)
    assert max(info["rtilde"]) <= dim < cap + p
    assert set(got) == {info["s"]}
