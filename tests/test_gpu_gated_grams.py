"""Wide sums (concatenation above n > 160): the R-side Gram of a mode is formed
only while its active ranks fit order 160, the others' blocks are left out of
the same launch.  Modes of both kinds in one sum, in every combination; widths
and ranks equal the oracle's, the sum to its tolerance."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("wide", [(0, 0, 0), (1, 0, 0), (0, 1, 1), (1, 1, 1)])
@pytest.mark.parametrize("form,tau", [(0, None), (0, 1e-3), (1, 1e-3)])
def test_modes_with_and_without(wide, form, tau):
    import paper_2608_11091_amd as tk
    rng = np.random.default_rng(4 * wide[0] + 2 * wide[1] + wide[2])
    n, r, nb, dim, cap, p = 176, 24, 8, 14, 24, 4          # nb r = 192 > n
    ranks = [tuple(r if wd or b == 0 else 16 for wd in wide) for b in range(nb)]  # 192 or 136 in all
    B = [np.linalg.qr(rng.standard_normal((n, dim)))[0] for _ in range(3)]
    blocks = [(float(rng.uniform(0.5, 1.5)), O.Tucker(rng.standard_normal(rk), [
        b @ rng.standard_normal((dim, k)) for b, k in zip(B, rk)])) for rk in ranks]
    Om = [rng.standard_normal((n, cap + p)) for _ in range(3)]
    eps = 1e-10 if form == 0 else 1e-4
    ref, info = O.roundsum(blocks, Om, O.RoundParams(eps=eps, cap=cap, p=p, tau=tau))
    got, s = tk.rhosvd([(c, tk.Tucker.from_numpy(X.core, X.U, rcap=(r,) * 3)) for c, X in blocks],
                       [torch.from_numpy(np.ascontiguousarray(o.T)).cuda() for o in Om], eps, cap, p,
                       tau=-1.0 if tau is None else tau, form=form)
    dist = O.exact_norm([(1.0, O.Tucker(*got.to_numpy())), (-1.0, ref)]) / O.exact_norm([(1.0, ref)])
    print(f"wide {wide} form {form} tau {tau}: oracle s {info['s']}, gpu s {s} ranks {got.ranks} dist {dist:.1e}",
          flush=True)
    assert max(info["rtilde"]) <= dim
    assert s == info["s"] and got.ranks == tuple(info["ranks"])
    assert dist <= 2 * eps
