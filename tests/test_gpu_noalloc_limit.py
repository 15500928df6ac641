"""Allocation-free sketches just inside the 64 MiB scratch: inputs, their copies
in the capacity layout and the two contractions' results alone take 62 to 64
MiB, so that the buffers of products split over the chip would not fit beside
them.  The call is planned without those and gives the sketch of the workspace
entry point (the same contractions, summed in another order: 1e-12)."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,r,nb,s", [((238, 205, 423), 85, 6, 83), ((423, 419, 479), 88, 4, 134),
                                      ((221, 228, 394), 54, 8, 237), ((81, 121, 478, 206), 13, 17, 193)])
def test_near_the_limit(n, r, nb, s):
    import paper_2608_11091_amd as tk
    rng = np.random.default_rng(sum(n))
    blocks = [(float(rng.uniform(-2, 2)), O.Tucker(rng.standard_normal((r,) * len(n)),
                                                   [rng.standard_normal((nk, r)) for nk in n])) for _ in range(nb)]
    S = [rng.standard_normal((nk, s)) for nk in n]
    gb = [(c, tk.Tucker.from_numpy(X.core, X.U)) for c, X in blocks]
    St = [torch.from_numpy(np.ascontiguousarray(m.T)).cuda() for m in S]
    ref = tk.sketch(gb, St).cpu().numpy()
    want = O.sketch_krp(blocks, S)
    out = torch.full((s,), float("nan"), dtype=torch.float64, device="cuda")
    got = tk.sketch_noalloc(gb, St, out).cpu().numpy()
    dist = [float(np.linalg.norm(got - x) / np.linalg.norm(x)) for x in (ref, want)]
    print(f"noalloc n {n} r {r} blocks {nb} s {s}: {dist}", flush=True)
    assert max(dist) <= 1e-12
