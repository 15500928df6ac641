"""The workspace of the exact norm depends on sizes alone: not on which factor
pointers coincide, nor on which ranks reach the capacity (the query may be asked
with placeholder pointers, and a sum that shares factors when it is asked may
have distinct ones later).  The queries need no GPU; the calls with that
workspace do."""
import ctypes as C
import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2608_11091_amd", "libtsgmres.so")


def _query(n, ranks, rcap, factors, nb):
    """tucker_norm_workspace of nb blocks with made-up addresses; factors(b, k)
    numbers the factor of block b in mode k."""
    from paper_2608_11091_amd import _abi
    blocks = []
    for b in range(nb):
        t = _abi.TkTucker()
        t.d, t.core = len(n), 0x10000000 * (b + 1)
        for k in range(len(n)):
            t.n[k], t.r[k], t.rcap[k] = n[k], ranks[b][k], rcap[k]
            t.U[k] = 0x1000 + 0x100000 * factors(b, k)
        blocks.append(t)
    arr, coef = (_abi.TkTucker * nb)(*blocks), (C.c_double * nb)(*[1.0] * nb)
    bs = _abi.TkBlockSum()
    bs.nblocks, bs.coef, bs.blocks = nb, coef, arr
    need = C.c_size_t()
    _abi.check(_abi.load().tucker_norm_workspace(C.byref(bs), C.byref(need)))
    return need.value


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")
@pytest.mark.parametrize("n,r,nb", [((20, 20), 6, 2), ((20, 31, 24), 5, 3), ((65, 65, 65), 12, 2),
                                    ((256, 256, 256), 32, 4), ((24, 24, 24, 24), 4, 3)])
def test_query_depends_on_sizes_alone(n, r, nb):
    d = len(n)
    full = [(r,) * d] * nb
    mixed = [(r,) * d] + [tuple(max(1, r - (b + k) % 3) for k in range(d)) for b in range(1, nb)]
    sizes = {name: _query(n, rk, (r,) * d, f, nb) for name, rk, f in [
        ("distinct", full, lambda b, k: 100 * b + k), ("one address", full, lambda b, k: 0),
        ("shared by mode", full, lambda b, k: k), ("one mode shared", full, lambda b, k: 0 if k == 0 else 100 * b + k),
        ("ranks below the capacity", mixed, lambda b, k: 100 * b + k), ("both", mixed, lambda b, k: k)]}
    assert len(set(sizes.values())) == 1, sizes


@pytest.mark.gpu
@pytest.mark.parametrize("n,r,nb", [((20, 31, 24), 5, 3), ((65, 65, 65), 12, 2), ((130, 130), 17, 4)])
def test_call_with_the_queried_workspace(n, r, nb):
    import torch

    import oracle as O
    import paper_2608_11091_amd as tk
    from paper_2608_11091_amd import _abi, api
    rng = np.random.default_rng(sum(n) + nb)
    d = len(n)
    need = _query(n, [(r,) * d] * nb, (r,) * d, lambda b, k: 0, nb)
    U = [[rng.standard_normal((nk, r)) for nk in n] for _ in range(nb)]
    cores = [rng.standard_normal((r,) * d) for _ in range(nb)]
    for shared in (lambda b, k: b, lambda b, k: 0, lambda b, k: 0 if k != 1 else b):
        fac = [[U[shared(b, k)][k] for k in range(d)] for b in range(nb)]
        dev = {}
        blocks = []
        for b in range(nb):
            us = [dev.setdefault((shared(b, k), k), torch.from_numpy(np.ascontiguousarray(fac[b][k].T)).cuda())
                  for k in range(d)]
            blocks.append((1.0 + b, tk.Tucker(torch.from_numpy(cores[b]).cuda(), us, (r,) * d)))
        bs, keep = api._blocks_struct(blocks)
        ref = O.exact_norm([(1.0 + b, O.Tucker(cores[b], fac[b])) for b in range(nb)])
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        out = C.c_double(0.0)
        lib = _abi.load()
        assert lib.tucker_norm(C.byref(bs), C.byref(out), C.c_void_p(ws.data_ptr()), need - 1, api._stream()) == -4
        rc = lib.tucker_norm(C.byref(bs), C.byref(out), C.c_void_p(ws.data_ptr()), need, api._stream())
        assert rc == 0
        print(f"norm n {n} r {r} blocks {nb}: {out.value / ref - 1.0:.1e}", flush=True)
        assert abs(out.value / ref - 1.0) <= 1e-12
