"""Pair transforms of every compiled grid and kept-set instance against the oracle.

One case per grid and instance (the alias-free window, one below it, and a
kept set beyond it, where the caller's grid aliases as part of the model),
one and several slabs per field, ragged rounds of a workgroup, a diagonal and
an off-diagonal pair.  Two occupied and three virtual orbitals with random
real-orbital coefficients keep the oracle cheap at every grid size.

Tolerance: relative to B = sum_G' v(G') sum_ij sum_G v(G) |A_ij(G)| |A_ji(G)|,
the sum of the magnitudes of the terms.  Each A is a few hundred roundings
deep at most (three transforms of length <= 40 and one product per point,
whose errors add like a random walk): 64 units in the last place of the
compute type, FP64 and FP32; the split-BF16 product carries 2^-16 per term.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# caller grid, its transform grid, side, E_cut, E_aux, largest auxiliary index
CASES = [
    (12, 12, 8.0, 6.0, 4.0, 3), (12, 12, 8.0, 6.0, 2.4, 2), (12, 12, 8.0, 6.0, 7.8, 5),
    (15, 15, 9.3, 7.5, 5.0, 4), (15, 15, 9.3, 7.5, 3.4, 3), (15, 15, 9.3, 7.5, 11.5, 7),
    (16, 16, 9.6, 7.0, 6.4, 5), (18, 18, 11.0, 7.5, 5.0, 5), (18, 18, 11.0, 7.5, 10.6, 8),
    (20, 20, 12.2, 7.0, 5.2, 6), (24, 24, 14.1, 7.5, 5.0, 7), (24, 24, 14.1, 7.5, 4.0, 6),
    (25, 25, 14.8, 7.2, 6.1, 8), (27, 27, 16.0, 7.5, 5.0, 8), (27, 27, 16.0, 7.5, 4.2, 7),
    (30, 30, 18.0, 7.2, 5.0, 9), (32, 32, 19.0, 7.6, 5.5, 10), (36, 36, 20.0, 7.6, 5.0, 10),
    (40, 40, 23.0, 7.5, 3.77, 10), (40, 40, 23.0, 7.5, 3.2, 9),
]


def _cell(L, ecut, n_states, seed):
    from synthetic.model import orbital_miller
    m = orbital_miller(L, 64, ecut)
    rng = np.random.default_rng(seed)
    pos = {tuple(v): k for k, v in enumerate(m.tolist())}
    neg = np.array([pos[tuple(v)] for v in (-m).tolist()])
    a = rng.standard_normal((n_states, len(m))) + 1j * rng.standard_normal((n_states, len(m)))
    a = a + np.conj(a[:, neg])                       # c(-G) = conj c(G): real orbitals
    a *= np.exp(-0.5 * (2 * math.pi / L) ** 2 * (m * m).sum(1) / ecut)[None, :]
    r = np.concatenate([a.real, a.imag], axis=1)     # real inner products
    q = np.linalg.qr(r.T)[0].T
    c = q[:, :len(m)] + 1j * q[:, len(m):]
    return m, np.array([-0.4, -0.3, 0.1, 0.25, 0.5])[:n_states], c


@pytest.mark.parametrize("n,n_grid,L,ecut,eaux,kmax", CASES)
def test_pair_forms_vs_oracle(n, n_grid, L, ecut, eaux, kmax):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle.mp2 import Problem
    from paper_1611_06797_amd import Context
    m, e, c = _cell(L, ecut, 5, n)
    P = Problem(L, n, eaux, m, e, c, 2)
    tau, w = np.array([1.3]), np.array([1.0])
    first, count = 1, 3
    ref = bound = 0.0
    for prec, u in ((0, 2.0 ** -53), (1, 2.0 ** -24), (2, 2.0 ** -18)):
        print("[gpu-case] pair forms", n, kmax, "prec", prec, flush=True)
        with Context(L, n, ecut, eaux, m, e, c, 2, 1, tau=tau, w=w, prec=prec) as ctx:
            aux = ctx.aux_miller()
            assert ctx.info.n_grid == n_grid and np.abs(aux).max() == kmax
            x = ctx.exchange(0, first, count)
        if prec == 0:
            index = {tuple(v): k for k, v in enumerate(P.aux.tolist())}
            for g in range(first, first + count):
                k = index[tuple(aux[g].tolist())]
                A = P.fock_overlaps(tau[0], k)
                AA = A * np.conj(np.transpose(A, (1, 0, 2))) * P.v[None, None, :]
                ref += 2.0 * P.v[k] * AA.sum().real
                bound += 2.0 * P.v[k] * np.abs(AA).sum()
        assert abs(x - ref) <= 64 * u * bound, (prec, x, ref, bound)
