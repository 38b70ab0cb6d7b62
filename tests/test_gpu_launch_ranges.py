"""A block of outer vectors whose pair items take more than one launch (2^32 threads).

520 occupied orbitals on the 30 grid: 8.5 million items of 512 threads.  The
exchange sum of the block against the sum over its two halves, which are one
launch each: the same FP64 terms in another order.  All terms of the diagonal
pairs are positive and dominate, so 1e-11 relative is 1e5 units in the last
place of a sum of 8.5 million.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_exchange_over_two_launches():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_06797_amd import Context, FP32
    from synthetic.model import orbital_miller
    L, n, ecut, no, nst = 18.0, 30, 7.2, 520, 560
    m = orbital_miller(L, 64, ecut)
    pos = {tuple(v): k for k, v in enumerate(m.tolist())}
    neg = np.array([pos[tuple(v)] for v in (-m).tolist()])
    rng = np.random.default_rng(30)
    a = rng.standard_normal((nst, len(m))) + 1j * rng.standard_normal((nst, len(m)))
    a = a + np.conj(a[:, neg])
    a *= np.exp(-0.5 * (2 * math.pi / L) ** 2 * (m * m).sum(1) / ecut)[None, :]
    q = np.linalg.qr(np.concatenate([a.real, a.imag], axis=1).T)[0].T
    c = q[:, :len(m)] + 1j * q[:, len(m):]
    e = np.concatenate([np.linspace(-1.0, -0.5, no), np.linspace(0.3, 1.0, nst - no)])
    with Context(L, n, ecut, 5.0, m, e, c, no, 1, tau=np.array([1.0]), w=np.array([1.0]),
                 prec=FP32) as ctx:
        gb = ctx.info.g_block
        assert ctx.info.n_grid == 30 and no * (no + 1) // 2 * gb * 512 >= 1 << 32
        half = gb // 2
        for rep in range(2):
            print("[gpu-case] exchange over two launches, call", rep, flush=True)
            whole = ctx.exchange(0, 0, gb)
            parts = ctx.exchange(0, 0, half) + ctx.exchange(0, half, gb - half)
            assert abs(whole - parts) <= 1e-11 * abs(whole)
