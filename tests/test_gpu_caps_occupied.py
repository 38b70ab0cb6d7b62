"""The smallest workspace cap of a cell with more occupied states than auxiliary
vectors: its occupied orbitals in the pair transforms' order need the chi
scratch, chi(r, G') is smaller.  Values of the uncapped context, bit for bit.
"""
import numpy as np
import pytest

from tests.test_gpu_pair_forms import _cell
from tests.test_gpu_workspace_edges import TAU, W, _smallest_cap

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("second", [False, True])
def test_more_occupied_states_than_vectors(prec, second):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_06797_amd import Context
    m, _, c = _cell(9.3, 2.5, 5, 3)
    # 14 orthonormal real orbitals: cosine and sine waves of the sphere
    half = [k for k, v in enumerate(m.tolist()) if v > [0, 0, 0]][:7]
    at = {tuple(v): k for k, v in enumerate(m.tolist())}
    c = np.zeros((14, len(m)), complex)
    for s, k in enumerate(half):
        neg = at[tuple((-m[k]).tolist())]
        c[2 * s, [k, neg]] = np.sqrt(0.5)
        c[2 * s + 1, [k, neg]] = np.sqrt(0.5) * np.array([1j, -1j])
    q = np.linalg.qr(np.random.default_rng(2).standard_normal((14, 14)))[0]
    c = q @ c
    e = np.concatenate([np.linspace(-0.6, -0.3, 9), np.linspace(0.2, 0.9, 5)])
    kw = {"second_spin": (e, q.T @ c, 8)} if second else {}

    def make(cap):
        return Context(9.3, 15, 2.5, 0.3, m, e, c, 9, 2, tau=TAU, w=W, prec=prec,
                       workspace_cap=cap, **kw)

    print("[gpu-case] capped occupied states", prec, second, flush=True)
    with make(0) as ctx:
        assert 2 * ctx.info.n_h < 9
        ref = ctx.energy()[2]
        hart = None if second else ctx.direct_hartree(1)
    with make(_smallest_cap(make)) as ctx:
        for _ in range(3):
            got = ctx.energy()[2]
            assert np.allclose(got, ref, rtol=1e-13, atol=0)
            assert ctx.chi(1) == got[1, 0] and ctx.exchange(0) == got[0, 1]
            if hart is not None:
                assert abs(ctx.direct_hartree(1) - hart) <= 1e-12 * abs(hart)
