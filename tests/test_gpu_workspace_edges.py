"""Cells at the edge of a workspace cap: few states and small orbital spheres.

Under a cap the occupied orbitals in the pair transforms' order share memory
that is there anyway (the coefficients', or the chi scratch); the values are
those of the uncapped context, bit for bit, for one and two spin channels, and
in a batch.
"""
import numpy as np
import pytest

from tests.test_gpu_pair_forms import _cell

pytestmark = pytest.mark.gpu

TAU, W = np.array([0.4, 1.9]), np.array([0.5, 0.8])


def _smallest_cap(make):
    lo, hi = 1 << 10, 1 << 31
    from paper_1611_06797_amd import ltmp2
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            make(mid).close()
            hi = mid
        except ltmp2.LTMP2Error as e:
            assert "cap" in str(e), e
            lo = mid
    return hi


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("ecut,second", [(2.5, False), (2.5, True), (7.5, False)])
def test_values_at_the_smallest_cap(prec, ecut, second):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_06797_amd import Context
    m, e, c = _cell(9.3, ecut, 5, 3)
    kw = {}
    if second:
        kw["second_spin"] = (e, _cell(9.3, ecut, 5, 4)[2], 1)

    def make(cap):
        return Context(9.3, 15, ecut, 4.0, m, e, c, 2, 2, tau=TAU, w=W, prec=prec,
                       workspace_cap=cap, **kw)

    print("[gpu-case] workspace cap", prec, ecut, second, flush=True)
    with make(0) as ctx:
        ref = ctx.energy()[2]
        hart = None if second else ctx.direct_hartree(1)
    with make(_smallest_cap(make)) as ctx:
        for _ in range(3):
            got = ctx.energy()[2]
            assert np.allclose(got, ref, rtol=1e-13, atol=0)
            assert ctx.chi(1) == got[1, 0]
            assert ctx.exchange(0) == got[0, 1]
            if hart is not None:
                assert abs(ctx.direct_hartree(1) - hart) <= 1e-12 * abs(hart)


def test_capped_cells_in_a_batch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_06797_amd import Batch, Context
    m, e, c = _cell(9.3, 2.5, 5, 3)
    with Context(9.3, 15, 2.5, 4.0, m, e, c, 2, 2, tau=TAU, w=W, prec=0) as ctx:
        ed, ex, _, _ = ctx.energy()
    cell = dict(L=9.3, n_fft=15, ecut=2.5, eaux=4.0, miller=m, eps=e, coeff=c, n_occ=2, n_tau=2,
                tau=TAU, w=W, workspace_cap=1 << 26)
    with Batch([cell, dict(cell)], prec=0) as b:
        for k in range(3):
            print("[gpu-case] capped cells in a batch, call", k, flush=True)
            d, x = b.energy()
            assert np.allclose(d, ed, rtol=1e-13, atol=0) and np.allclose(x, ex, rtol=1e-13, atol=0)
