"""Pair instances with the split by cutoff shell, on every compiled grid and kept set.

Two checks per instance.  The bins add up to the unsplit sum: the same FP64
terms in another order (1e-11 relative, a hundred thousand units in the last
place of a sum of a few million terms).  The bins beyond the first few give
the energy of a cell set up with the smaller auxiliary sphere, whose kernels do
not split: the tolerances of the FP64 and FP32 forms against the oracle, 1e-9
and 1e-5 relative.  The second check needs a grid that aliases nothing (else
the smaller sphere may run on a smaller grid, which is another model).
"""
import numpy as np
import pytest

from tests.test_gpu_pair_forms import CASES, _cell

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_grid,L,ecut,eaux,kmax", CASES)
def test_shell_bins(n, n_grid, L, ecut, eaux, kmax):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_06797_amd import Context
    m, e, c = _cell(L, ecut, 5, n)
    kw = dict(tau=np.array([1.3]), w=np.array([1.0]))
    alias_free = 2 * np.abs(m).max() + kmax + 1 <= n
    for prec, tol in ((0, 1e-9), (1, 1e-5)):
        print("[gpu-case] shell bins", n, kmax, "prec", prec, flush=True)
        with Context(L, n, ecut, eaux, m, e, c, 2, 1, prec=prec, n_extrap=4, extrap_alpha=1.2,
                     **kw) as ctx:
            assert ctx.info.n_grid == n_grid and np.abs(ctx.aux_miller()).max() == kmax
            ed, ex = ctx.energy()[:2]
            cut, bd, bx, _ = ctx.extrapolation(4)
        assert abs(bx[0] - ex) <= 1e-11 * abs(ex) and abs(bd[0] - ed) <= 1e-11 * abs(ed)
        if not alias_free:
            continue
        for q in (1, 3):
            with Context(L, n, ecut, cut[q], m, e, c, 2, 1, prec=prec, **kw) as ctx:
                d, x = ctx.energy()[:2]
            assert abs(bx[q] - x) <= tol * abs(x) and abs(bd[q] - d) <= tol * abs(d), (prec, q)
