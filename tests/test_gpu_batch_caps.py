"""Cells of a batch under workspace caps (the C interface's per-cell cap): values of
the uncapped cells, and every cell's own memory within its cap.
"""
import numpy as np
import pytest

from tests.test_gpu_pair_forms import _cell
from tests.test_gpu_workspace_edges import TAU, W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_values_and_memory(prec, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_06797_amd import Batch, ltmp2
    cap = 5 << 20

    class Capped(ltmp2.Params):    # the bindings of a batch leave a cell's cap at 0
        def __init__(self, *a):
            super().__init__(*((a[:10] + (cap,)) if len(a) == 11 else a))

    cells = []
    for seed, ecut in ((3, 2.5), (4, 4.5)):
        m, e, c = _cell(9.3, ecut, 5, seed)
        cells.append(dict(L=9.3, n_fft=15, ecut=ecut, eaux=4.0, miller=m, eps=e, coeff=c,
                          n_occ=2, n_tau=2, tau=TAU, w=W))
    print("[gpu-case] capped batch", prec, flush=True)
    with Batch(cells, prec=prec) as b:
        ref = b.energy()
    monkeypatch.setattr(ltmp2, "Params", Capped)
    with Batch(cells, prec=prec) as b:
        assert all(b.cell_info(k).device_bytes <= cap for k in range(2))
        for _ in range(3):
            assert np.array_equal(np.array(b.energy()), np.array(ref))
