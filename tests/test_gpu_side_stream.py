"""Energies whose direct terms run on a second stream beside the exchange terms.

The same kernels run in either order, so the values per Laplace point are the
ones that chi and exchange give one at a time, bit for bit: on the null stream,
on a stream of the caller's, with stage timing (one stream), with other calls on
the same buffers in between, from several threads, and for two spin channels.
"""
import threading

import numpy as np
import pytest

from tests.test_gpu_pair_forms import _cell

pytestmark = pytest.mark.gpu

TAU, W = np.array([0.2, 0.9, 2.5]), np.array([0.3, 0.5, 0.7])


def _context(n, L, ecut, eaux, prec, stream=None, second=False):
    from paper_1611_06797_amd import Context
    m, e, c = _cell(L, ecut, 5, n)
    kw = {}
    if second:
        _, _, cb = _cell(L, ecut, 5, n + 1)
        kw["second_spin"] = (e, cb, 1)
    return Context(L, n, ecut, eaux, m, e, c, 2, 3, tau=TAU, w=W, prec=prec, stream=stream, **kw)


def _single(ctx):
    return np.array([[ctx.chi(t), ctx.exchange(t)] for t in range(len(TAU))])


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("second", [False, True])
def test_energy_equals_single_terms(prec, second):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    own = torch.cuda.Stream()
    for stream in (0, own.cuda_stream):
        print("[gpu-case] side stream", prec, second, stream != 0, flush=True)
        with _context(12, 8.0, 6.0, 4.0, prec, stream, second) as ctx:
            ref = _single(ctx)
            for _ in range(5):
                ed, ex, pt, _q = ctx.energy()
                assert np.array_equal(pt, ref)
                assert ctx.chi(1) == ref[1, 0]      # rewrites chi's buffers
                assert ctx.exchange(2) == ref[2, 1]
            ctx.set_timing(True)
            assert np.array_equal(ctx.energy()[2], ref)
            ctx.set_timing(False)
            assert np.array_equal(ctx.energy()[2], ref)


def test_energies_from_several_threads():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[gpu-case] side stream, threads", flush=True)
    ctxs = [_context(n, L, ec, ea, 1) for n, L, ec, ea in
            ((12, 8.0, 6.0, 4.0), (15, 9.3, 7.5, 5.0), (18, 11.0, 7.5, 5.0))]
    refs = [_single(c) for c in ctxs]
    bad = []

    def work(c, r):
        for _ in range(10):
            if not np.array_equal(c.energy()[2], r):
                bad.append(1)

    th = [threading.Thread(target=work, args=a) for a in zip(ctxs, refs)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for c in ctxs:
        c.close()
    assert not bad


def test_batch_graph_equals_contexts():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_06797_amd import Batch
    spec = ((12, 8.0, 6.0, 4.0), (15, 9.3, 7.5, 5.0), (15, 9.3, 7.5, 3.4), (18, 11.0, 7.5, 5.0))
    cells, ref = [], []
    for n, L, ec, ea in spec:
        m, e, c = _cell(L, ec, 5, n)
        cells.append(dict(L=L, n_fft=n, ecut=ec, eaux=ea, miller=m, eps=e, coeff=c, n_occ=2,
                          n_tau=3, tau=TAU, w=W))
        with _context(n, L, ec, ea, 1) as ctx:
            ref.append(ctx.energy()[:2])
    ref = np.array(ref).T
    with Batch(cells, prec=1) as b:
        for k in range(5):  # eager, then replays of the captured graph
            print("[gpu-case] batch with direct terms beside, call", k, flush=True)
            ed, ex = b.energy()
            assert np.allclose(ed, ref[0], rtol=1e-14, atol=0)
            assert np.allclose(ex, ref[1], rtol=1e-14, atol=0)
            torch.cuda.synchronize()
