"""Every sphere inside a grid's orbital window runs in a kernel compiled for the window.

A sphere whose largest index is K can hold a quarter more vectors than the
sphere of radius K; counted for the latter, the shared memory of two instances
(36 grid K = 11 in FP32, 40 grid K = 13 in FP64) left the larger spheres to the
general kernel.  The host library runs against a stand-in for the HIP runtime.
"""
import pytest

from tests import fake_hip

CODE = """
import math
GRIDS = L.supported_grids()
for n in GRIDS:
    kw = (n - 1) // 3
    ko = (n - 1 - kw) // 2
    ka = min(kw, 10)
    side = 0.5 * n
    b = 2 * math.pi / side
    for k in (ko - 1, ko):
        if min(g for g in GRIDS if g >= min(2 * k + ka + 1, n)) != n:
            continue               # a smaller grid holds the cell
        for r2 in (k * k, (k + 1) ** 2 - 1):
            r = np.arange(-k - 1, k + 2)
            m = np.stack([a.ravel() for a in np.meshgrid(r, r, r, indexing="ij")], axis=1)
            m = m[(m * m).sum(1) <= r2].astype(np.int32)
            c = np.zeros((2, len(m)), complex)
            c[0, np.nonzero((m == 0).all(1))[0]] = 1
            c[1, np.nonzero((m == [1, 0, 0]).all(1))[0]] = math.sqrt(0.5)
            c[1, np.nonzero((m == [-1, 0, 0]).all(1))[0]] = math.sqrt(0.5)
            with L.Context(side, n, 0.5 * b * b * (r2 + 0.5), 0.5 * b * b * (ka * ka + 0.25), m,
                           np.array([-0.5, 0.5]), c, 1, 1, tau=np.array([1.0]),
                           w=np.array([1.0]), prec={prec}) as ctx:
                assert ctx.info.n_grid == n and np.abs(m).max() == k
                ctx.exchange(0, 0, 1)
            print(json.dumps([n, k, r2]))
"""


@pytest.mark.parametrize("prec", [0, 1])
def test_window_spheres(tmp_path, prec):
    lines, cases = fake_hip.run(fake_hip.build(tmp_path), tmp_path, CODE.replace("{prec}", str(prec)),
                                timeout=300)
    names = [l[1] for l in lines if l[0] == "launch" and "k_wstates" in l[1]]
    assert len(names) == len(cases) >= 24
    assert [c for c, n in zip(cases, names) if "k_wstates_real" not in n] == []
