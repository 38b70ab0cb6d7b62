"""When an energy may use its second stream.

The direct terms run on a stream of the library's own beside the caller's.
That stream has the default priority and all compute units; a caller whose
stream has another priority or a set of compute units of its own keeps
everything on it (streams of different priorities waiting for each other are a
hazard of their own, so this is checked against a stand-in for the HIP runtime
only).
"""
import pytest

from tests import fake_hip

CODE = """
def cell():
    m = np.array([[0, 0, 0], [1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1]],
                 np.int32)
    c = np.zeros((3, 7), complex)
    c[0, 0] = 1
    c[1, 1:3] = np.sqrt(0.5)
    c[2, 3:5] = np.sqrt(0.5)
    return m, np.array([-0.5, 0.3, 0.4]), c
m, e, c = cell()
main = {main}
for extra in ({{}}, dict(second_spin=(e, c, 1))):
    with L.Context(8.0, 12, 0.5, 1.0, m, e, c, 1, 2, tau=np.array([0.5, 1.5]),
                   w=np.array([1.0, 1.0]), stream=main, **extra) as ctx:
        ctx.energy()
d = dict(L=8.0, n_fft=12, ecut=0.5, eaux=1.0, miller=m, eps=e, coeff=c, n_occ=1, n_tau=2,
         tau=np.array([0.5, 1.5]), w=np.array([1.0, 1.0]))
with L.Batch([d, d], stream=main) as b:
    b.energy()
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    d = tmp_path_factory.mktemp("fakehip")
    return fake_hip.build(d), d


def _streams(fake, main, **env):
    lines, _ = fake_hip.run(*fake, CODE.format(main=main), **env)
    return {l[-1] for l in lines if l[0] == "launch" and "k_real_forward" in l[1]
            and "Lb0E" in l[1]}, lines


def test_ordinary_streams_have_a_second_one(fake):
    for main in (0, 0x5000):
        direct, _ = _streams(fake, main)
        assert len(direct) == 3 and "%#x" % main not in direct and "(nil)" not in direct


@pytest.mark.parametrize("env", [dict(FAKE_HIP_PRIORITY="-1"), dict(FAKE_HIP_PRIORITY="1"),
                                 dict(FAKE_HIP_CU_MASK="0xff")])
def test_special_streams_keep_everything(fake, env):
    direct, lines = _streams(fake, 0x5000, **env)
    assert direct == {"0x5000"}
    if "FAKE_HIP_PRIORITY" in env:
        assert ["stream", "nonblocking"] not in lines
