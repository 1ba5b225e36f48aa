"""The sweep of a small replica in one workgroup against the launches per colour
class: a replica alone takes the first, beside a larger one the second, and the
state has to be the same to the last bit."""
import numpy as np
import pytest

from paper_2606_14073_amd import nepspin, workload as W

pytestmark = pytest.mark.gpu

LANDAU = (-0.02, 0.01)


def lattice(cells, **kw):
    return W.fege_lattice(*cells, seed=5, **kw)


def system(name):
    """a request (types, pos, spin, box, pbc, colour, params)"""
    ip = dict(dt=1.0, T0=200.0, alpha_s=0.1, gamma_L=0.01, ensemble=1, B0=(0, 0, 0.5), seed=77)
    if name == "one spin":
        s = lattice((2, 2, 2), pbc=(0, 0, 0))
        t = np.ones_like(s.types)
        t[5] = 0
        spin = np.zeros_like(s.spin)
        spin[5] = (0.6, 0.0, 0.8)
        return t, s.pos, spin, s.box, (0, 0, 0), None, ip
    if name == "no spin":
        s = lattice((2, 2, 2), pbc=(0, 0, 0))
        return np.ones_like(s.types), s.pos, np.zeros_like(s.spin), s.box, (0, 0, 0), None, ip
    if name == "many couplings":      # more than 32 of them, classes of two or three spins
        s = lattice((4, 4, 4))
        rng = np.random.default_rng(9)
        t = (rng.uniform(size=len(s.types)) > 0.68).astype(np.int32)
        spin = rng.normal(size=s.pos.shape)
        spin /= np.linalg.norm(spin, axis=1, keepdims=True)
        spin[t == 1] = 0
        return t, s.pos, spin, s.box, (1, 1, 1), None, dict(ip, skin=0.1)
    cells, over = {"tiny": ((3, 3, 3), {}), "odd free": ((5, 3, 4), {}), "fp64 most": ((5, 5, 9), {}),
                   "fp32 most": ((6, 6, 9), {}), "capped": ((4, 4, 4), dict(mid_cap=3)),
                   "self-consistent": ((4, 4, 4), dict(sc_tol=1e-9)),
                   "lengths": ((4, 4, 4), dict(alpha_s=0.0, longitudinal=1, gamma_lsf=0.05))}[name]
    pbc = (1, 0, 1) if name == "odd free" else (1, 1, 1)
    s = lattice(cells, pbc=pbc)
    spin = s.spin * np.linspace(0.8, 1.2, len(s.spin))[:, None] if name == "lengths" else s.spin
    return s.types, s.pos, spin, s.box, pbc, None, dict(ip, **over)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["one spin", "no spin", "tiny", "odd free", "fp64 most", "fp32 most", "many couplings",
                                  "capped", "self-consistent", "lengths"])
def test_one_workgroup_equals_class_launches(name, precision):
    m = nepspin.Model(W.random_params(), short_range=W.SHORT_RANGE_FEGE, landau=LANDAU)
    big = lattice((8, 8, 8))
    t, p, s, box, pbc, col, ip = system(name)

    def run(beside):
        sv = nepspin.Server(m, precision=precision, steps_per_batch=3)
        if beside:
            sv.submit(big.types, big.pos, big.spin, big.box, big.pbc, colour=big.colour, n_steps=3,
                      params=nepspin.integrator_params(dt=1.0, B0=(0, 0, 0.5)))
        k = sv.submit(t, p, s, box, pbc, colour=col, params=nepspin.integrator_params(**ip), n_steps=3)
        sv.drain()
        assert sv.poll(k)["state"] == nepspin.SL_DONE
        out = sv.fetch(k)
        sv.close()
        return out

    for a, b in zip(run(False), run(True)):
        assert np.array_equal(a, b)
