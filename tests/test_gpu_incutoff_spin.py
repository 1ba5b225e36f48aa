"""The spin couplings of pairs at 4.5 A to the last bit of r^2, where the lists
decide whether a pair has a spin-angular part, against the oracle: the rotation
of a step so short that nothing moves."""
import numpy as np
import pytest

from paper_2606_14073_amd import nepspin, workload as W
from tests.helpers import rel_inf

pytestmark = pytest.mark.gpu

DT = 1e-6     # a first half step of 1e-16 A: below half the spacing of coordinates beyond 8 A


def stars(prec, n=40, seed=9):
    """clusters of six spins 60 A apart: a centre, two neighbours inside rc_A, three at 4.5 A with r^2 within two
    spacings of 20.25 (in single precision for fp32)"""
    rng = np.random.default_rng(seed)
    f = np.float64 if prec == "fp64" else np.float32
    ulp = np.spacing(f(20.25))
    pos = []
    for k in range(n):
        c = 64.0 + 64.0 * np.array([k % 4, k // 4 % 4, k // 16])
        star = [c]
        while len(star) < 6:
            u = rng.normal(size=3)
            u /= np.linalg.norm(u)
            p = c + u * (rng.uniform(2.4, 3.2) if len(star) < 3 else 4.5)
            d = (p - c).astype(f)
            if len(star) >= 3 and abs((d * d).sum() - f(20.25)) > 2 * ulp:
                continue
            if min(np.linalg.norm(p - q) for q in star) > 1.8:
                star.append(p)
        pos += star
    pos = np.array(pos)
    spin = rng.normal(size=pos.shape)
    spin /= np.linalg.norm(spin, axis=1, keepdims=True)
    return pos, spin, np.tile(np.arange(6, dtype=np.int32), n)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_couplings_of_pairs_on_the_angular_cutoff(oracle, prec):
    pos, spin, col = stars(prec)
    t = np.zeros(len(pos), np.int32)
    box, pbc = np.full(3, 1.0e6), np.zeros(3, np.int32)
    par = W.random_params()
    sim = nepspin.Sim(nepspin.Model(par), t, pos, spin, box, pbc, colour=col, precision=prec,
                      params=nepspin.integrator_params(dt=DT, alpha_s=0.1))
    sim.integrate(1)
    p1, _, s1, _ = sim.state()
    sim.close()
    assert np.array_equal(p1, pos)
    rs = oracle.run(t, pos, np.zeros_like(pos), spin, box, pbc, par, col, oracle.step_params(dt=DT, alpha=0.1), 1)[2]
    # spins round at 1e-16, the rotations are some 1e-7; FP32 fields carry 1e-5
    assert rel_inf(s1 - spin, rs - spin) <= (1e-7 if prec == "fp64" else 1e-4)
