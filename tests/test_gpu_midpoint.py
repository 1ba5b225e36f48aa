"""The midpoint solve against the oracle where its start can differ: caps below
and above the ones its single-precision start needs, rotations from far below
single precision's resolution of the spin to beyond a radian, both signs of the
step and lane layouts of one, two and four quads per spin."""
import numpy as np
import pytest

from paper_2606_14073_amd import nepspin, workload as W
from tests.helpers import rel_inf

pytestmark = pytest.mark.gpu

TOL = 1e-12     # parity of every FP64 step


@pytest.mark.parametrize("cap,B,alpha,dt", [(4, 1.0, 0.1, 1.0), (5, 1.0, 0.1, 1.0), (50, 1.0, 0.1, -1.0), (50, 0.0, 0.0, 1e-6),
                                            (50, 2000.0, 0.5, 1.0), (12, 20000.0, 0.3, 1.0), (50, 20000.0, 0.3, -1.0)])
def test_midpoint_start_matches_oracle(oracle, cap, B, alpha, dt):
    s = W.fege_lattice(4, 4, 4)
    p = W.random_params()
    kw = dict(dt=dt, B0=(0.1 * B, 0.0, B), K_corr=1)
    sim = nepspin.Sim(nepspin.Model(p), s.types, s.pos, s.spin, s.box, s.pbc, colour=s.colour,
                      params=nepspin.integrator_params(alpha_s=alpha, mid_cap=cap, **kw))
    ob = sim.integrate(1)
    pos, vel, spin, _ = sim.state()
    sim.close()
    rp, rv, rs, _, _ = oracle.run(s.types, s.pos, np.zeros_like(s.pos), s.spin, s.box, s.pbc, p, s.colour,
                                  oracle.step_params(alpha=alpha, mid_cap=400, **kw), 1)
    assert ob[0, 11] == 0               # no rotation stopped at the cap
    assert rel_inf(spin, rs) <= TOL
    assert rel_inf(vel, rv) <= TOL


@pytest.mark.parametrize("cells", [(42, 42, 42), (64, 64, 64)])
def test_midpoint_same_bits_in_every_lane_layout(cells):
    """a 4^3 replica (16 lanes per spin) beside a crystal swept with 8 or 4"""
    p = nepspin.Model(W.random_params(), short_range=W.SHORT_RANGE_FEGE)
    small, big = W.fege_lattice(4, 4, 4), W.fege_lattice(*cells, seed=3)
    ip = nepspin.integrator_params(dt=1.0, T0=300.0, alpha_s=0.1, gamma_L=0.01, ensemble=1, B0=(0, 0, 1.0))

    def run(systems):
        sv = nepspin.Server(p, precision="fp32", steps_per_batch=2)
        ids = [sv.submit(s.types, s.pos, s.spin, s.box, s.pbc, colour=s.colour, params=ip, n_steps=2) for s in systems]
        sv.drain()
        out = sv.fetch(ids[-1])
        sv.close()
        return out

    for a, b in zip(run([small])[:3], run([big, small])[:3]):
        assert np.array_equal(a, b)
