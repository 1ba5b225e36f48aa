"""Kernel timing of small systems, whose groups share launches when they are not
timed: each timed group is its own work, and timing changes no bit."""
import numpy as np
import pytest

from paper_2606_14073_amd import nepspin, workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,prec", [("crystal", "fp64"), ("crystal", "fp32"), ("water", "fp64")])
def test_groups_of_small_systems_are_timed_apart(kind, prec):
    if kind == "crystal":
        s, model, mass = W.fege_lattice(16, 16, 16), nepspin.Model(W.random_params()), (0.0, 0.0)
    else:
        s, model, mass = W.water_box(20), nepspin.Model(W.random_params_structural()), tuple(W.MASS_WATER)

    def run(groups):
        sim = nepspin.Sim(model, s.types, s.pos, s.spin if kind == "crystal" else None, s.box, s.pbc, colour=s.colour,
                          precision=prec, params=nepspin.integrator_params(dt=0.5, alpha_s=0.1, mass=mass))
        sim.integrate(1)            # first launches load code
        sim.profile(groups)
        obs = sim.integrate(3)
        t = sim.profile_read()
        sim.profile(())
        out = (obs,) + sim.state()[:3]
        sim.close()
        return out, t

    plain, _ = run(())
    timed, t = run(nepspin.PROFILE_GROUPS)
    for a, b in zip(plain, timed):
        assert np.array_equal(a, b)
    ms = {k: v[0] for k, v in t.items()}
    print(ms, flush=True)
    # the radial sets and the second species are between a quarter and all of the work they were launched with
    assert ms["desc_radial"] > 0.1 * ms["desc_angular"]
    assert ms["bwd_radial"] > 0.1 * ms["bwd_angular"]
    assert ms["bwd_angular_1"] > 0.1 * ms["bwd_angular"]
