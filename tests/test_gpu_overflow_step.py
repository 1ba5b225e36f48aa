"""A replica whose spin lists overflow inside a step, beyond the slots that the
spin-angular parts of the couplings have: that replica fails, and a replica in
the same batch keeps the bits that it has alone."""
import numpy as np
import pytest

from paper_2606_14073_amd import nepspin, workload as W

pytestmark = pytest.mark.gpu

N, A0, A1 = 7, 3.0, 2.0     # spins per edge; spacing at the start and after the first half step


def collapsing(dt=1.0):
    """a free cubic grid of spins shrinking so fast that the list rebuilt in the first step has 80 spin neighbours
    within rc_A + skin (capacity 64, of any species 96) and 146 within rc_R + skin (160)"""
    g = np.stack(np.meshgrid(*[np.arange(N)] * 3, indexing="ij"), -1).reshape(-1, 3) - (N - 1) / 2
    for a in (A0, A1):
        r = np.linalg.norm(g * a, axis=1)
        assert ((r > 0) & (r < 5.0)).sum() == (18 if a == A0 else 80)
        assert ((r > 0) & (r < 6.5)).sum() == (32 if a == A0 else 146)
    n = len(g)
    spin = np.tile([0.0, 0.6, 0.8], (n, 1))
    vel = g * (A1 - A0) / (0.5 * dt)
    return (np.zeros(n, np.int32), g * A0, spin, np.zeros(3), np.zeros(3, np.int32)), vel, np.arange(n, dtype=np.int32)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_overflow_inside_a_step_stays_in_its_replica(prec):
    model = nepspin.Model(W.random_params(), short_range=W.SHORT_RANGE_FEGE)
    s = W.fege_lattice(4, 4, 4)
    ip = nepspin.integrator_params(dt=1.0, T0=300.0, alpha_s=0.1, gamma_L=0.01, ensemble=1, B0=(0, 0, 1.0))

    def run(with_other):
        sv = nepspin.Server(model, precision=prec, steps_per_batch=3)
        ids = []
        if with_other:
            sys, vel, col = collapsing()
            ids.append(sv.submit(*sys, vel=vel, colour=col, params=nepspin.integrator_params(dt=1.0), n_steps=3))
        ids.append(sv.submit(s.types, s.pos, s.spin, s.box, s.pbc, colour=s.colour, params=ip, n_steps=3))
        sv.drain()
        if with_other:
            with pytest.raises(nepspin.NepError) as e:
                sv.fetch(ids[0])
            assert e.value.code == nepspin.SL_E_OVERFLOW
        out = sv.fetch(ids[-1])
        sv.close()
        return out

    for a, b in zip(run(False), run(True)):
        assert np.array_equal(a, b)


def test_overflow_inside_a_step_is_reported():
    sys, vel, col = collapsing()
    sim = nepspin.Sim(nepspin.Model(W.random_params()), *sys, vel=vel, colour=col,
                      params=nepspin.integrator_params(dt=1.0))
    with pytest.raises(nepspin.NepError) as e:
        sim.integrate(1)
    assert e.value.code == nepspin.SL_E_OVERFLOW
    sim.close()
