"""Positions given in any periodic image: half the atoms shifted by whole boxes, many
of their pairs on the cutoffs, against the same configuration inside the box and
the oracle. Coordinates are multiples of 2^-30 A and the box edges short binary
fractions, so the shifts and every minimum-image displacement are exact: the
shifted configuration has the same bits as the wrapped one."""
import numpy as np
import pytest

from paper_2606_14073_amd import nepspin, workload as W
from tests.helpers import min_image_delta, rel_inf

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-4}     # parity with the oracle, as for every evaluation


def grid(x):
    return np.rint(x * 2.0 ** 30) * 2.0 ** -30


def on_the_cutoffs(pos, box, rng, most=120):
    """pairs moved to 4.5 and 6 A up to +-1e-6 ... 1e-3 A, each atom in one pair at most; wrapped, on the grid"""
    pos, used = pos.copy(), set()
    for i in rng.permutation(len(pos)):
        d = min_image_delta(pos, pos[i], box, (1, 1, 1))
        r = np.sqrt((d * d).sum(1))
        rc = 4.5 if rng.uniform() < 0.5 else 6.0
        near = [j for j in np.nonzero(abs(r - rc) < 0.15)[0] if j not in used and j != i]
        if i in used or not near:
            continue
        j = near[0]
        off = 10.0 ** rng.uniform(-6.0, -3.0) * rng.choice([-1.0, 1.0])
        pos[j] = pos[i] + d[j] * ((rc + off) / r[j])
        used |= {i, j}
        if len(used) >= 2 * most:
            break
    return grid(np.mod(grid(pos), box))


def shifted(pos, box, boxes, rng):
    """every other atom up to that many boxes away on each axis, the rest where they were"""
    return pos + box * rng.integers(-boxes, boxes + 1, size=pos.shape) * (rng.uniform(size=(len(pos), 1)) < 0.5)


def crystal(seed=11):
    s = W.fege_lattice(4, 4, 4, seed=seed)
    box = np.array([18.8125, 19.0, 18.75])
    rng = np.random.default_rng(seed)
    return s.types, on_the_cutoffs(s.pos / s.box * box, box, rng), s.spin, box


def water(seed=12):
    s = W.water_box(5, seed=seed)
    box = np.full(3, 15.5)
    rng = np.random.default_rng(seed)
    return s.types, on_the_cutoffs(s.pos / s.box * box, box, rng, most=60), s.spin, box


@pytest.mark.parametrize("boxes", [1, 5, 50, 1000])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["crystal", "water"])
def test_shifted_evaluation(oracle, name, prec, boxes):
    t, p, s, box = crystal() if name == "crystal" else water()
    par = W.random_params() if name == "crystal" else W.random_params_structural()
    spin = s if name == "crystal" else None
    pbc = np.ones(3, np.int32)
    far = shifted(p, box, boxes, np.random.default_rng(boxes))
    want = ("E", "Ei", "F", "H")
    model = nepspin.Model(par)
    wrapped = model.eval(t, p, spin, box, pbc, precision=prec, want=want)
    ref = oracle.evaluate(t, p, spin, box, pbc, par, want=("E", "F", "H", "Ei"))
    # another configuration of the same sizes in between: the work arrays hold its records
    ot, op, osp, obox = crystal(31) if name == "crystal" else water(32)
    model.eval(ot, op, osp if name == "crystal" else None, obox, pbc, precision=prec, want=want)
    got = model.eval(t, far, spin, box, pbc, precision=prec, want=want)
    for k in ("Ei", "F", "H"):
        assert np.array_equal(got[k], wrapped[k]), k
        assert rel_inf(got[k], ref[k]) <= TOL[prec], k
    q = [model.descriptors(t, x, spin, box, pbc, precision=prec) for x in (p, far)]
    assert np.array_equal(q[0][0], q[1][0]) and np.array_equal(q[0][1], q[1][1])


@pytest.mark.parametrize("boxes", [10 ** 6, 10 ** 7, 10 ** 9])
def test_pairs_stay_mutual_far_out(boxes):
    """so far out that coordinates round at up to 4e-6 A: each pair is still in both atoms' lists or in neither, so
    that the forces add up to zero, to the rounding of 512 sums of some 100 terms"""
    t, p, s, box = crystal()
    far = shifted(p, box, boxes, np.random.default_rng(3))
    F = nepspin.Model(W.random_params()).eval(t, far, s, box, np.ones(3, np.int32), want=("F",))["F"]
    assert np.abs(F.sum(0)).max() <= 512 * 100 * 2.0 ** -53 * np.abs(F).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_shifted_start_of_dynamics(prec):
    """the initial forces of a simulation and of a server's replica enter its first kick. Coordinates 50 boxes out
    round at 1.1e-13 A in the first drift and forces change by some 10 of their scale per A: 1e-11, in FP32-mixed
    1e-6 (a displacement that rounds the other way)"""
    t, p, s, box = crystal()
    pbc = np.ones(3, np.int32)
    far = shifted(p, box, 50, np.random.default_rng(5))
    model = nepspin.Model(W.random_params())
    col = W.colour_greedy(t, p, box, pbc, 7.0)
    ip = nepspin.integrator_params(dt=1e-3, alpha_s=0.1, B0=(0, 0, 1.0))
    out = []
    for x in (p, far):
        sim = nepspin.Sim(model, t, x, s, box, pbc, colour=col, params=ip, precision=prec)
        sim.integrate(1)
        out.append(sim.state()[1:3])
        sim.close()
        sv = nepspin.Server(model, precision=prec, steps_per_batch=1)
        k = sv.submit(t, x, s, box, pbc, colour=col, params=ip, n_steps=1)
        sv.drain()
        out.append(sv.fetch(k)[1:3])
        sv.close()
    for vel, spin in out[1:]:
        assert rel_inf(vel, out[0][0]) <= (1e-9 if prec == "fp64" else 1e-5)
        assert rel_inf(spin, out[0][1]) <= (1e-9 if prec == "fp64" else 1e-5)
