"""The in-cutoff neighbour lists against the oracle where they can go wrong:
atom counts around a workgroup's 32 atoms, dense clusters whose lists run to
many rounds, pairs on the cutoffs, and coordinates so far from the origin that
the single-precision cutoff test decides nothing."""
import numpy as np
import pytest

from paper_2606_14073_amd import nepspin, workload as W
from tests.helpers import rel_inf

pytestmark = pytest.mark.gpu

TOL = 1e-12     # FP64 parity, as for every evaluation


def cluster(n, spacing, seed, offset):
    """n atoms of both species (three in ten carry spins) near a cubic grid of that spacing, shifted by offset"""
    rng = np.random.default_rng(seed)
    m = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n].astype(float)
    pos = g * spacing + rng.normal(0.0, 0.05, (n, 3)) + offset
    types = (rng.uniform(size=n) > 0.3).astype(np.int32)
    spin = rng.normal(size=(n, 3))
    spin /= np.linalg.norm(spin, axis=1, keepdims=True)
    spin[types == 1] = 0
    return types, pos, spin


@pytest.mark.parametrize("n,spacing,offset", [
    (1, 2.5, 0.0), (2, 2.5, 0.0), (8, 2.5, 0.0), (31, 2.5, 0.0), (32, 2.5, 1.0e3), (33, 2.5, 0.0), (65, 2.2, 0.0),
    (125, 1.9, 0.0),            # more ranks inside the cutoffs than the lists are put together for
    (343, 2.0, 0.0),            # lists near the longest allowed, several rounds of 64 pairs
    (216, 2.5, 1.0e5),          # single-precision coordinates 0.008 A apart
])
def test_cluster_matches_oracle(oracle, n, spacing, offset):
    t, p, s = cluster(n, spacing, n, offset)
    if n > 8:                   # two pairs on the cutoffs, to rounding
        t[:3] = 0
        s[:3] = (0.0, 0.6, 0.8)
        p[1] = p[0] + (-6.0, 0.0, 0.0)
        p[2] = p[0] + (0.0, -4.5, 0.0)
    par = W.random_params()
    box, pbc = np.full(3, 1.0e6), np.zeros(3, np.int32)
    got = nepspin.Model(par).eval(t, p, s, box, pbc, want=("E", "Ei", "F", "H"))
    ref = oracle.evaluate(t, p, s, box, pbc, par, want=("E", "F", "H", "Ei"))
    for k in ("Ei", "F", "H"):
        assert rel_inf(got[k], ref[k]) <= TOL, k
