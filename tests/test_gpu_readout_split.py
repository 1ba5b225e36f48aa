"""The read-out of small batches, a 16-atom tile over four wavefronts, against
the one that gives each wavefront a tile: a replica alone takes the first,
beside a large one the second, and the state has to be the same to the last bit."""
import numpy as np
import pytest

from paper_2606_14073_amd import nepspin, workload as W

pytestmark = pytest.mark.gpu


def lattice(n_atoms, spins):
    """the first n_atoms of a free crystal"""
    s = W.fege_lattice(5, 5, 5, seed=3, pbc=(0, 0, 0))
    k = slice(0, n_atoms)
    return s.types[k], s.pos[k], s.spin[k] if spins else None, s.box


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("spins", [True, False])
@pytest.mark.parametrize("n_atoms", [1, 15, 16, 31, 33, 130, 1000])
def test_split_readout_same_bits(n_atoms, spins, precision):
    m = nepspin.Model(W.random_params() if spins else W.random_params_structural())
    big = W.fege_lattice(15, 15, 15)
    t, p, s, box = lattice(n_atoms, spins)
    ip = nepspin.integrator_params(dt=1.0, T0=50.0, alpha_s=0.1 if spins else 0.0, gamma_L=0.01, ensemble=1)

    def run(beside):
        sv = nepspin.Server(m, precision=precision, steps_per_batch=2)
        if beside:
            sv.submit(big.types, big.pos, big.spin if spins else None, big.box, big.pbc,
                      colour=big.colour if spins else None, params=ip, n_steps=2)
        k = sv.submit(t, p, s, box, (0, 0, 0), params=ip, n_steps=2)
        sv.drain()
        assert sv.poll(k)["state"] == nepspin.SL_DONE
        out = sv.fetch(k)
        sv.close()
        return out

    for a, b in zip(run(False), run(True)):
        assert np.array_equal(a, b)
