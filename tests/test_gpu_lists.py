"""Neighbour lists at the limits of the list builder: energies, forces and
stress of one configuration against the oracle's all-pairs sum, for tiles
that touch both x faces (three cells per edge), tiles whose masks come in
several batches, tiles with a compact halo beyond the LDS capacity, cells
with more candidates than the builder numbers, and rows of mostly empty
cells."""
import numpy as np
import pytest

import aqs_synth as S
import oracle as O

pytestmark = pytest.mark.gpu
POT = O.kob_andersen()

CASES = [
    # dim, lattice side, density, lanes per atom, list capacity
    (3, 10, 1.2, 2, 0),      # three cells per edge: a tile's row has both wrapped cells
    (3, 11, 1.2, 1, 0),      # ... and its masks come in batches
    (3, 11, 1.2, 8, 0),
    (3, 14, 1.6, 2, 256),    # compact halo beyond the LDS capacity: word lists
    (3, 14, 3.2, 2, 512),    # more candidates per cell than are numbered
    (2, 20, 1.2, 2, 0),
    (2, 51, 1.2, 1, 96),
    (2, 90, 0.1, 2, 0),      # rows of more cells than a tile may span, most of them empty
]


@pytest.mark.parametrize("dim,m,density,tpa,max_nb", CASES)
def test_lists_against_all_pairs(dim, m, density, tpa, max_nb):
    from paper_2507_20802_amd import Engine, Fire, LJParams, Tuning
    s = S.jittered_lattice_start(dim, m, 31, m, jitter=0.2, density=density)
    dg, k = 1e-2, 7
    x = O.affine(s.pos, k * dg)
    eng = Engine(dim, [s.n], s.L, dg, pot=LJParams(), fire=Fire(),
                 tuning=Tuning(threads_per_atom=tpa, max_neighbors=max_nb))
    eng.set_replica(0, s.types, x, k)
    H = O.strain_box(dim, s.L, k, dg)
    Eo, Fo, So, _ = O.energy_forces(x, s.types, H, POT)
    E, F = eng.energy_forces(0)
    assert abs(E - Eo) <= 1e-12 * abs(Eo)
    assert np.abs(F - Fo).max() <= 1e-11 * max(1.0, np.abs(Fo).max())
    sig, E2 = eng.stress(0)
    assert abs(E2 - Eo) <= 1e-12 * abs(Eo)
    assert np.allclose(sig, So, rtol=1e-10, atol=1e-12 * max(1.0, np.abs(So).max()))
