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


def _counts(x, types, H, dim, skin):
    """Neighbours of each atom by their type, within rc_ab + skin (all image pairs)."""
    rc = POT.rc_factor * np.array(POT.sigma) + skin
    img = np.array([(i, j, k) for i in (-1, 0, 1) for j in (-1, 0, 1)
                    for k in ((-1, 0, 1) if dim == 3 else (0,))], dtype=float)[:, :dim]
    out = np.zeros((len(x), 2), dtype=int)
    for sh in img @ np.asarray(H)[:dim, :dim].T:
        d = np.linalg.norm(x[None] + sh - x[:, None], axis=2)
        near = (d > 0) & (d < rc[types[:, None], types[None]])
        for b in (0, 1):
            out[:, b] += (near & (types[None] == b)).sum(1)
    return out


def _fits(counts, cap):
    """(fits as words, fits as whole groups of four)"""
    groups = -(-counts // 4)
    return bool(counts.sum(1).max() <= cap), bool(groups.sum(1).max() <= cap // 4)


def test_stress_with_lists_that_fit_only_as_words():
    """A skin at which some atom's neighbours fit in the capacity one by one,
    but its A and B neighbours, padded to whole groups of four, do not:
    iterations and evaluations refuse the configuration, the stress has it."""
    from paper_2507_20802_amd import Engine, Fire, LJParams, Tuning
    from paper_2507_20802_amd._lib import AQSError
    dim, dg, k, cap = 2, 1e-2, 7, 32
    s = S.jittered_lattice_start(dim, 20, 31, 20, jitter=0.2, density=1.2)
    x = O.affine(s.pos, k * dg)
    H = O.strain_box(dim, s.L, k, dg)
    # the builder's distances may pass pairs up to 1e-3 beyond the skin
    skin = next(v for v in np.arange(0.02, 0.6, 0.004)
                if all(_fits(_counts(x, s.types, H, dim, w), cap) == (True, False) for w in (v, v + 2e-3)))
    eng = Engine(dim, [s.n], s.L, dg, pot=LJParams(), fire=Fire(),
                 tuning=Tuning(max_neighbors=cap, skin=float(skin)))
    eng.set_replica(0, s.types, x, k)
    with pytest.raises(AQSError):
        eng.energy_forces(0)
    Eo, _, So, _ = O.energy_forces(x, s.types, H, POT)
    sig, E2 = eng.stress(0)
    assert abs(E2 - Eo) <= 1e-12 * abs(Eo)
    assert np.allclose(sig, So, rtol=1e-10, atol=1e-12 * max(1.0, np.abs(So).max()))
