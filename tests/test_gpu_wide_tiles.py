"""Force tiles over many cells of a row (short cutoffs, tiles filled to the limit,
dilute slots): the list builder gives them an LDS halo like any other unless
the cells are nearly empty, and their energies, forces and stress are the oracle's
all-pairs sums."""
import numpy as np
import pytest

import aqs_synth as S
import oracle as O

pytestmark = pytest.mark.gpu

CASES = [
    # box, density, cutoff (sigma), lanes per atom, tile fill, cells per tile; an LDS halo
    ((300.0, 12.0), 1.2, 2.0 ** (1.0 / 6.0), 1, 2.0, 105, True),
    ((590.0, 145.0), 0.3, 2.5, 2, 2.0, 105, True),
    ((590.0, 145.0), 0.2, 2.5, 1, 2.0, 210, False),         # fewer than two atoms per cell: searched in FP64
    ((285.0, 285.0), 0.1, 2.5, 2, 0.0, 101, False),
    ((640.0, 640.0), 0.02, 2.5, 2, 0.0, 228, False),
    ((2000.0, 450.0), 0.001, 2.5, 2, 0.0, 714, False),
    ((310.0, 9.0, 9.0), 0.3, 2.5, 1, 2.0, 55, False),       # groups because of the chunks; halo too large
    ((600.0, 9.0, 9.0), 0.02, 2.5, 2, 0.0, 214, False),
]


def halos(eng, n):
    """The tiles' halo sizes (-1: none), found in the workspace as the headers
    (first atom, end, 0, halo) that chain from atom 0 to n (without empty tiles
    before the first atom)."""
    w = eng.workspace.cpu().numpy()
    w = w[(-eng.workspace.data_ptr()) % 16:]
    v = w[:w.size // 16 * 16].view(np.int32).reshape(-1, 4)
    first = (v[:-1, 0] == 0) & (v[:-1, 1] > 0) & (v[:-1, 2] == 0) & (v[1:, 0] == v[:-1, 1]) & (v[1:, 2] == 0)
    for i in np.flatnonzero(first):
        j = i
        while j + 1 < len(v) and v[j, 1] < n and v[j + 1, 0] == v[j, 1] and v[j + 1, 1] >= v[j, 1] and v[j + 1, 2] == 0:
            j += 1
        if v[j, 1] == n and v[i:j + 1, 3].min() >= -1:
            return v[i:j + 1, 3]
    raise AssertionError("no tile headers found")


def jittered(box, density, seed):
    """Atoms on a grid of about that density, each moved by up to a tenth of the
    spacing; below 0.5 half of them on the grid, each with a partner 1 to 2 sigma away."""
    box, pairs = np.array(box), density < 0.5
    a = (density / (2 if pairs else 1)) ** (-1.0 / len(box))
    grid = np.maximum(1, np.floor(box / a)).astype(int)
    x = np.stack(np.meshgrid(*[np.arange(g) for g in grid], indexing="ij"), -1).reshape(-1, len(box))
    rng = S.rng_for(2507, 31, seed)
    x = (x + 0.5 + 0.1 * rng.uniform(-1, 1, x.shape)) * (box / grid)
    if pairs:
        d = rng.normal(size=x.shape)
        x = np.concatenate([x, x + d / np.linalg.norm(d, axis=1, keepdims=True) * rng.uniform(1, 2, (len(x), 1))])
    return x, (rng.uniform(size=len(x)) < 0.2).astype(np.uint8)


@pytest.mark.parametrize("box,density,rc,tpa,fill,cells,lds", CASES)
def test_wide_tiles(box, density, rc, tpa, fill, cells, lds):
    from paper_2507_20802_amd import Engine, Fire, LJParams, Tuning
    dim = len(box)
    x0, types = jittered(box, density, cells)
    n = len(x0)
    dg, k = 1e-3, 7
    x = O.affine(x0, k * dg)
    eng = Engine(dim, [n], np.array([box]), dg, pot=LJParams(rc_factor=rc), fire=Fire(),
                 tuning=Tuning(threads_per_atom=tpa, tile_fill=fill))
    eng.set_replica(0, types, x, k)
    H = eng.box(0)
    E, F = eng.energy_forces(0)
    h = halos(eng, n)
    rows = int(np.prod([L // (rc + 0.3) for L in box[1:]]))
    per_row = int(np.ceil(n / rows / ((fill or 0.9) * 256 / tpa)))
    print(f"{n} atoms, {per_row} tiles a row, halo {h.min()} .. {h.max()}")
    assert box[0] // (rc + 0.3) / per_row >= cells - 1
    if lds:
        assert h.min() >= 0
    Eo, Fo, So, _ = O.energy_forces(x, types, H, O.Potential(rc_factor=rc))
    scale = max(1.0, np.abs(Fo).max())
    assert abs(E - Eo) <= 1e-12 * max(1.0, np.abs(Eo))
    assert np.abs(F - Fo).max() <= 1e-11 * scale
    sig, E2 = eng.stress(0)
    assert abs(E2 - Eo) <= 1e-12 * max(1.0, np.abs(Eo))
    assert np.allclose(sig, So, rtol=1e-10, atol=1e-12 * scale)


def test_crowded_cell():
    """Several hundred atoms in one cell of an otherwise empty box, loaded in
    another order than their ids' after a first evaluation."""
    from paper_2507_20802_amd import Engine, Fire, LJParams, Tuning
    rng = S.rng_for(2507, 31, 400)
    g = np.stack(np.meshgrid(np.arange(20), np.arange(20), indexing="ij"), -1).reshape(-1, 2)
    x = rng.permutation(14.2 + 0.12 * (g + 0.1 * rng.uniform(-1, 1, g.shape)))
    types = (rng.uniform(size=400) < 0.2).astype(np.uint8)
    eng = Engine(2, [400], 30.0, 1e-4, pot=LJParams(), fire=Fire(), tuning=Tuning(max_neighbors=512))
    for y in (x, x[::-1].copy()):
        eng.set_replica(0, types, y, 0)
        E, F = eng.energy_forces(0)
        Eo, Fo, _, _ = O.energy_forces(y, types, O.strain_box(2, 30.0, 0, 1e-4), O.kob_andersen())
        assert abs(E - Eo) <= 1e-12 * abs(Eo) and np.abs(F - Fo).max() <= 1e-11 * np.abs(Fo).max()
