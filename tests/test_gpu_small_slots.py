"""Whole iterations of small 2D slots in one workgroup (k_small): the lanes per
atom and the two workgroup sizes at their limits against the oracle's
minimisation, list rebuilds inside the kernel, a slot beside larger ones, and
a launch's length not mattering."""
import numpy as np
import pytest

import aqs_synth as S
import oracle as O
from gpu_common import E_REL_TOL, POS_TOL, fire_pair

pytestmark = pytest.mark.gpu
POT = O.kob_andersen()


def quenched(n, seed):
    from paper_2507_20802_amd import Engine
    s = S.uniform_glass_start(2, n, 77, seed)
    fire, ofire = fire_pair()
    eng = Engine(2, [n], s.L, 1e-4, fire=fire)
    eng.set_replica(0, s.types, s.pos, 0)
    assert eng.minimize([0])[0, 0]["status"] == 0
    return s, eng.positions(0), fire, ofire


# lanes per atom 8, 4, 2, 1 of 512 threads, then one of 1024; one size past it (tiles)
@pytest.mark.parametrize("n", [120, 128, 129, 256, 257, 511, 512, 513, 1023, 1024, 1025])
def test_one_step_against_the_oracle(n):
    from paper_2507_20802_amd import Engine
    s, x0, fire, ofire = quenched(n, n)
    dg = 1e-4
    eng = Engine(2, [n], s.L, dg, fire=fire)
    eng.set_replica(0, s.types, x0, 0)
    rec = eng.minimize([0], n_steps=[1])[0]
    H = O.strain_box(2, s.L, 1, dg)
    ref = O.fire(O.affine(x0, dg), s.types, H, POT, ofire)
    assert rec[1]["status"] == 0 and ref.status == O.CONVERGED
    assert abs(rec[1]["energy"] - ref.E) <= E_REL_TOL * abs(ref.E)
    assert O.compare(eng.positions(0), ref.pos, H)[0] <= POS_TOL


@pytest.mark.parametrize("n,start", [(256, 0), (700, 0), (256, 3)])
def test_rebuilds_in_the_kernel_keep_the_chain(n, start):
    """A thin skin makes the kernel rebuild its lists many times (in place; start
    3 extrapolates): the chain's energies and its end are those of a wide skin."""
    from paper_2507_20802_amd import Engine, Tuning
    s, x0, fire, _ = quenched(n, n)
    out = []
    for skin in (0.3, 0.004):
        eng = Engine(2, [n], s.L, 1e-4, fire=fire, tuning=Tuning(skin=skin))
        eng.set_replica(0, s.types, x0, 0)
        eng.counters(reset=True)
        rec = eng.minimize([0], n_steps=[8], start=start)[0]
        assert (rec["status"] == 0).all()
        out.append((rec["energy"], eng.positions(0), eng.box(0), eng.counters()["rebuilds"]))
    assert out[1][3] > out[0][3] + 2
    assert np.abs(out[0][0] / out[1][0] - 1.0).max() <= E_REL_TOL
    assert O.compare(out[0][1], out[1][1], out[0][2])[0] <= POS_TOL


@pytest.mark.parametrize("minimizer", ["fire", "cg"])
def test_beside_tiles_and_in_launches_of_any_length(minimizer):
    """Bitwise the same alone, beside a slot of the tiles and one of the other
    workgroup size, and with short launches."""
    from paper_2507_20802_amd import Cg, Engine, Tuning
    sizes = (256, 1400, 700)
    glasses = [quenched(n, n) for n in sizes]
    fire = glasses[0][2]

    def run(which, block):
        eng = Engine(2, [sizes[w] for w in which], np.array([[glasses[w][0].L] * 2 for w in which]), 1e-4, fire=fire,
                     tuning=Tuning(block_iters=block))
        if minimizer == "cg":
            eng.set_minimizer("cg", Cg())
        for r, w in enumerate(which):
            eng.set_replica(r, glasses[w][0].types, glasses[w][1], 0)
        rec = eng.minimize(list(range(len(which))), n_steps=[2] * len(which))
        return {w: (rec[r], eng.positions(r)) for r, w in enumerate(which)}

    alone = {**run([0], 32), **run([1], 32), **run([2], 32)}
    for got in (run([0, 1, 2], 32), run([2, 0], 2)):
        for w, (rec, x) in got.items():
            assert np.array_equal(rec, alone[w][0]) and np.array_equal(x, alone[w][1])
