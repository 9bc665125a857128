"""The linear-response start with lists so short-lived that every solve needs
new ones first: the chain of a wide skin, also with every launch timed, in one
workgroup (2D) and on tiles, alone and in a live round."""
import numpy as np
import pytest

import oracle as O
from gpu_common import E_REL_TOL, POS_TOL, fire_pair, load_glass

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,dg,nst", [("glass2d_256", 1e-4, 4), ("glass3d_1500", 2e-5, 2)])
@pytest.mark.parametrize("profiled", [0, 1])
def test_thin_skin_keeps_the_chain(name, dg, nst, profiled):
    from paper_2507_20802_amd import AQS_START_LINEAR, Engine, Tuning
    pos, types, L, dim = load_glass(name)
    fire, _ = fire_pair()
    out = []
    for skin in (0.3, 2 * dg):   # the strain of a step alone (2.5 dg) outlives 2 dg
        eng = Engine(dim, [len(types)] * 2, L, dg, fire=fire, tuning=Tuning(skin=skin))
        for r in (0, 1):
            eng.set_replica(r, types, pos, 0)
        eng.counters(reset=True)
        eng.set_profiling(profiled)
        rec = eng.minimize([0, 1], n_steps=[nst, nst], start=AQS_START_LINEAR)
        assert (rec["status"] == 0).all()
        out.append((rec, [eng.positions(r) for r in (0, 1)], eng.box(0), eng.counters()))
    (ra, xa, H, ca), (rb, xb, _, cb) = out
    assert cb["rebuilds"] >= ca["rebuilds"] + nst
    assert np.abs(ra["energy"] / rb["energy"] - 1.0).max() <= E_REL_TOL
    assert np.array_equal(ra["start"], rb["start"])
    for r in (0, 1):
        assert O.compare(xa[r], xb[r], H)[0] <= POS_TOL


def test_live_round_of_thin_skins():
    """A live round whose chains rebuild before their solves, on both streams."""
    from paper_2507_20802_amd import AQS_START_LINEAR, Engine, Tuning, parallel
    pos, types, L, dim = load_glass("glass2d_256")
    fire, _ = fire_pair()
    ends = []
    for skin, live in ((0.3, False), (2e-4, True)):
        eng = Engine(dim, [len(types)] * parallel.slots_needed(1, 3), L, 1e-4, fire=fire, tuning=Tuning(skin=skin))
        g = parallel.layout(1, 3)[0]
        eng.set_replica(g.star, types, pos, 0)
        parallel.run(eng, [g], 12, 4, 3, start=AQS_START_LINEAR, live=live)
        ends.append((eng.strain_index(g.star), eng.positions(g.star), eng.box(g.star)))
    assert ends[0][0] == ends[1][0]
    assert O.compare(ends[0][1], ends[1][1], ends[0][2])[0] <= POS_TOL
