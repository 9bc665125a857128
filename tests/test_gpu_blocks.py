"""Iteration blocks whose length follows the slots' waits for the host: the
same bits as blocks of one length (captured ones), in fewer launches where all
slots wait together."""
import numpy as np
import pytest

import aqs_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("minimizer,replicas,block", [("fire", 1, 32), ("fire", 1, 2), ("fire", 3, 64), ("cg", 1, 32)])
def test_block_lengths_change_no_result(minimizer, replicas, block):
    """A small skin makes the lists short-lived: many waits at few iterations."""
    from paper_2507_20802_amd import Cg, Engine, Fire, Tuning
    starts = [S.jittered_lattice_start(3, 11, 40 + r, 11, jitter=0.1, density=1.2) for r in range(replicas)]
    out = []
    for graph in (0, 1):
        eng = Engine(3, [s.n for s in starts], np.array([s.L for s in starts]), 1e-4, fire=Fire(max_iter=150),
                     tuning=Tuning(skin=0.05, use_graph=graph, block_iters=block))
        if minimizer == "cg":
            eng.set_minimizer("cg", Cg(max_iter=150))
        for r, s in enumerate(starts):
            eng.set_replica(r, s.types, s.pos, 0)
        rec = eng.minimize(list(range(replicas)), n_steps=[1] * replicas)
        out.append((rec, [eng.positions(r) for r in range(replicas)], eng.counters()))
    (ra, xa, ca), (rb, xb, cb) = out
    assert np.array_equal(ra, rb) and all(np.array_equal(x, y) for x, y in zip(xa, xb))
    assert ca["atom_evals"] == cb["atom_evals"]
    if block == 32:
        assert cb["rebuilds"] > 4 and ca["force_launches"] < cb["force_launches"]
