"""Launches of the small slots' kernel are counted and timed apart from the
force kernel's, and the benchmark runs at a size where there are no others."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

import aqs_synth as S
from gpu_common import fire_pair, load_glass

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COUNTERS = {"force_ms": 0.0, "force_timed": 0, "update_ms": 0.0, "update_timed": 0, "timed_atom_evals": 0,
            "small_ms": 6.0, "small_timed": 3, "small_launches": 9, "small_timed_atom_evals": 3000}


def test_benchmark_names_the_kernel_that_was_timed():
    sys.path.insert(0, ROOT)
    import bench
    t = bench.launch_times(COUNTERS, 2)
    assert t == {"kernel": "k_small", "avg_launch_ms": 2.0, "timed_launches": 3, "atoms_per_launch": 1000.0,
                 "update_avg_ms": None}
    both = dict(COUNTERS, force_ms=1.0, force_timed=4, timed_atom_evals=400, update_ms=2.0, update_timed=4)
    t = bench.launch_times(both, 3)
    assert t == {"kernel": "k_force<3>", "avg_launch_ms": 0.25, "timed_launches": 4, "atoms_per_launch": 100.0,
                 "update_avg_ms": 0.5}


@pytest.mark.gpu
def test_small_launches_are_not_force_launches():
    """A small slot alone: no force launches, all evaluations timed with the
    small ones; with a slot of tiles beside it, both kinds apart."""
    from paper_2507_20802_amd import Engine
    pos, types, L, dim = load_glass("glass2d_256")
    fire, _ = fire_pair(max_iter=100)
    s = S.uniform_glass_start(2, 1400, 77, 6)
    eng = Engine(dim, [256, 1400], np.array([[L] * 2, [s.L] * 2]), 1e-4, fire=fire)
    eng.set_replica(0, types, pos + 0.01 * S.rng_for(5).normal(size=pos.shape), 0)
    eng.set_replica(1, s.types, s.pos, 0)
    eng.set_profiling(1)
    eng.counters(reset=True)
    eng.minimize([0])
    c = eng.counters(reset=True)
    assert c["force_launches"] == c["force_timed"] == c["update_timed"] == c["timed_atom_evals"] == 0
    assert c["small_launches"] == c["small_timed"] >= 1 and c["small_ms"] > 0.0
    assert c["small_timed_atom_evals"] == c["atom_evals"] > 0
    eng.minimize([0, 1])
    c = eng.counters(reset=True)
    assert c["force_timed"] == c["update_timed"] == c["force_launches"] > 0
    assert c["timed_atom_evals"] % 1400 == 0 and c["small_timed_atom_evals"] % 256 == 0
    assert c["timed_atom_evals"] + c["small_timed_atom_evals"] == c["atom_evals"]
    assert eng.counters()["small_launches"] == 0


@pytest.mark.gpu
def test_benchmark_at_a_small_2d_size():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--dim", "2", "--n", "256", "--P", "2", "--K", "3",
                        "--dgamma", "1e-4", "--steps", "1", "--warmup", "0", "--only-plain", "--plain-rounds", "0",
                        "--sequential", "0", "--no-cpu-baseline", "--forms", "kernel", "--kernel-K", "2",
                        "--profile-every", "1"], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr
    res = json.loads(r.stdout.strip().splitlines()[-1])
    k = res["force_kernel_all_chains"]
    assert k["kernel"] == "k_small" and k["update_avg_ms"] is None and k["avg_launch_ms"] > 0.0
    assert res["roofline"]["kernel"] == "k_small"
