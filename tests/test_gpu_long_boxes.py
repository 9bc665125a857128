"""Boxes far longer than a list distance: pairs of atoms near the far end of a
2D box of 9 10^6 sigma (single precision resolves 1 sigma there) relax to the
potential's minimum, side by side or spread over the box."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spread", [0, 1])
def test_pairs_at_the_far_end_of_a_long_box(spread):
    """Four pairs, 2.2 sigma apart, every pair out of the others' reach.  A force
    below 1e-5 leaves a pair within 1e-5 / 57 (its stiffness) of 2^(1/6), the
    coordinates are multiples of 1.9e-9: 1e-6 for the distance, and far less than
    1e-9 for the energy."""
    from paper_2507_20802_amd import Engine, Fire
    L = np.array([9.0e6, 9.0])
    x = np.array([8.9e6 - (2.0e6 * k if spread else 8.0 * k) + 0.4 for k in range(4)])
    pos = np.stack([np.stack([x, np.full(4, 4.0)], 1), np.stack([x + 2.2, np.full(4, 4.0)], 1)], 1).reshape(8, 2)
    eng = Engine(2, [8], L[None], 1e-4, fire=Fire(ftol=1e-5))
    eng.set_replica(0, np.zeros(8, np.uint8), pos, 0)
    rec = eng.minimize([0])[0, 0]
    p = eng.positions(0).reshape(4, 2, 2)
    d = p[:, 1] - p[:, 0]
    d -= L * np.rint(d / L)
    rc = 2.5
    assert rec["status"] == 0
    assert np.abs(np.hypot(d[:, 0], d[:, 1]) - 2.0 ** (1.0 / 6.0)).max() <= 1e-6
    assert abs(rec["energy"] - 4.0 * (-1.0 - 4.0 * (rc ** -12 - rc ** -6))) <= 1e-9
