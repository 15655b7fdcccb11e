"""The pairs' order by counting (more than 2048 sorted pairs, up to 2^27
comparisons in a launch) and by the bitonic network beyond that, against the
oracle's pattern and rank order (exact): the first sizes past a tile, every
pair sorted, equal spectra (no inclusion), 3D, and a batch with one M per map."""
import numpy as np
import pytest

import synth
from oracle import pattern

pytestmark = pytest.mark.gpu


def _fibres(n):
    return synth.rsa_fibres(n, n, n / 32, n / 16, seed=300 + n, target_vf=0.35).g


@pytest.mark.parametrize("make,Ms", [
    (lambda: _fibres(256), [4096, 4100, 9001, 20000]),
    (lambda: _fibres(128), [9000]),
    (lambda: np.zeros((128, 96), np.uint8), [5000]),
    (lambda: synth.rsa_spheres(32, 32, 32, r_lo=4.0, r_hi=6.0, seed=5, target_vf=0.2).g, [4500, 16001]),
], ids=["256", "128_all", "zeros", "32cubed"])
def test_rank_order_exact(make, Ms):
    import paper_2103_10203_amd as mor
    g = make()
    checked = 0
    for M, plan in zip(Ms, mor.make_plans([g] * len(Ms), Ms)):
        ref = pattern.build_pattern(g, M)
        if ref.unstable:
            continue
        for p in (plan, mor.Plan(g, M)):
            s, r = p.pattern()
            assert p.info["M_actual"] == ref.M_actual
            assert np.array_equal(s, ref.sorted_idx) and np.array_equal(r, ref.rank_idx)
        checked += 1
    assert checked >= 1
