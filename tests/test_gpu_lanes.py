"""Grids of one call that run side by side on streams of their own: the same
bits as one call per grid, on the default and on another stream, call after
call, with more grids than streams, in 3D, FP64 and load paths."""
import math

import numpy as np
import pytest

import synth
from gpu_common import native_phases

pytestmark = pytest.mark.gpu

GRIDS2 = [(48, 64), (64, 48), (96, 72), (32, 36), (128, 64), (54, 54)]
GRIDS3 = [(24, 32, 36), (32, 24, 24), (16, 24, 32)]


def _plans(mor, shapes):
    gs = [synth.rsa_fibres(*s, 3.0, 5.0, seed=i, target_vf=0.3).g if len(s) == 2 else
          synth.rsa_spheres(*s, 3.0, 5.0, seed=i, target_vf=0.2).g for i, s in enumerate(shapes)]
    return mor.make_plans(gs, [int(math.ceil(0.06 * g.size)) for g in gs])


@pytest.mark.parametrize("shapes,prec,other_stream", [(GRIDS2, 0, False), (GRIDS2[:3], 0, True), (GRIDS2[:2], 2, False),
                                                       (GRIDS3, 0, True)])
def test_grids_side_by_side_equal_one_by_one(shapes, prec, other_stream):
    import paper_2103_10203_amd as mor
    import torch
    plans = _plans(mor, shapes)
    K, B = len(shapes), 3 * len(shapes)
    po = np.arange(B) % K
    eb = synth.macro_strains(B, 3 if len(shapes[0]) == 2 else 6, 4e-3, seed=3)
    kw = {"want_fields": True, "precision": prec, "stream": torch.cuda.Stream() if other_stream else None}
    want = [mor.solve_multi(plans, po[k::K], eb[k::K], native_phases(), 1e-6, **kw) for k in range(K)]
    for _ in range(3):
        got = mor.solve_multi(plans, po, eb, native_phases(), 1e-6, **kw)
        at = 0
        for b in range(B):
            k, i = b % K, b // K
            assert got.iterations[b] == want[k].iterations[i]
            assert got.residual[b] == want[k].residual[i]
            assert np.array_equal(got.eff_stress[b], want[k].eff_stress[i])
            n = want[k].strain.numel() // 3
            assert bool((got.strain[at:at + n] == want[k].strain[i * n:(i + 1) * n]).all())
            at += n


@pytest.mark.parametrize("n,B", [(128, 256), (64, 1030)])
def test_pairs_equal_one_run(n, B):
    """Batches that iterate as pairs of runs against one run (limit off): the
    same bits; just at the rule's line and beyond it, fields included."""
    import paper_2103_10203_amd as mor
    g = synth.rsa_fibres(n, n, n / 32, n / 16, seed=n, target_vf=0.35).g
    plan = mor.Plan(g, int(math.ceil(0.05 * g.size)))
    eb = synth.macro_strains(B, 3, 5e-3, seed=8)
    pairs = mor.solve(plan, eb, native_phases(), 1e-6, want_fields=True)
    keep = mor.tune_subbatch(nbytes=0)
    try:
        one = mor.solve(plan, eb, native_phases(), 1e-6, want_fields=True)
    finally:
        mor.tune_subbatch(*keep)
    assert np.array_equal(pairs.iterations, one.iterations)
    assert np.array_equal(pairs.residual, one.residual)
    assert np.array_equal(pairs.eff_stress, one.eff_stress)
    assert bool((pairs.strain == one.strain).all()) and bool((pairs.stress == one.stress).all())


def test_paths_side_by_side_equal_one_by_one():
    import paper_2103_10203_amd as mor
    import torch
    plans = _plans(mor, GRIDS2[:3])
    d = np.random.default_rng(4).normal(size=(6, 1, 3))
    paths = 0.006 * d / np.linalg.norm(d, axis=2, keepdims=True) * np.array([0.5, 1.0])[None, :, None]
    po = np.arange(6) % 3
    pts = [plans[k].N for k in po]
    state = torch.zeros(5 * sum(pts), dtype=torch.float32, device="cuda")
    got = mor.solve_path_multi(plans, po, paths, native_phases(j2=True), 1e-6, state)
    parts = torch.split(state, [5 * n for n in pts])
    for k in range(3):
        one = torch.zeros(2 * 5 * plans[k].N, dtype=torch.float32, device="cuda")
        want = mor.solve_path_multi([plans[k]], [0, 0], paths[k::3], native_phases(j2=True), 1e-6, one)
        assert np.array_equal(got.iterations[k::3], want.iterations)
        assert np.array_equal(got.eff_stress[k::3], want.eff_stress)
        assert bool((torch.cat([parts[k], parts[k + 3]]) == one).all())
