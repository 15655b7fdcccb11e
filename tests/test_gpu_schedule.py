"""Calls beyond the line of the row kernel for few workgroups (512 of four
rows), where row_fast iterates: its default variant against the oracle, ragged
row counts included, and the persistent schedule's queue (which it walks in calls
of every size) against the grid schedule, bit for bit."""
import math

import numpy as np
import pytest

import synth
from gpu_common import native_phases, oracle_reduced, rel_l2, stress_comps
from oracle import solver

pytestmark = pytest.mark.gpu


def _map(shape, seed=0):
    m = min(shape)
    if len(shape) == 3:
        return synth.rsa_spheres(*shape, r_lo=m / 6, r_hi=m / 4, seed=seed + sum(shape), target_vf=0.2).g
    return synth.rsa_fibres(*shape, r_lo=m / 10, r_hi=m / 6, seed=seed + sum(shape), target_vf=0.35).g


def _beyond(shape):
    return 512 // math.ceil(math.prod(shape[:-1]) / 4) + 1


@pytest.mark.parametrize("shape", [(36, 64), (64, 64), (36, 128), (72, 256), (18, 384), (36, 512), (12, 6, 64),
                                   (18, 6, 128), (8, 12, 256)])
def test_default_variant_of_large_calls(shape):
    import paper_2103_10203_amd as mor
    g = _map(shape)
    M = max(9, int(math.ceil(0.05 * g.size)))
    plan = mor.Plan(g, M)
    B = _beyond(shape)
    eb = synth.macro_strains(B, 3 if g.ndim == 2 else 6, 2e-3, seed=7)
    out = mor.solve(plan, eb, native_phases(), 1e-6, want_fields=True)
    for b in (0, B - 1):
        _, r = oracle_reduced(g, eb[b], M, 1e-6)
        want = stress_comps(r.sigma_bar, g.ndim)
        assert abs(int(out.iterations[b]) - r.iterations) <= 1
        # the repository's bars: 1e-5 of sigma_bar, 1e-4 of the fields
        assert np.max(np.abs(out.eff_stress[b][:len(want)] - want)) < 1e-5 * np.max(np.abs(want))
        eps = np.moveaxis(solver.tensor_comps(r.eps, g.ndim), -1, 0)
        assert rel_l2(out.strain[b].cpu().numpy(), eps) < 1e-4


@pytest.mark.parametrize("shapes", [[(64, 64), (72, 256), (36, 128)], [(18, 384), (36, 512)],
                                    [(12, 6, 64), (18, 6, 128)]])
def test_persistent_equals_grid(shapes):
    import paper_2103_10203_amd as mor
    gs = [_map(s, 50) for s in shapes]
    plans = [mor.Plan(g, int(math.ceil(0.05 * g.size))) for g in gs]
    B = len(shapes) * max(_beyond(s) for s in shapes)
    po = np.arange(B) % len(shapes)
    eb = synth.macro_strains(B, 3 if len(shapes[0]) == 2 else 6, 5e-3, seed=21)
    eb[3] = 0.0  # converges at once
    grid = mor.solve_multi(plans, po, eb, native_phases(), 1e-6, want_fields=True)
    assert len(set(grid.iterations.tolist())) > 1
    for kw in ({}, {"use_graph": 1}):
        pers = mor.solve_multi(plans, po, eb, native_phases(), 1e-6, want_fields=True, schedule=mor.SCHED_PERSISTENT,
                               **kw)
        assert np.array_equal(grid.eff_stress, pers.eff_stress)
        assert np.array_equal(grid.iterations, pers.iterations)
        assert bool((grid.strain == pers.strain).all()) and bool((grid.stress == pers.stress).all())


@pytest.mark.parametrize("shape", [(64, 64), (36, 512)])
def test_persistent_equals_grid_j2(shape):
    import paper_2103_10203_amd as mor
    import torch
    g = _map(shape, 75)
    plan = mor.Plan(g, int(math.ceil(0.05 * g.size)))
    B = _beyond(shape)
    d = np.random.default_rng(3).normal(size=(B, 1, 3))
    paths = 0.006 * d / np.linalg.norm(d, axis=2, keepdims=True) * np.array([0.5, 1.0])[None, :, None]
    res = []
    for kw in ({}, {"schedule": mor.SCHED_PERSISTENT}):
        state = torch.zeros(5 * g.size * B, dtype=torch.float32, device="cuda")
        res.append((mor.solve_path_multi([plan], [0] * B, paths, native_phases(j2=True), 1e-6, state, **kw), state))
    assert np.array_equal(res[0][0].iterations, res[1][0].iterations)
    assert np.array_equal(res[0][0].eff_stress, res[1][0].eff_stress)
    assert bool((res[0][1] == res[1][1]).all())


def test_pairs_beside_runs_that_go_alone():
    """Under a limit of 24 MiB: 256 RVEs of 128^2 go as a pair of runs, 40 of 256^2
    (too few workgroups for a pair, beyond half the limit) alone, and 20 of 64^2
    beside the pair; with a set minimum of 129 RVEs nothing is paired.  The bits
    are those of one run per grid."""
    import paper_2103_10203_amd as mor
    sizes = [128] * 256 + [256] * 40 + [64] * 20
    plans = [mor.Plan(g, int(math.ceil(0.05 * g.size))) for g in (_map((n, n), 9) for n in (128, 256, 64))]
    po = np.array([{128: 0, 256: 1, 64: 2}[n] for n in sizes])[np.random.default_rng(2).permutation(len(sizes))]
    eb = synth.macro_strains(len(po), 3, 5e-3, seed=4)
    keep = mor.tune_subbatch(0)
    try:
        want = mor.solve_multi(plans, po, eb, native_phases(), 1e-6, want_fields=True)
        for limit, least in ((24 << 20, -1), (24 << 20, 129), (24 << 20, 64), (4 << 20, 1)):
            mor.tune_subbatch(limit, least)
            for _ in range(2):
                got = mor.solve_multi(plans, po, eb, native_phases(), 1e-6, want_fields=True)
                assert np.array_equal(got.iterations, want.iterations)
                assert np.array_equal(got.residual, want.residual)
                assert np.array_equal(got.eff_stress, want.eff_stress)
                assert bool((got.strain == want.strain).all()) and bool((got.stress == want.stress).all())
    finally:
        mor.tune_subbatch(*keep)
