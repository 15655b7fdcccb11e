"""Compile-time kernels of the 2^a 3^b lengths: every row length with a column
length, one RVE and many (the same bits where one kernel serves both; within
rounding on the lengths with a kernel for few workgroups), FP32 and FP64, 2D and 3D, against the oracle."""
import math

import numpy as np
import pytest

import synth
from gpu_common import native_phases, oracle_reduced, rel_l2, stress_comps
from oracle import solver

pytestmark = pytest.mark.gpu

ROWS2 = [32, 36, 48, 54, 72, 96, 108, 144, 162, 192, 216, 288, 324, 432]
COLS2 = [54, 32, 36, 48, 96, 72, 108, 162, 144, 216, 192, 288, 432, 324]
SHARED = [(36, 64), (24, 128), (18, 256), (12, 384), (10 * 2 + 4, 512)]


def _map(shape, seed):
    m = min(shape)
    if len(shape) == 3:
        return synth.rsa_spheres(*shape, r_lo=m / 8, r_hi=m / 5, seed=seed, target_vf=0.25).g
    return synth.rsa_fibres(*shape, r_lo=m / 12, r_hi=m / 6, seed=seed, target_vf=0.35).g


def _check(mor, g, M, eb, out, b, precision32=True):
    p, r = oracle_reduced(g, eb, M, 1e-6 if precision32 else 1e-8)
    want = stress_comps(r.sigma_bar, g.ndim)
    assert abs(int(out.iterations[b]) - r.iterations) <= 1
    # FP32 fields: the repository's bars (1e-5 of sigma_bar, 1e-4 of the fields); FP64: 1e-9
    tol, ftol = (1e-5, 1e-4) if precision32 else (1e-9, 1e-6)
    assert np.max(np.abs(out.eff_stress[b][:len(want)] - want)) < tol * np.max(np.abs(want))
    eps = np.moveaxis(solver.tensor_comps(r.eps, g.ndim), -1, 0)
    assert rel_l2(out.strain[b].cpu().numpy(), eps) < ftol


@pytest.mark.parametrize("n0,n1", list(zip(COLS2, ROWS2)) + SHARED)
def test_2d_few_and_many(n0, n1):
    import paper_2103_10203_amd as mor
    g = _map((n0, n1), n0 + n1)
    M = max(9, int(math.ceil(0.06 * g.size)))
    plan = mor.Plan(g, M)
    # more than 512 workgroups of eight rows: the form for many
    B = 520 * 16 // n0 + 1
    eb = synth.macro_strains(B, 3, 5e-3, seed=n1)
    many = mor.solve(plan, eb, native_phases(), 1e-6, want_fields=True)
    few = mor.solve(plan, eb[:1], native_phases(), 1e-6, want_fields=True)
    _check(mor, g, M, eb[0], few, 0)
    if (n0, n1) in SHARED:
        # two kernels: FP32 rounding apart (a few 1e-7 of the field after some
        # 30 iterations), and an iteration where rounding crosses the tolerance
        assert abs(int(many.iterations[0]) - int(few.iterations[0])) <= 1
        assert rel_l2(many.strain[0].cpu().numpy(), few.strain[0].cpu().numpy()) < 3e-6
    else:
        assert many.iterations[0] == few.iterations[0]
        assert np.array_equal(many.eff_stress[0], few.eff_stress[0])
        assert bool((many.strain[0] == few.strain[0]).all())
    if n0 * n1 <= 72 * 72:
        _check(mor, g, M, eb[-1], many, B - 1)


@pytest.mark.parametrize("n0,n1", [(n, m) for n, m in zip(COLS2, ROWS2) if n * m <= 200 * 200] +
                         [(64, 64), (128, 48), (256, 32), (384, 36), (512, 32), (32, 128), (32, 256), (32, 384), (32, 512)])
def test_2d_fp64(n0, n1):
    import paper_2103_10203_amd as mor
    g = _map((n0, n1), n0 + n1)
    M = int(math.ceil(0.06 * g.size))
    plan = mor.Plan(g, M)
    eb = synth.macro_strains(3, 3, 5e-3, seed=n1)
    out = mor.solve(plan, eb, native_phases(), 1e-8, want_fields=True, precision=mor.PREC_FP64)
    _check(mor, g, M, eb[2], out, 2, precision32=False)


@pytest.mark.parametrize("n1", ROWS2 + [64, 128, 256])
def test_2d_j2(n1):
    import paper_2103_10203_amd as mor
    import torch
    from oracle import pattern
    from gpu_common import ORACLE_J2
    g = _map((32, n1), n1)
    M = int(math.ceil(0.08 * g.size))
    plan = mor.Plan(g, M)
    end = np.array([0.008, -0.002, 0.003])
    path = np.stack([end * (k + 1) / 2 for k in range(2)])
    state = torch.zeros(5 * g.size, dtype=torch.float32, device="cuda")
    out = mor.solve_path(plan, path, native_phases(j2=True), 3e-7, state)
    p = pattern.build_pattern(g, M)
    ref = solver.solve_path(g, ORACLE_J2, solver.macro_tensor(end, 2), 2, mask=p.mask(), tol=3e-7, max_iter=4000)
    for k in range(2):
        want = stress_comps(ref[k].sigma_bar, 2)
        assert np.max(np.abs(out.eff_stress[k] - want)) < 1e-5 * np.max(np.abs(want))
    alpha = state.view(5, *g.shape)[4].cpu().numpy()
    assert rel_l2(alpha, ref[-1].alpha) < 1e-4


@pytest.mark.parametrize("shape", [(24, 36, 24), (36, 24, 32), (32, 48, 36), (48, 54, 48), (54, 72, 24), (72, 24, 54),
                                   (96, 24, 72), (108, 24, 24), (24, 96, 24), (24, 108, 96), (24, 24, 108),
                                   (36, 32, 64), (24, 24, 128)])
def test_3d(shape):
    import paper_2103_10203_amd as mor
    g = _map(shape, sum(shape))
    M = int(math.ceil(0.03 * g.size))
    plan = mor.Plan(g, M)
    B = 520 * 16 // (shape[0] * shape[1]) + 1
    eb = synth.macro_strains(max(B, 2), 6, 2e-3, seed=5)
    many = mor.solve(plan, eb, native_phases(), 1e-6, want_fields=True)
    few = mor.solve(plan, eb[:1], native_phases(), 1e-6, want_fields=True)
    _check(mor, g, M, eb[0], few, 0)
    if shape[2] in (64, 128):
        assert rel_l2(many.strain[0].cpu().numpy(), few.strain[0].cpu().numpy()) < 3e-6
    else:
        assert many.iterations[0] == few.iterations[0]
        assert bool((many.strain[0] == few.strain[0]).all())


@pytest.mark.parametrize("n0,n1", SHARED + [(64, 64)])
def test_2d_j2_few_and_many(n0, n1):
    import paper_2103_10203_amd as mor
    import torch
    g = _map((n0, n1), n0 * n1)
    plan = mor.Plan(g, int(math.ceil(0.06 * g.size)))
    B = 520 * 4 // n0 + 1  # more than 512 workgroups of four rows
    d = np.random.default_rng(n1).normal(size=(B, 1, 3))
    paths = 0.006 * d / np.linalg.norm(d, axis=2, keepdims=True) * np.array([0.5, 1.0])[None, :, None]
    state = torch.zeros(5 * g.size * B, dtype=torch.float32, device="cuda")
    many = mor.solve_path_multi([plan], [0] * B, paths, native_phases(j2=True), 1e-6, state)
    one = torch.zeros(5 * g.size, dtype=torch.float32, device="cuda")
    few = mor.solve_path(plan, paths[3], native_phases(j2=True), 1e-6, one)
    # two kernels, both within the FP32 bars of the oracle (1e-5 of sigma_bar,
    # 1e-4 of the fields), so within twice those of each other
    assert np.all(np.abs(many.iterations[3] - few.iterations) <= 1)
    assert np.max(np.abs(many.eff_stress[3][:, :4] - few.eff_stress)) < 2e-5 * np.max(np.abs(few.eff_stress))
    assert rel_l2(state.view(B, 5, -1)[3, 4].cpu().numpy(), one.view(5, -1)[4].cpu().numpy()) < 2e-4
