"""An RVE gives the same bits alone, in a small call and in a large batch,
although the row lengths of row_fast iterate on another row kernel while the
call has at most 512 workgroups of four rows: every such length, Hooke and J2,
2D and 3D, on both sides of that line."""
import math

import numpy as np
import pytest

import synth
from gpu_common import native_phases

pytestmark = pytest.mark.gpu

SHAPES = [(36, 64), (64, 64), (24, 128), (18, 256), (12, 384), (24, 512), (16, 8, 64), (8, 12, 128), (8, 8, 256)]


def _plan(mor, shape):
    m = min(shape)
    if len(shape) == 3:
        g = synth.rsa_spheres(*shape, r_lo=m / 6, r_hi=m / 4, seed=sum(shape), target_vf=0.2).g
    else:
        g = synth.rsa_fibres(*shape, r_lo=m / 10, r_hi=m / 6, seed=sum(shape), target_vf=0.35).g
    return mor.Plan(g, max(9, int(math.ceil(0.06 * g.size))))


def _beyond(shape):
    """RVEs of the first call beyond 512 workgroups of four rows."""
    return 512 // math.ceil(math.prod(shape[:-1]) / 4) + 1


@pytest.mark.parametrize("shape", SHAPES)
def test_hooke(shape):
    import paper_2103_10203_amd as mor
    plan = _plan(mor, shape)
    B = _beyond(shape)
    eb = synth.macro_strains(B, 3 if len(shape) == 2 else 6, 5e-3, seed=shape[-1])
    many = mor.solve(plan, eb, native_phases(), 1e-6, want_fields=True)
    few = mor.solve(plan, eb[:B - 1], native_phases(), 1e-6, want_fields=True)
    assert np.array_equal(many.iterations[:B - 1], few.iterations)
    assert np.array_equal(many.residual[:B - 1], few.residual)
    assert np.array_equal(many.eff_stress[:B - 1], few.eff_stress)
    assert bool((many.strain[:B - 1] == few.strain).all()) and bool((many.stress[:B - 1] == few.stress).all())
    for b in (0, B - 1):
        one = mor.solve(plan, eb[b:b + 1], native_phases(), 1e-6, want_fields=True)
        assert many.iterations[b] == one.iterations[0] and many.residual[b] == one.residual[0]
        assert np.array_equal(many.eff_stress[b], one.eff_stress[0])
        assert bool((many.strain[b] == one.strain[0]).all()) and bool((many.stress[b] == one.stress[0]).all())


@pytest.mark.parametrize("shape", SHAPES)
def test_j2(shape):
    import paper_2103_10203_amd as mor
    import torch
    plan = _plan(mor, shape)
    dim, N = len(shape), math.prod(shape)
    C, K = (3, 5) if dim == 2 else (6, 7)
    B = _beyond(shape)
    d = np.random.default_rng(shape[-1]).normal(size=(B, 1, C))
    paths = 0.006 * d / np.linalg.norm(d, axis=2, keepdims=True) * np.array([0.5, 1.0])[None, :, None]
    state = torch.zeros(K * N * B, dtype=torch.float32, device="cuda")
    many = mor.solve_path_multi([plan], [0] * B, paths, native_phases(j2=True), 1e-6, state)
    assert float(state.view(B, K, N)[:, K - 1].max()) > 0.0  # some points yield
    for b in (0, B - 1):
        one = torch.zeros(K * N, dtype=torch.float32, device="cuda")
        few = mor.solve_path_multi([plan], [0], paths[b:b + 1], native_phases(j2=True), 1e-6, one)
        assert np.array_equal(many.iterations[b], few.iterations[0])
        assert np.array_equal(many.eff_stress[b], few.eff_stress[0])
        assert bool((state.view(B, -1)[b] == one).all())


def test_decision_in_row_kernel_equals_launch_for_one():
    """64^2: 513 RVEs decide in a launch of its own, one in its row kernel."""
    import paper_2103_10203_amd as mor
    g = synth.rsa_fibres(64, 64, 3.0, 6.0, seed=8, target_vf=0.35).g
    plan = mor.Plan(g, 205)
    eb = synth.macro_strains(513, 3, 5e-3, seed=9)
    for kw in ({}, {"check_every": 1}, {"check_every": 3, "max_iter": 7}):
        many = mor.solve(plan, eb, native_phases(), 1e-6, **kw)
        one = mor.solve(plan, eb[7:8], native_phases(), 1e-6, **kw)
        for name in ("iterations", "residual", "eff_stress"):
            assert np.array_equal(getattr(many, name)[7:8], getattr(one, name)), name
