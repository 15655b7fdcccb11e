"""The stop decision inside the row kernel (few workgroups) against the
decision as a launch of its own (many): the same bits of every RVE."""
import numpy as np
import pytest

import synth
from gpu_common import native_phases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("check_every,max_iter", [(0, 0), (1, 0), (5, 0), (3, 7)])
def test_decision_in_row_kernel_equals_launch(check_every, max_iter):
    import paper_2103_10203_amd as mor
    # 64^2: four row workgroups per RVE, so 512 RVEs are the last batch that
    # decides in the row kernel (2048 workgroups) and 513 the first that does not
    g = synth.rsa_fibres(64, 64, 3.0, 6.0, seed=8, target_vf=0.35).g
    plan = mor.Plan(g, 205)
    eb = synth.macro_strains(513, 3, 5e-3, seed=9)
    kw = {"check_every": check_every, "max_iter": max_iter}
    many = mor.solve(plan, eb, native_phases(), 1e-6, **kw)
    few = mor.solve(plan, eb[:512], native_phases(), 1e-6, **kw)
    assert many.status == few.status
    for name in ("iterations", "residual", "eff_stress"):
        assert np.array_equal(getattr(many, name)[:512], getattr(few, name)), name
