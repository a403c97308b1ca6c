"""gmg_plan_get_tile where there is no tile: refused, for every role and level."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
def test_one_mcgs_sweep_has_no_tile(dim):
    from paper_1208_4247_amd import capi
    from paper_1208_4247_amd.solver import Plan

    plan = Plan(dim, 4, smoother="mcgs", nu1=1, nu2=1, flags=capi.GMG_FE_TRANSFER)
    for level in range(4):
        for role in (0, 1, 2):
            with pytest.raises(capi.GmgError) as e:
                plan.get_tile(level, role)
            assert e.value.status == capi.GMG_ERR_INVALID_ARG
    assert Plan(dim, 4, nu1=1, nu2=1).get_tile(0, 0)[0] == 2
