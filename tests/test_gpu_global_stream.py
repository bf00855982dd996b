"""Batches whose global state is streamed past the caches (plan_global, tabx_kernels.hip): whole and half chunks
at the end of an env's state, zone slots of many envs per wavefront, partial last groups, a level bank, disabled
units; every env against the checker, with the parity tests' own comparison."""
import pytest

from tests.test_gpu_parity import _rollout
from tests.test_gpu_row_forms import _scene

pytestmark = pytest.mark.gpu


STREAMED = [
    (10, 8, 14300, True, 0), (16, 3, 9901, True, 0), (1, 5, 84701, True, 0), (1, 5, 84701, False, 0),
    (12, 0, 13700, True, 0), (10, 8, 14300, True, 61), (20, 1, 8200, True, 7)]


@pytest.mark.parametrize("team,zones,E,fused,levels", STREAMED)
def test_streamed_global_state(team, zones, E, fused, levels):
    rows = levels or E
    w, sc = _scene(team, zones, rows)
    sc["enabled"] = sc["enabled"].copy()
    sc["enabled"][1::3, -1] = 0
    print(f"[gpu] streamed global state N={2 * team} Z={zones} E={E} fused={fused} levels={levels}", flush=True)
    over = dict(num_levels=levels, level_seed=5) if levels else {}
    _rollout(w, E, 2, fused, scenario=sc, max_steps=2, **over)
