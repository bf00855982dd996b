"""Batches whose global state is streamed past the caches (plan_global, tabx_kernels.hip): whole and half chunks
at the end of an env's state, zone slots of many envs per wavefront, partial last groups, a level bank, disabled
units; every env against the checker, with the parity tests' own comparison."""
import pytest

from tests.test_gpu_parity import _rollout
from tests.test_gpu_policy import _policy_rollout, _scripted_rollout
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


# scripted and policy ticks, streamed and (the last of each) stored by the lanes that hold the units
SCRIPTED = [(10, 8, 14300), (16, 3, 9901), (1, 5, 84701), (20, 1, 8200), (10, 8, 60), (33, 7, 9), (40, 0, 1300)]
POLICY = [(15, 5, 10401), (10, 3, 15603), (10, 8, 60), (33, 7, 9)]
STORED = {(10, 8, 60), (33, 7, 9), (40, 0, 1300)}


@pytest.mark.parametrize("team,zones,E", SCRIPTED)
def test_global_state_of_scripted_ticks(team, zones, E):
    w, sc = _scene(team, zones, E)
    sc["enabled"] = sc["enabled"].copy()
    sc["enabled"][1::3, -1] = 0
    print(f"[gpu] global state, scripted N={2 * team} Z={zones} E={E}", flush=True)
    _scripted_rollout(w, E, 2, "medium", "adversaries", scenario=sc, global_state=True, max_steps=2)


@pytest.mark.parametrize("team,zones,E", POLICY)
def test_global_state_of_policy_ticks(team, zones, E):
    w, sc = _scene(team, zones, E)
    print(f"[gpu] global state, policy N={2 * team} Z={zones} E={E}", flush=True)
    _policy_rollout(w, E, 2, "medium", "adversaries", scenario=sc, fused=True, global_state=True, max_steps=2)
