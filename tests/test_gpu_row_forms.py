"""How the observation rows are made depends on the row length (whole 16-byte chunks or not), the
zone slots, the units per env and the batch size; every form at sizes where it can go wrong: tiles
that end inside an env, rows that start in the middle of a chunk, inactive zone slots between active
ones, partial last groups, few envs of many units (further wavefronts write rows) and many of them.
Every env and field against the checker, with the parity tests' own comparison."""
import numpy as np
import pytest

from paper_2602_01665_amd import inputs as I
from tests.test_gpu_parity import _rollout
from tests.test_gpu_policy import _policy_rollout, _scripted_rollout

pytestmark = pytest.mark.gpu


def _scene(team, zones, E):
    w = I.Workload(f"rows_{2 * team}u_{zones}z", E, team, 40.0, 20, "iid", 0.6, "iid", max_zones=zones,
                   steps=9, seed=700 + 17 * team + zones)
    sc = I.make_scenario(w, E)
    if zones:
        rng = np.random.default_rng(zones)
        d = rng.uniform(1.0, 30.0, size=(E, zones, 6)).astype(np.float32)
        d[..., 0] = rng.integers(0, 4, size=(E, zones))       # a type of 0 leaves the slot out
        sc["zone_desc"] = d
    return w, sc


TICKS = [
    # team size, zone slots, envs, ticks
    (1, 16, 70, 12), (1, 5, 33, 12), (2, 1, 9, 12), (5, 3, 61, 12), (8, 7, 9, 12), (16, 11, 5, 9),
    (32, 1, 3, 9),                                            # one row per tile
    (8, 1, 8300, 3), (10, 3, 6200, 3), (16, 8, 4200, 3),      # a full machine, two passes per tile or not
    (33, 0, 5, 9), (50, 5, 5, 9), (64, 16, 3, 9), (64, 15, 2, 9),        # few envs of many units
    (33, 8, 520, 4), (33, 7, 520, 4), (64, 1, 515, 3),        # many of them
    (64, 0, 20, 6), (60, 0, 270, 3), (33, 2, 1030, 2),        # six and four wavefronts, two
    (33, 0, 1290, 2), (33, 7, 1030, 2), (40, 1, 1290, 2),     # three wavefronts per SIMD at most; half a chunk
    (12, 0, 70, 6), (20, 2, 300, 4), (2, 16, 70, 8), (2, 16, 4200, 3), (1, 16, 8203, 3),       # more zone chunks than lanes: few envs per wavefront or not
]


@pytest.mark.parametrize("fused", [True, False], ids=["fused", "separate"])
@pytest.mark.parametrize("team,zones,E,ticks", TICKS)
def test_rows(team, zones, E, ticks, fused):
    w, sc = _scene(team, zones, E)
    print(f"[gpu] rows N={2 * team} Z={zones} E={E} fused={fused}", flush=True)
    _rollout(w, E, ticks, fused, scenario=sc, max_steps=5)


DECIDING = [(8, 3, 9, 8), (25, 0, 7, 6), (10, 8, 50, 6), (31, 5, 300, 3), (10, 8, 2100, 3), (33, 0, 520, 3), (33, 3, 520, 3), (50, 4, 5, 6), (64, 16, 3, 6),
            (33, 3, 1030, 2), (33, 0, 1290, 2), (64, 0, 20, 4), (10, 8, 2400, 2),
            (33, 7, 1290, 2), (40, 1, 1540, 2)]


@pytest.mark.parametrize("form", ["scripted", "scan"])
@pytest.mark.parametrize("team,zones,E,ticks", DECIDING)
def test_rows_with_deciding_units(team, zones, E, ticks, form):
    w, sc = _scene(team, zones, E)
    print(f"[gpu] deciding N={2 * team} Z={zones} E={E} {form}", flush=True)
    if form == "scripted":
        _scripted_rollout(w, E, ticks, "medium", "adversaries", scenario=sc, max_steps=4)
    else:
        _policy_rollout(w, E, ticks, "medium", "adversaries", scenario=sc, fused=True, max_steps=4)


@pytest.mark.parametrize("slop", [-0.8, 0.0, 0.4])
@pytest.mark.parametrize("team,E", [(5, 40), (32, 5), (40, 4)])
@pytest.mark.parametrize("dynamics", [False, True], ids=["kinematic", "persistent"])
def test_contacts_near_the_reach(team, E, slop, dynamics):
    """Crowded arenas: many pairs at about the distance where the pair test of body collisions stops
    (a negative slop pushes bodies that do not touch yet)."""
    w = I.Workload(f"crowd_{team}", E, team, 14.0, 0, "none", 1.0, "iid", steps=9, seed=31 + team)
    over = dict(collision_alpha=0.8, collision_slop=slop, max_steps=6)
    if dynamics:
        over.update(dynamics=1, move_gain=2.0, restitution=0.5)
    print(f"[gpu] contacts N={2 * team} slop={slop} {over}", flush=True)
    _rollout(w, E, 8, True, **over)


@pytest.mark.parametrize("team,zones,E,over", [
    (4, 4, 50, {}), (10, 8, 40, {}), (12, 8, 41, dict(collision_alpha=0.8)), (21, 5, 270, {}), (30, 4, 300, {}),
    (30, 4, 9, dict(num_levels=5, level_seed=3)), (16, 6, 3300, {}),
])
def test_rows_with_elliptical_zones(team, zones, E, over):
    """Zones that the step looks up before the rows: two or four wavefronts per group, two passes per tile."""
    w = I.Workload(f"ellipses_{2 * team}u", E, team, 40.0, 0, "ellipses", 1.0, "iid", max_zones=zones, steps=9,
                   seed=300 + team)
    sc = I.make_scenario(w, over.get("num_levels", E))
    print(f"[gpu] ellipses N={2 * team} Z={zones} E={E} {over}", flush=True)
    _rollout(w, E, 5, True, scenario=sc, max_steps=3, **over)


@pytest.mark.parametrize("N,E", [(9, 40), (19, 100), (31, 70), (33, 30)])
def test_separate_rows_of_odd_units(N, E):
    """Stand-alone observe of odd numbers of units: one row a flush, more workgroups per env group."""
    import torch
    from oracle.ref import RefEnv
    from paper_2602_01665_amd.binding import TabxEnv
    from tests.parity import compare_outputs
    w = I.Workload(f"odd_{N}", E, (N + 1) // 2, 40.0, 0, "none", 1.0, "iid", seed=50 + N)
    sc = I.make_scenario(w, E)
    sc = {k: (v if v is None or v.ndim != 2 else np.ascontiguousarray(v[:, :N])) for k, v in sc.items()}
    p = I.make_params(w, E, num_units=N)
    ref, gpu = RefEnv(p, sc), TabxEnv(p, sc)
    ref.reset()
    gpu.reset()
    ref.observe()
    gpu.observe()
    torch.cuda.synchronize()
    print(f"[gpu] observe N={N} E={E}", flush=True)
    compare_outputs(gpu, ref, f"N={N} E={E}: ")
