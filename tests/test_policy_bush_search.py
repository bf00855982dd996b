"""The Rangers' bush search inside the policy tick.  Every unit is a Ranger that sees nobody and remembers
nothing, so the nearest bush among the zone slots decides every action: whatever else the wavefronts that
step the envs might read in place of their envs' descriptors, actions and everything after them differ."""
import numpy as np
import pytest

from paper_2602_01665_amd import inputs as I

# team size, zone slots, envs: rows that end on half a 16-byte chunk, and few envs of many units
SHAPES = [(8, 3, 9), (10, 7, 200), (1, 5, 40), (33, 3, 6), (33, 8, 500), (50, 8, 5), (64, 16, 3)]
POLICY = dict(I.policy("expert", 3), epsilon=0.0)


def _scene(team, zones, E):
    w = I.Workload(f"bush_{2 * team}u_{zones}z", E, team, 40.0, 0, "none", 1.0, "iid", max_zones=zones,
                   seed=90 + team + zones)
    sc = I.make_scenario(w, E)
    row = I.ROSTER["archer"]
    for k, v in zip(("hmax", "radius", "mass", "speed", "dmg", "range", "cooldown"), row):
        sc[k][:] = np.float32(v)
    sc["sight_range"][:] = np.float32(1e-6)
    rng = np.random.default_rng(5 * team + zones)
    d = rng.uniform(1.0, 39.0, size=(E, zones, 6)).astype(np.float32)
    kind = rng.choice([0, 1, 2, 2, 3], size=(E, zones))
    kind[np.arange(E), rng.integers(0, zones, size=E)] = I.ZONE_BUSH
    d[..., 0] = kind
    sc["zone_desc"] = d
    return I.make_params(w, E, max_steps=4), sc


def _ref(p, sc):
    from oracle.ref import RefEnv
    ref = RefEnv(p, sc)
    ref.reset()
    return ref


@pytest.mark.parametrize("team,zones,E", SHAPES)
def test_the_slots_decide(team, zones, E):
    """(With the checker alone.)  Every unit walks, and to another place if its env had no bush, or the
    descriptors of another env."""
    p, sc = _scene(team, zones, E)
    every = np.ones((E, 2 * team), np.uint8)

    def first(zone_desc):
        a = np.zeros((E, 2 * team), np.uint8)
        _ref(p, dict(sc, zone_desc=zone_desc)).heuristic_actions(POLICY, every, a)
        return a

    a = first(sc["zone_desc"])
    assert ((a >= I.ACT_XP) & (a <= I.ACT_YM)).all()
    none = sc["zone_desc"].copy()
    none[..., 0] = 0.0
    assert (first(none) != a).all()
    assert (first(np.roll(sc["zone_desc"], 1, axis=0)) != a).mean() > 0.2


@pytest.mark.gpu
@pytest.mark.parametrize("team,zones,E", SHAPES)
def test_policy_tick(team, zones, E):
    import torch
    from paper_2602_01665_amd import binding as B
    from tests.parity import compare_outputs, compare_state
    p, sc = _scene(team, zones, E)
    N = 2 * team
    ref = _ref(p, sc)
    gpu = B.TabxEnv(p, sc, want_global_state=True)
    gpu.reset()
    info = B.tabx_launch_info(gpu.params, "policy_step_observe")
    # (further wavefronts than those that step: they may write the rows only)
    assert info["wavefronts_per_env_group"] == (4 if N > 64 else 2), info
    print(f"[gpu] bush search N={N} Z={zones} E={E}", flush=True)
    every = np.ones((E, N), np.uint8)
    for s in range(6):
        where = f"bush search N={N} Z={zones} E={E} step {s}: "
        a = np.zeros((E, N), np.uint8)
        ad = torch.zeros(E, N, dtype=torch.uint8, device=gpu.device)
        ref.policy_step(POLICY, every, a)
        ref.observe()
        gpu.policy_step_observe(POLICY, None, ad)
        torch.cuda.synchronize()
        assert np.array_equal(ad.cpu().numpy(), a), where + "actions"
        compare_state(gpu.state_numpy(), ref.st, where)
        compare_outputs(gpu, ref, where)
        assert np.array_equal(gpu.gs_live.cpu().numpy(), ref.global_state()), where + "global state"
