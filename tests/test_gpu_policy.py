"""Heuristic policy: HIP library vs CPU checker through the C ABI (needs an MI355X).

Actions and the memory-valid flags are bit-exact, remembered positions equal as floats;
the rollouts feed each side its own actions, so a single differing action would also show
as a state mismatch on the following tick.
"""
import sys

import numpy as np
import pytest

from paper_2602_01665_amd import inputs as I
from tests.parity import compare_outputs, compare_state

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _check_memory(gpu, ref, E, N, where):
    valid = gpu.mem["mem_valid"].cpu().numpy().reshape(E, N)
    assert np.array_equal(valid, ref.mem["mem_valid"]), where + "mem_valid"
    for k in ("mem_x", "mem_y"):
        g = gpu.mem[k].cpu().numpy().reshape(E, N)
        assert np.array_equal(g[valid == 1], ref.mem[k][valid == 1]), where + k


def _policy_rollout(w, E, steps, tier, who, scenario=None, seed=5, fused=False, global_state=False, **override):
    """who: "adversaries" (allies act at random), "both", or "allies".  fused: the policy runs
    inside the tick launch (tabx_policy_step_observe).  global_state: the tick leaves it as well."""
    import torch
    from oracle.ref import RefEnv
    from paper_2602_01665_amd.binding import TabxEnv
    p = I.make_params(w, E, **override)
    sc = I.make_scenario(w, E) if scenario is None else scenario
    N = p["num_units"]
    ref = RefEnv(p, sc)
    gpu = TabxEnv(p, sc, want_metrics=True, want_global_state=global_state)
    ref.reset()
    gpu.reset()
    team = np.asarray(sc["team"]).reshape(E, N)
    ctl = {"adversaries": team == 1, "allies": team == 0,
           "both": np.ones_like(team, bool)}[who].astype(np.uint8)
    ctl_d = None if who == "both" else torch.from_numpy(ctl).to(gpu.device)
    pol = I.policy(tier, seed)
    hist = np.zeros(8, np.int64)
    dones = 0
    for s in range(steps):
        a = I.actions_for_step(w.seed, s, E, N)
        ad = torch.from_numpy(a).to(gpu.device)
        where = f"{w.name} E={E} {tier}/{who} step {s}: "
        if fused:
            ref.policy_step(pol, ctl, a)
            ref.observe()
            gpu.policy_step_observe(pol, ctl_d, ad)
            torch.cuda.synchronize()
            got = ad.cpu().numpy()
            bad = np.argwhere(got != a)
            assert bad.size == 0, where + f"actions differ at {bad[:5].tolist()}"
            _check_memory(gpu, ref, E, N, where)
            compare_state(gpu.state_numpy(), ref.st, where)
            compare_outputs(gpu, ref, where, check_obs=True)
            if global_state:
                assert np.array_equal(gpu.gs_live.cpu().numpy(), ref.global_state()), where + "global state"
            hist += np.bincount(a[ctl == 1], minlength=8)
            dones += int(ref.dones.sum())
            continue
        ref.heuristic_actions(pol, ctl, a)
        gpu.heuristic_actions(pol, ctl_d, ad)
        torch.cuda.synchronize()
        got = ad.cpu().numpy()
        bad = np.argwhere(got != a)
        assert bad.size == 0, where + f"actions differ at {bad[:5].tolist()}: " \
            f"{got[tuple(bad[0])]} vs {a[tuple(bad[0])]}"
        _check_memory(gpu, ref, E, N, where)
        hist += np.bincount(a[ctl == 1], minlength=8)
        ref.step(a)
        gpu.step(ad)
        torch.cuda.synchronize()
        compare_state(gpu.state_numpy(), ref.st, where)
        assert np.array_equal(gpu.dones.cpu().numpy(), ref.dones), where + "dones"
        done = ref.dones.astype(bool)
        if done.any():                       # a new episode starts with an empty memory
            ref.mem["mem_valid"][done] = 0
            gpu.mem["mem_valid"].view(E, N)[torch.from_numpy(done).to(gpu.device)] = 0
            dones += int(done.sum())
    return hist, dones


TIERS = ["random", "novice", "medium", "advanced", "expert"]


@pytest.mark.parametrize("fused", [False, True], ids=["separate", "fused"])
@pytest.mark.parametrize("tier", TIERS)
def test_adversaries_under_every_tier(tier, fused):
    _say(f"[gpu] policy c3 subset, adversaries, tier {tier}, fused={fused}")
    hist, dones = _policy_rollout(I.WORKLOADS["c3_16384env_10v10"], 48, 120, tier, "adversaries",
                                  fused=fused, max_steps=96)
    _say(f"[gpu]   action histogram {hist.tolist()} episodes ended {dones}")
    assert hist.sum() > 0


@pytest.mark.parametrize("name,E,steps,over", [
    ("c1_16env_3v3", 16, 256, dict()),
    ("c2_4096env_5v5", 200, 200, dict(max_steps=128)),
    ("c3_16384env_10v10", 70, 200, dict(max_steps=128)),
    ("c3e_16384env_10v10_ellipses", 70, 200, dict(max_steps=128)),
    ("c5_1024env_64v64", 3, 80, dict(max_steps=60)),
], ids=lambda v: v if isinstance(v, str) else None)
@pytest.mark.parametrize("fused", [False, True], ids=["separate", "fused"])
def test_self_play_rollouts(name, E, steps, over, fused):
    _say(f"[gpu] policy self-play {name} E={E} steps={steps} fused={fused}")
    hist, dones = _policy_rollout(I.WORKLOADS[name], E, steps, "expert", "both", fused=fused,
                                  **over)
    _say(f"[gpu]   action histogram {hist.tolist()} episodes ended {dones}")
    # seek-and-approach, combat, turning and search all occur
    assert hist[5] > 0 and hist[1:5].sum() > 0 and hist[6:].sum() > 0
    assert dones > 0


def test_every_roster_unit_and_role_mix():
    """All nine roster units on both teams (Healers, Assassin, Rangers, plain units), terrain
    with bushes, greedy and noisy tiers."""
    names = list(I.ROSTER)
    E, N = 40, 2 * len(names)
    w = I.Workload("roster_policy", E, len(names), 48.0, 24, "iid", 0.5, "iid", steps=150,
                   seed=777)
    sc = I.make_scenario(w, E)
    for u in range(N):
        row = I.ROSTER[names[u % len(names)]]
        for k, v in zip(("hmax", "radius", "mass", "speed", "dmg", "range", "cooldown"), row):
            sc[k][:, u] = np.float32(v)
        sc["hurt_halfwidth"][:, u] = np.float32(row[1])
    for tier in ("expert", "medium"):
        _say(f"[gpu] policy roster mix, tier {tier}")
        hist, dones = _policy_rollout(w, E, 150, tier, "both", scenario=sc,
                                      fused=tier == "medium", max_steps=120)
        _say(f"[gpu]   action histogram {hist.tolist()} episodes ended {dones}")
        assert hist[5] > 0


def test_units_that_hold_several_roles():
    """Fast Rangers (Ranger and Assassin), fast Healers (Healer, Ranger and Assassin), fast plain
    units, and a Healer just below the Ranger threshold, on both teams."""
    E = 48
    w = I.Workload("multi_role_policy", E, 8, 40.0, 20, "iid", 0.6, "iid", steps=120, seed=4242)
    sc = I.make_scenario(w, E)
    rows = [("archer", dict(speed=1.6)), ("healer", dict(speed=1.6)), ("farmer", dict(speed=1.6)),
            ("healer", dict(range=9.9)), ("archer", {}), ("assassin", dict(range=10.0)),
            ("deadeye", dict(speed=1.4)), ("farmer", {})]
    for u in range(w.num_units):
        name, over = rows[u % len(rows)]
        vals = dict(zip(("hmax", "radius", "mass", "speed", "dmg", "range", "cooldown"), I.ROSTER[name]))
        vals.update(over)
        for k, v in vals.items():
            sc[k][:, u] = np.float32(v)
        sc["hurt_halfwidth"][:, u] = np.float32(vals["radius"])
    for tier, fused in (("expert", False), ("advanced", True)):
        _say(f"[gpu] policy with multi-role units, tier {tier}")
        hist, dones = _policy_rollout(w, E, 120, tier, "both", scenario=sc, fused=fused, max_steps=90)
        _say(f"[gpu]   action histogram {hist.tolist()} episodes ended {dones}")
        assert hist[5] > 0 and hist[1:5].sum() > 0


def test_ragged_and_padded_units():
    for team_size, disabled in [(1, 0), (7, 2), (33, 4), (50, 9)]:
        w = I.Workload(f"ragged_policy_{team_size}", 5, team_size, 40.0, 20, "iid", 0.6, "iid",
                       steps=60, seed=5252 + team_size)
        sc = I.make_scenario(w, 5)
        rng = np.random.default_rng(team_size)
        for e in range(5):
            off = rng.choice(w.num_units, size=min(disabled, w.num_units - 2), replace=False)
            off = [u for u in off if u not in (0, w.num_units - 1)]
            sc["enabled"][e, off] = 0
        _say(f"[gpu] policy ragged N={w.num_units} disabled={disabled}")
        _policy_rollout(w, 5, 60, "advanced", "both", scenario=sc, max_steps=40)
        _policy_rollout(w, 5, 60, "advanced", "adversaries", scenario=sc, fused=True,
                        max_steps=40)


def test_uncontrolled_entries_are_left_alone_and_errors():
    import torch
    from paper_2602_01665_amd import binding as B
    w = I.WORKLOADS["c2_4096env_5v5"]
    E = 64
    p, sc = I.make_params(w, E), I.make_scenario(w, E)
    gpu = B.TabxEnv(p, sc)
    gpu.reset()
    N = p["num_units"]
    ctl = torch.zeros(E, N, dtype=torch.uint8, device=gpu.device)
    ctl[:, N // 2:] = 1
    a = torch.full((E, N), 99, dtype=torch.uint8, device=gpu.device)
    gpu.heuristic_actions(I.policy("expert", 1), ctl, a)
    torch.cuda.synchronize()
    got = a.cpu().numpy()
    assert (got[:, :N // 2] == 99).all() and (got[:, N // 2:] < 8).all()
    # NULL outputs / memory and a non-finite coefficient are refused on the host
    with pytest.raises(B.TabxError):
        B.tabx_heuristic_actions(gpu.params, gpu.scenario, gpu.state,
                                 B.TabxPolicy(**I.policy("expert", 1)), gpu.memory, None, None)
    with pytest.raises(B.TabxError):
        B.tabx_heuristic_actions(gpu.params, gpu.scenario, gpu.state,
                                 B.TabxPolicy(**I.policy("expert", 1)), B.TabxPolicyMemory(),
                                 None, a)
    with pytest.raises(B.TabxError):
        B.tabx_heuristic_actions(gpu.params, gpu.scenario, gpu.state,
                                 B.TabxPolicy(**dict(I.policy("expert", 1), xi=float("nan"))),
                                 gpu.memory, None, a)


def test_full_size_scripted_tick_with_level_bank():
    """The launch `bench.py --policy` times (16384 envs 10v10, adversaries scripted inside the
    tick), here also with a bank of levels; the checker replays a sample of the envs under their
    original indices and every tick of them is compared."""
    import torch
    from oracle.ref import RefEnv
    from paper_2602_01665_amd.binding import TabxEnv
    from tests.parity import compare_metrics
    w = I.WORKLOADS["c3_16384env_10v10"]
    E, N, L, steps = w.num_envs, w.num_units, 96, 300
    _say(f"[gpu] full size scripted tick E={E} levels={L} steps={steps}")
    p = I.make_params(w, max_steps=64, num_levels=L, level_seed=5)
    sc = I.make_scenario(w, L)
    rng = np.random.default_rng(3)
    rows = np.unique(np.concatenate([[0, 1, E - 1], rng.choice(E, 9, replace=False)]))
    ref = RefEnv(dict(p, num_envs=len(rows), env_ids=rows), sc)
    gpu = TabxEnv(p, sc, want_metrics=True)
    ref.st["next_level"][:] = rows % L           # what the full batch queues for these envs
    ref.reset()
    gpu.reset()
    rows_t = torch.from_numpy(rows).to("cuda:0")
    team = torch.from_numpy(np.ascontiguousarray(sc["team"])).to("cuda:0")
    pol = I.policy("medium", w.seed)
    # the bank's teams are the same in every level of this workload: one mask serves all
    assert (sc["team"] == sc["team"][0]).all()
    ctl_d = team[:1].expand(E, N).contiguous()
    ctl = np.broadcast_to(sc["team"][0], (len(rows), N)).astype(np.uint8)
    dones = 0
    for s in range(steps):
        a = I.actions_for_step(w.seed, s, E, N)
        ad = torch.from_numpy(a).to("cuda:0")
        ar = np.ascontiguousarray(a[rows])
        gpu.policy_step_observe(pol, ctl_d, ad)
        ref.policy_step(pol, ctl, ar)
        ref.observe()
        torch.cuda.synchronize()
        where = f"full size scripted step {s}: "
        assert np.array_equal(ad[rows_t].cpu().numpy(), ar), where + "actions"
        st = {k: (v.reshape(E, N)[rows_t] if v.numel() == E * N else v[rows_t]).cpu().numpy()
              for k, v in gpu.st.items()}
        compare_state(st, ref.st, where)
        compare_outputs(gpu, ref, where, rows=rows_t)
        compare_metrics(gpu, ref, where, rows=rows_t)
        valid = gpu.mem["mem_valid"].view(E, N)[rows_t].cpu().numpy()
        assert np.array_equal(valid, ref.mem["mem_valid"]), where + "mem_valid"
        dones += int(ref.dones.sum())
        if s % 100 == 0:
            _say(f"[gpu]   step {s} ok")
    _say(f"[gpu]   sampled episodes ended {dones}")
    assert dones > len(rows)
    assert torch.isfinite(gpu.obs).all()


def test_full_size_scripted_tick_every_env():
    """The launch `bench.py --policy medium` times, EVERY env of it: the checker (envs dealt to
    host threads) decides and steps the whole batch, and the actions applied, every state field,
    the outputs and the memory flags are compared bit for bit after every tick, past the
    truncation horizon.  (One-off runs of the same comparison: c4 / expert 300 ticks, c5 /
    novice 270, c3 with elliptical zones / advanced 300, all bit-identical.)"""
    import torch
    from paper_2602_01665_amd.binding import TabxEnv
    from tests.helpers import ShardedRef
    from tests.parity import FLOAT_STATE, INT_STATE
    w = I.WORKLOADS["c3_16384env_10v10"]
    E, N, ticks = w.num_envs, w.num_units, 280
    _say(f"[gpu] full size scripted tick, every env: E={E} N={N} ticks={ticks}")
    sc = I.make_scenario(w)
    ref = ShardedRef(w, lambda n: I.make_params(w, n), sc)
    gpu = TabxEnv(I.make_params(w), sc)
    ref.reset()
    gpu.reset()
    team = np.ascontiguousarray(sc["team"], np.uint8).reshape(E, N)
    ctl_d = torch.from_numpy(team).to("cuda:0")
    pol = I.policy("medium", w.seed)
    gpu.prime_scripted(pol, ctl_d)

    def same(t, want):
        want = torch.from_numpy(np.ascontiguousarray(want))
        return torch.equal(t.reshape(-1).view(torch.uint8), want.to(t.device).reshape(-1).view(torch.uint8))

    dones = 0
    for s in range(ticks):
        where = f"full size scripted, every env, tick {s}: "
        a = I.actions_for_step(w.seed, s, E, N).copy()
        ad = torch.from_numpy(a.copy()).to("cuda:0")
        waiting_flags = gpu.mem["mem_valid"].clone()       # after the decisions for this tick
        flags = ref.scripted_tick(pol, team, a)
        gpu.scripted_step_observe(pol, ctl_d, ad)
        assert same(waiting_flags, flags), where + "memory flags"
        assert same(ad, a), where + "actions applied"
        assert same(gpu.obs, ref.obs), where + "obs"
        for k in FLOAT_STATE + INT_STATE:
            assert same(gpu.st[k], ref.state(k)), where + k
        assert same(gpu.rewards, ref.output("rewards")), where + "rewards"
        assert same(gpu.dones, ref.output("dones")), where + "dones"
        assert same(gpu.vis, ref.output("vis").view(np.int64)), where + "vis_mask"
        assert same(gpu.amask, ref.output("amask")), where + "action_mask"
        dones += int(ref.output("dones").sum())
        if s % 50 == 0:
            _say(f"[gpu]   tick {s} ok")
    _say(f"[gpu]   all {ticks} ticks bit-identical, {dones} episodes ended")
    assert dones >= E


def _scripted_rollout(w, E, steps, tier, who, scenario=None, seed=5, global_state=False, **override):
    """tabx_scripted_step_observe (decisions taken inside the observe stage, applied by the next
    call) against the checker's decide-then-step sequence: actions, states, observations,
    memories and the waiting decisions must all agree, tick by tick."""
    import torch
    from oracle.ref import RefEnv
    from paper_2602_01665_amd.binding import TabxEnv
    p = I.make_params(w, E, **override)
    L = p.get("num_levels", 0)
    sc = I.make_scenario(w, L if L else E) if scenario is None else scenario
    N = p["num_units"]
    ref = RefEnv(p, sc)
    gpu = TabxEnv(p, sc, want_metrics=True, want_global_state=global_state)
    ref.reset()
    gpu.reset()
    team = np.asarray(sc["team"]).reshape(-1, N)
    team = team[ref.st["level"]] if L else team
    ctl = {"adversaries": team == 1, "both": np.ones_like(team, bool)}[who].astype(np.uint8)
    ctl_d = None if who == "both" else torch.from_numpy(ctl).to(gpu.device)
    pol = I.policy(tier, seed)
    gpu.prime_scripted(pol, ctl_d)
    hist = np.zeros(8, np.int64)
    dones = 0
    for s in range(steps):
        where = f"{w.name} E={E} scripted {tier}/{who} step {s}: "
        a = I.actions_for_step(w.seed, s, E, N)
        ad = torch.from_numpy(a).to(gpu.device)
        ref.heuristic_actions(pol, ctl, a)               # decides on the current state
        torch.cuda.synchronize()
        _check_memory(gpu, ref, E, N, where + "before the step: ")
        deciding = (ctl == 1) & (ref.st["alive"] == 1)
        waiting = gpu.mem["next_action"].cpu().numpy().reshape(E, N)
        assert np.array_equal(waiting[deciding], a[deciding]), where + "waiting decisions"
        ref.step(a)
        ref.mem["mem_valid"][ref.dones.astype(bool)] = 0
        ref.observe()
        gpu.scripted_step_observe(pol, ctl_d, ad)
        torch.cuda.synchronize()
        got = ad.cpu().numpy()
        assert np.array_equal(got, a), where + f"actions differ at {np.argwhere(got != a)[:4].tolist()}"
        compare_state(gpu.state_numpy(), ref.st, where)
        compare_outputs(gpu, ref, where, check_obs=True)
        if global_state:
            assert np.array_equal(gpu.gs_live.cpu().numpy(), ref.global_state()), where + "global state"
        hist += np.bincount(a[ctl == 1], minlength=8)
        dones += int(ref.dones.sum())
    return hist, dones


@pytest.mark.parametrize("tier", TIERS)
def test_scripted_tick_every_tier(tier):
    _say(f"[gpu] scripted tick c3 subset, adversaries, tier {tier}")
    hist, dones = _scripted_rollout(I.WORKLOADS["c3_16384env_10v10"], 48, 120, tier,
                                    "adversaries", max_steps=96)
    _say(f"[gpu]   action histogram {hist.tolist()} episodes ended {dones}")
    assert hist.sum() > 0


@pytest.mark.parametrize("name,E,steps,over", [
    ("c1_16env_3v3", 16, 256, dict()),
    ("c2_4096env_5v5", 200, 200, dict(max_steps=128)),
    ("c3_16384env_10v10", 70, 200, dict(max_steps=128)),
    ("c3e_16384env_10v10_ellipses", 70, 200, dict(max_steps=128)),
    ("c5_1024env_64v64", 3, 80, dict(max_steps=60)),
    ("c3_16384env_10v10", 40, 150, dict(max_steps=24, hurtbox_cone=1, hit_all=1)),
], ids=lambda v: v if isinstance(v, str) else None)
def test_scripted_tick_self_play(name, E, steps, over):
    _say(f"[gpu] scripted tick self-play {name} E={E} steps={steps} {over}")
    hist, dones = _scripted_rollout(I.WORKLOADS[name], E, steps, "expert", "both", **over)
    _say(f"[gpu]   action histogram {hist.tolist()} episodes ended {dones}")
    assert hist[5] > 0 and hist[1:5].sum() > 0 and hist[6:].sum() > 0
    assert dones > 0


def test_scripted_tick_roster_and_ragged():
    names = list(I.ROSTER)
    E, N = 40, 2 * len(names)
    w = I.Workload("roster_scripted", E, len(names), 48.0, 24, "iid", 0.5, "iid", steps=150,
                   seed=778)
    sc = I.make_scenario(w, E)
    for u in range(N):
        row = I.ROSTER[names[u % len(names)]]
        for k, v in zip(("hmax", "radius", "mass", "speed", "dmg", "range", "cooldown"), row):
            sc[k][:, u] = np.float32(v)
        sc["hurt_halfwidth"][:, u] = np.float32(row[1])
    _say("[gpu] scripted tick roster mix")
    hist, dones = _scripted_rollout(w, E, 150, "medium", "both", scenario=sc, max_steps=120)
    assert hist[5] > 0
    for team_size, disabled in [(1, 0), (7, 2), (33, 4), (50, 9)]:
        w = I.Workload(f"ragged_scripted_{team_size}", 5, team_size, 40.0, 20, "iid", 0.6, "iid",
                       steps=60, seed=6262 + team_size)
        sc = I.make_scenario(w, 5)
        rng = np.random.default_rng(team_size)
        for e in range(5):
            off = rng.choice(w.num_units, size=min(disabled, w.num_units - 2), replace=False)
            off = [u for u in off if u not in (0, w.num_units - 1)]
            sc["enabled"][e, off] = 0
        _say(f"[gpu] scripted tick ragged N={w.num_units} disabled={disabled}")
        _scripted_rollout(w, 5, 60, "advanced", "adversaries", scenario=sc, max_steps=40)
