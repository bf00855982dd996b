"""Rows whose tiles share 128-byte lines (LINES in write_rows, tabx_observe.h): rows of whole and of half chunks at
every place within a line, one and two passes per tile, runs and tiles taken in turn, envs of one and two wavefronts,
partial last groups, and batches on either side of the rules that choose the form; every env against the checker."""
import pytest

from paper_2602_01665_amd import inputs as I
from tests.test_gpu_parity import _rollout
from tests.test_gpu_policy import _policy_rollout, _scripted_rollout
from tests.test_gpu_row_forms import _scene
from tests.test_launch_forms import _waves

BIG = [
    # team size, zone slots, envs (50 MB of rows and more)
    (10, 3, 1901), (10, 4, 2003), (10, 3, 10001), (10, 5, 2500), (16, 5, 1000), (16, 1, 1801), (15, 5, 4801), (12, 2, 2503),
    (11, 7, 2001), (32, 3, 390), (24, 4, 803), (30, 9, 401), (5, 3, 8003), (5, 1, 17003), (2, 7, 56001), (1, 1, 300007),
    (33, 7, 601), (50, 3, 520), (36, 2, 700), (10, 5, 4001)]
OBSERVED = [(5, 3, 8003), (5, 3, 40001), (8, 1, 6001), (11, 7, 2001), (33, 7, 601)]
SCRIPTED = [(10, 5, 2500), (16, 5, 4100), (24, 4, 803), (33, 3, 700), (28, 2, 801), (10, 5, 4001)]
# units, zone slots, envs
ODD = [(9, 7, 12001), (17, 7, 3001), (21, 3, 2501), (23, 7, 2001), (31, 1, 1001), (17, 0, 9001), (3, 9, 40001), (1, 3, 400009)]


def _scripted(team, zones, E):
    w, sc = _scene(team, zones, E)
    _scripted_rollout(w, E, 2, "medium", "adversaries", scenario=sc, max_steps=4)


@pytest.mark.gpu
@pytest.mark.parametrize("team,zones,E", BIG)
def test_ticks(team, zones, E):
    w, sc = _scene(team, zones, E)
    print(f"[gpu] shared lines N={2 * team} Z={zones} E={E}", flush=True)
    _rollout(w, E, 2, True, scenario=sc, max_steps=5)


@pytest.mark.gpu
@pytest.mark.parametrize("team,zones,E", OBSERVED)
def test_observe(team, zones, E):
    w, sc = _scene(team, zones, E)
    print(f"[gpu] shared lines, observe N={2 * team} Z={zones} E={E}", flush=True)
    _rollout(w, E, 1, False, scenario=sc, max_steps=5)


@pytest.mark.gpu
@pytest.mark.parametrize("team,zones,E", SCRIPTED)
def test_scripted(team, zones, E):
    print(f"[gpu] shared lines, scripted N={2 * team} Z={zones} E={E}", flush=True)
    _scripted(team, zones, E)


@pytest.mark.gpu
@pytest.mark.parametrize("N,Z,E", ODD)
def test_odd_numbers_of_units(N, Z, E):
    """Against the same rows in a batch too small for any of the rules."""
    import torch
    from paper_2602_01665_amd.binding import TabxEnv
    few = 7
    print(f"[gpu] shared lines N={N} Z={Z} E={E}", flush=True)
    w, sc = _scene(max(N // 2 + 1, 1), Z, E)
    w2 = 2 * (N // 2 + 1)
    sc = {k: (v[:, :N].copy() if getattr(v, "ndim", 0) == 2 and v.shape[1] == w2 else v) for k, v in sc.items()}
    p = I.custom_params(N, w.map_size, w.grid, Z, num_envs=E)
    env = TabxEnv(p, sc)
    env.reset()
    acts = torch.randint(0, 6, (E, N), dtype=torch.uint8, device=env.device, generator=torch.Generator(env.device).manual_seed(1))
    for _ in range(2):
        env.step_observe(acts)
    for first in (0, E // 2 // few * few, E - few):
        part = {k: (v[first:first + few].copy() if getattr(v, "ndim", 0) and v.shape[0] == E else v) for k, v in sc.items()}
        one = TabxEnv(I.custom_params(N, w.map_size, w.grid, Z, num_envs=few), part)
        one.reset()
        for _ in range(2):
            one.step_observe(acts[first:first + few].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(env.obs[first:first + few], one.obs), first
        assert torch.equal(env.vis[first:first + few], one.vis), first


# the policy as a scan stage
POLICY = [(10, 3, 3501), (15, 5, 4801), (11, 7, 2001), (32, 3, 1001), (33, 3, 700), (8, 7, 6007), (17, 1, 9001)]


@pytest.mark.gpu
@pytest.mark.parametrize("team,zones,E", POLICY)
def test_policy(team, zones, E):
    w, sc = _scene(team, zones, E)
    print(f"[gpu] shared lines, policy N={2 * team} Z={zones} E={E}", flush=True)
    _policy_rollout(w, E, 2, "medium", "adversaries", scenario=sc, fused=True, max_steps=4)


# tiles that start on lines, share them, hand them on; units in registers; of envs of one and of two wavefronts
OFF_LINES = [(20, 8, 2501), (20, 7, 4001), (20, 3, 1901), (24, 4, 803), (10, 0, 9001), (66, 7, 601), (128, 0, 40),
             (66, 0, 700), (17, 7, 3001)]


@pytest.mark.gpu
@pytest.mark.parametrize("call", ["step_observe", "scripted_step_observe"])
@pytest.mark.parametrize("off", [4, 8, 20, 28])
@pytest.mark.parametrize("N,Z,E", OFF_LINES)
def test_rows_that_start_off_a_line(N, Z, E, off, call):
    """`obs` needs 16 bytes: the same rows 16 ... 112 bytes off a 128-byte line, and nothing written beside them.
    (Parts of a batch start there: 17 units with 7 slots, a part of a multiple of four envs.)"""
    import torch
    from paper_2602_01665_amd.binding import TabxEnv
    print(f"[gpu] obs {4 * off} bytes off a line, {call} N={N} Z={Z} E={E}", flush=True)
    _, sc = _scene((N + 1) // 2, Z, E)
    sc = {k: (v[:, :N].copy() if getattr(v, "ndim", 0) == 2 else v) for k, v in sc.items()}
    p = I.custom_params(N, 40.0, 20, Z, num_envs=E)
    on, beside = TabxEnv(p, sc), TabxEnv(p, sc)
    assert on.obs.data_ptr() % 128 == 0
    pad = torch.full((on.obs.numel() + 64,), 7.5, device=on.device)
    assert pad.data_ptr() % 128 == 0
    beside.obs = pad[32 + off:32 + off + on.obs.numel()].view_as(on.obs)
    acts = torch.randint(0, 8, (E, N), dtype=torch.uint8, device=on.device, generator=torch.Generator(on.device).manual_seed(2))
    pol = I.policy("medium", 3)
    for env in (on, beside):
        env.reset()
        env.prime_scripted(pol, None)
        for _ in range(2):
            if call == "step_observe":
                env.step_observe(acts)
            else:
                env.scripted_step_observe(pol, None, acts.clone())
    torch.cuda.synchronize()
    assert torch.equal(on.obs, beside.obs) and torch.equal(on.vis, beside.vis)
    assert bool((pad[:32 + off] == 7.5).all()) and bool((pad[32 + off + on.obs.numel():] == 7.5).all())


@pytest.mark.parametrize("N,Z,E,tick,scripted", [(56, 2, 800, 4, 4), (24, 4, 2048, 4, 4), (24, 4, 2049, 2, 2), (23, 7, 2000, 4, 4),
                                                 (20, 5, 3000, 2, 2), (48, 0, 1000, 4, 2), (24, 16, 2000, 2, 2)])
def test_wavefronts(N, Z, E, tick, scripted):
    assert (_waves(N, Z, E, "step_observe"), _waves(N, Z, E, "scripted_step_observe")) == (tick, scripted)
