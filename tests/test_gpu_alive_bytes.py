"""A caller's own `alive` bytes (a restored or edited state): every non-zero byte means alive, in every
form of the rows and in the policy, as in the checker."""
import numpy as np
import pytest

from paper_2602_01665_amd import inputs as I
from tests.parity import compare_outputs, compare_state

pytestmark = pytest.mark.gpu


# team size, zone slots, envs: stand-alone rows from registers and in tiles, one and two wavefronts per env
@pytest.mark.parametrize("team,zones,E", [(10, 0, 40), (10, 3, 40), (33, 0, 5), (33, 0, 520)])
def test_any_nonzero_byte_is_alive(team, zones, E):
    import torch
    from oracle.ref import RefEnv
    from paper_2602_01665_amd.binding import TabxEnv
    w = I.Workload(f"alive_{team}_{zones}", E, team, 40.0, 20, "iid", 0.6, "iid", max_zones=zones, seed=61)
    p, sc = I.make_params(w, E, max_steps=50), I.make_scenario(w, E)
    N = w.num_units
    ref, gpu = RefEnv(p, sc), TabxEnv(p, sc, want_global_state=True)
    ref.reset()
    gpu.reset()
    rng = np.random.default_rng(team + zones + E)
    pol = I.policy("expert", 3)
    every = np.ones((E, N), np.uint8)
    for s in range(3):
        print(f"[gpu] alive bytes N={N} Z={zones} E={E} step {s}", flush=True)
        dead = ref.st["alive"] == 0
        ref.st["alive"][:] = np.where(dead, 0, rng.choice([1, 2, 3, 4, 64, 128, 254, 255], size=(E, N)))
        gpu.st["alive"].copy_(torch.from_numpy(ref.st["alive"].reshape(-1)))
        where = f"N={N} Z={zones} E={E} step {s}: "
        ref.observe()
        gpu.observe()
        torch.cuda.synchronize()
        compare_outputs(gpu, ref, where)
        assert np.array_equal(gpu.gs_live.cpu().numpy(), ref.global_state()), where + "global state"
        a = I.actions_for_step(w.seed, s, E, N)
        ad = torch.from_numpy(a).to(gpu.device)
        ref.heuristic_actions(pol, every, a)
        gpu.heuristic_actions(pol, None, ad)
        torch.cuda.synchronize()
        assert np.array_equal(ad.cpu().numpy(), a), where + "actions"
        ref.step(a)
        ref.observe()
        gpu.step_observe(ad)
        torch.cuda.synchronize()
        compare_state(gpu.state_numpy(), ref.st, where)
        compare_outputs(gpu, ref, where)
