"""The policy scan marks the partners that may be in sight before it tests them: pairs that sit exactly on the edge
of the sight range or of the cone, coincident units, distances that underflow, cones and ranges without an
edge, for every way the lanes are dealt to the deciding units.  Actions and memories against the checker."""
import math

import numpy as np
import pytest

from paper_2602_01665_amd import inputs as I
from tests.test_gpu_policy import _check_memory

pytestmark = pytest.mark.gpu


def _edges(N, E, seed):
    rng = np.random.default_rng(seed)
    w = I.Workload(f"edges_{N}", E, (N + 1) // 2, 24.0, 0, "none", 1.0, "iid", seed=seed)
    sc = {k: (v if v is None or v.ndim != 2 else np.ascontiguousarray(v[:, :N])) for k, v in I.make_scenario(w, E).items()}
    f = np.float32
    span = 4 + int(math.sqrt(N) * 1.5)                       # whole numbers: 3-4-5 triangles, coincident units
    for k in ("init_x", "init_y"):
        v = rng.integers(0, span, (E, N)).astype(f)
        tiny = rng.choice(np.array([1e-45, 1e-38, 3e-23, 1e-20, 1e-15], f), (E, N))
        sc[k] = np.where((v == 0) & (rng.random((E, N)) < 0.5), tiny, v).astype(f)
    turn = np.concatenate([np.arange(4) * (math.pi / 2), [math.atan2(3, 4), math.atan2(4, 3), 0.1, 5.9]]).astype(f)
    sc["init_theta"] = rng.choice(turn, (E, N))
    sc["sight_range"] = rng.choice(np.array([0.0, 1.0, 5.0, 10.0, math.sqrt(2), 1e-22, 3e38, math.inf], f), (E, N))
    sc["sight_cos_half"] = rng.choice(np.array([1.0, 0.8, 0.6, 0.5, math.sqrt(0.5), 0.0, -0.6, -1.0, 2.0, -2.0], f), (E, N))
    sc["team"] = (rng.random((E, N)) < 0.5).astype(np.uint8)
    return I.make_params(w, E, num_units=N), sc


@pytest.mark.parametrize("who", ["few", "half", "all"])
@pytest.mark.parametrize("N,E", [(1, 9), (4, 300), (9, 200), (20, 150), (31, 60), (33, 40), (64, 30), (66, 20), (128, 12)])
def test_marks_on_the_edges(N, E, who):
    import torch
    from oracle.ref import RefEnv
    from paper_2602_01665_amd.binding import TabxEnv
    p, sc = _edges(N, E, 91 + N)
    ref, gpu = RefEnv(p, sc), TabxEnv(p, sc)
    ref.reset()
    gpu.reset()
    ctl = (np.random.default_rng(N).random((E, N)) < dict(few=0.08, half=0.5, all=2.0)[who]).astype(np.uint8)
    print(f"[gpu] marks N={N} E={E} {who}", flush=True)
    for seed in (3, 4):
        pol = I.policy("expert", seed)
        a = np.full((E, N), 7, np.uint8)
        ad = torch.from_numpy(a.copy()).to(gpu.device)
        ref.heuristic_actions(pol, ctl, a)
        gpu.heuristic_actions(pol, torch.from_numpy(ctl).to(gpu.device), ad)
        torch.cuda.synchronize()
        bad = np.argwhere(ad.cpu().numpy() != a)
        assert bad.size == 0, f"N={N} {who}: actions differ at {bad[:5].tolist()}"
        _check_memory(gpu, ref, E, N, f"N={N} {who}: ")
