"""Launches of one generation of workgroups are held to a common pace (plan_pace, tabx_kernels.hip): every form
of the rows at a size that is paced, against the checker, and what the rule takes for granted of the kernels."""
import re

import pytest

from paper_2602_01665_amd import inputs as I
from paper_2602_01665_amd.binding import make_params, tabx_launch_info
from tests.test_gpu_parity import _rollout
from tests.test_gpu_policy import _scripted_rollout
from tests.test_gpu_row_forms import _scene
from tests.test_kernel_resources import kernels  # noqa: F401  (the module's fixture)


def _kernel(waves, policy, step, scripted, twin, even):
    return "tabx_tick_kernelILi%dELb%dELb%dELb1ELb%dELi%dELb%dE" % (waves, policy, step, scripted, twin, even)


# kernel, and how many of its wavefronts a SIMD holds
HELD = [
    (_kernel(1, 0, 1, 0, 0, 0), 3), (_kernel(1, 1, 1, 0, 0, 0), 3),
    (_kernel(1, 0, 0, 0, 2, 0), 5), (_kernel(1, 0, 1, 0, 2, 0), 5), (_kernel(1, 0, 1, 0, 4, 0), 5),
    (_kernel(1, 0, 1, 0, 8, 0), 5), (_kernel(1, 1, 1, 0, 2, 0), 5), (_kernel(1, 0, 1, 1, 2, 0), 4),
    (_kernel(1, 0, 1, 1, 4, 0), 4), (_kernel(1, 0, 1, 1, 8, 0), 4),
    (_kernel(2, 0, 0, 0, 0, 0), 4), (_kernel(2, 0, 1, 0, 0, 0), 4), (_kernel(2, 1, 1, 0, 0, 0), 4),
    (_kernel(2, 0, 1, 1, 0, 0), 4), (_kernel(2, 0, 0, 0, 0, 1), 3), (_kernel(2, 0, 1, 0, 0, 1), 3),
    (_kernel(2, 1, 1, 0, 0, 1), 3), (_kernel(2, 0, 1, 0, 2, 0), 5), (_kernel(2, 0, 1, 0, 3, 0), 5),
    (_kernel(2, 1, 1, 0, 2, 0), 5), (_kernel(2, 0, 1, 1, 2, 0), 4), (_kernel(2, 0, 1, 1, 3, 0), 4),
    (_kernel(2, 0, 0, 0, 2, 0), 5), (_kernel(2, 0, 0, 0, 3, 0), 5), (_kernel(2, 0, 1, 1, 0, 1), 3),
]


def test_wavefronts_a_simd_holds(kernels):  # noqa: F811
    """512 vector registers per lane and SIMD, given out in eights."""
    registers = {name: int(re.search(r"\.vgpr_count:\s+(\d+)", meta).group(1)) for name, meta in kernels[0]}
    for part, held in HELD:
        (count,) = [v for k, v in registers.items() if part in k]
        assert 512 // (-(-count // 8) * 8) == held, (part, count)


def test_scripted_tiles_of_two_wavefronts_need_no_fifth(kernels):  # noqa: F811
    """Four per SIMD are all that the CUs' LDS or the batch ask for: a fifth, which fewer than 97 registers would
    allow, is never there."""
    text = kernels[1]
    seen = 0
    for N in range(65, 129):
        for Z in (0, 1, 2, 3, 7, 16):
            for E in (64, 300, 512, 513, 900):
                info = tabx_launch_info(make_params(I.custom_params(N, 40.0, 0, Z, num_envs=E)), "scripted_step_observe")
                w = info["wavefronts_per_env_group"]
                if w == 2:
                    continue
                name = _kernel(2, 0, 1, 1, w // 2, 0)
                static = int(re.search(r"\.amdhsa_kernel \w*" + name + r"\w*\n\s+\.amdhsa_group_segment_fixed_size (\d+)",
                                       text).group(1))
                block = -(-(static + info["dynamic_lds_bytes"]) // 1280) * 1280
                assert min(160 * 1024 // block, -(-E // 256)) * w <= 16, (N, Z, E, w, block)
                seen += 1
    assert seen > 500


PACED = [
    # team size, zone slots, envs, overrides
    (10, 8, 4000, {}), (12, 3, 3000, {}), (16, 0, 1300, {}), (32, 0, 500, {}),   # tiles: two, four, eight wavefronts
    (40, 0, 400, {}), (33, 7, 1000, {}), (64, 2, 400, {}),                       # ... of envs of two
    (40, 0, 1200, {}), (33, 7, 1400, {}),                                        # two wavefronts, units in registers
    (10, 8, 8192, dict(collision_alpha=0.8)),                                    # one
]


@pytest.mark.gpu
@pytest.mark.parametrize("team,zones,E,over", PACED)
def test_paced_rows(team, zones, E, over):
    w, sc = _scene(team, zones, E)
    print(f"[gpu] paced N={2 * team} Z={zones} E={E} {over}", flush=True)
    _rollout(w, E, 2, True, scenario=sc, max_steps=5, **over)


SCRIPTED = [(10, 8, 4000), (40, 0, 1200)]


@pytest.mark.gpu
@pytest.mark.parametrize("team,zones,E", SCRIPTED)
def test_paced_rows_with_deciding_units(team, zones, E):
    w, sc = _scene(team, zones, E)
    print(f"[gpu] paced scripted N={2 * team} Z={zones} E={E}", flush=True)
    _scripted_rollout(w, E, 2, "medium", "adversaries", scenario=sc, max_steps=4)
