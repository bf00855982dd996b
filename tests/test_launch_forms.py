"""Which form of a launch a batch gets (host only): the GPU tests of the forms mean what they say only as
long as their shapes select them, and a rule of a dispatch lies where both sides were measured."""
import pytest

from paper_2602_01665_amd import binding as B
from paper_2602_01665_amd import inputs as I
from tests import test_gpu_row_forms as rows


def _info(N, Z, E, call, **over):
    return B.tabx_launch_info(B.make_params(I.custom_params(N, 40.0, 0, Z, num_envs=E, **over)), call)


def _waves(N, Z, E, call, **over):
    info = _info(N, Z, E, call, **over)
    assert info["threads_per_workgroup"] == 64 * info["wavefronts_per_env_group"]
    return info["wavefronts_per_env_group"]


# units, zone slots, envs: wavefronts per env group of observe, the tick, the scripted and the policy tick
TWO = [
    (128, 0, 64, 6, 6, 6, 4), (128, 0, 256, 6, 6, 6, 4), (128, 0, 257, 4, 4, 4, 4),
    (128, 0, 512, 4, 4, 4, 4), (128, 0, 513, 2, 2, 2, 2), (127, 0, 64, 6, 6, 6, 4),
    (66, 0, 512, 6, 6, 6, 4), (66, 0, 513, 2, 2, 2, 2), (66, 7, 512, 6, 6, 6, 4),
    (66, 7, 513, 4, 4, 4, 4), (66, 7, 1024, 4, 4, 4, 4), (66, 7, 1025, 2, 2, 2, 2),
    (100, 0, 300, 6, 6, 6, 4), (100, 0, 400, 4, 4, 4, 4), (127, 1, 600, 2, 2, 2, 2),
    (128, 16, 3, 4, 4, 4, 4),                  # (six staging areas would not fit a workgroup's LDS)
]


@pytest.mark.parametrize("N,Z,E,observe,tick,scripted,policy", TWO)
def test_envs_of_two_wavefronts(N, Z, E, observe, tick, scripted, policy):
    got = [_waves(N, Z, E, c) for c in ("observe", "step_observe", "scripted_step_observe", "policy_step_observe")]
    assert got == [observe, tick, scripted, policy]


# the same of envs of at most 64 units
ONE = [
    (64, 0, 200, 1, 8, 8, 1), (32, 1, 3, 2, 8, 4, 2), (33, 0, 200, 1, 8, 8, 1), (33, 0, 300, 1, 8, 4, 1), (33, 0, 513, 1, 4, 4, 1), (22, 0, 500, 1, 8, 4, 1), (20, 0, 500, 1, 4, 4, 1),
    (20, 8, 700, 1, 4, 4, 1), (20, 8, 16384, 1, 2, 2, 1), (10, 0, 65536, 1, 1, 2, 1),
    (16, 3, 9, 2, 4, 4, 2), (20, 7, 200, 2, 4, 4, 2), (2, 16, 8200, 2, 2, 2, 2),
]


@pytest.mark.parametrize("N,Z,E,observe,tick,scripted,policy", ONE)
def test_envs_of_one_wavefront(N, Z, E, observe, tick, scripted, policy):
    got = [_waves(N, Z, E, c) for c in ("observe", "step_observe", "scripted_step_observe", "policy_step_observe")]
    assert got == [observe, tick, scripted, policy]


@pytest.mark.parametrize("N,Z,E,envs", [
    (4, 16, 64, 2), (4, 16, 4096, 2), (4, 16, 4097, 16), (8, 16, 2048, 2), (8, 16, 2049, 8), (9, 12, 2304, 3),
    (9, 12, 2305, 7), (10, 8, 4096, 6), (2, 16, 8192, 4), (2, 16, 20000, 32), (1, 16, 16384, 8),
    (1, 16, 16385, 64), (20, 8, 64, 3), (64, 16, 64, 1)])
def test_envs_of_a_wavefront(N, Z, E, envs):
    """As many as the lanes hold, unless the zone chunks are more than the lanes and the batch is small."""
    for call in ("reset", "step", "observe", "step_observe", "heuristic_actions", "scripted_step_observe"):
        info = _info(N, Z, E, call)
        assert info["envs_per_workgroup"] == envs, (call, info)
        assert info["workgroups"] * envs >= E


@pytest.mark.parametrize("N,E,rows_", [(40, 400, 1), (40, 600, 1), (24, 800, 4), (24, 1400, 2), (24, 500, 2),
                                       (20, 1200, 3), (20, 16384, 6), (64, 1536, 2), (64, 1280, 1)])
def test_rows_of_a_tile(N, E, rows_):
    assert _info(N, 0, E, "step_observe")["rows_per_flush"] == rows_


@pytest.mark.parametrize("N,Z,E,waves,rows_", [(20, 8, 700, 2, 6), (20, 8, 4000, 2, 3), (24, 8, 500, 4, 4), (32, 8, 6000, 4, 4),
                                               (43, 5, 100, 8, 1), (8, 4, 2000, 2, 16)])
def test_elliptical_zones(N, Z, E, waves, rows_):
    info = _info(N, Z, E, "step_observe", zone_shapes=1)
    assert (info["wavefronts_per_env_group"], info["rows_per_flush"]) == (waves, rows_), info


@pytest.mark.parametrize("N,share", [(10, 3), (19, 5), (20, 3), (31, 8), (32, 4), (33, 7), (5, 3)])
def test_workgroups_that_share_an_observe(N, share):
    groups = -(-3000 // (64 // N))
    assert _info(N, 0, 3000, "observe")["workgroups"] == share * 8 * -(-groups // 8)


def test_every_form_has_a_gpu_test():
    """The shapes of the GPU tests of the rows between them select every number of wavefronts (a single one
    for a plain tick is in test_gpu_parity's own list)."""
    ticks = {(2 * t > 64, _waves(2 * t, z, E, "step_observe")) for t, z, E, _ in rows.TICKS}
    assert ticks >= {(False, 2), (False, 4), (False, 8), (True, 2), (True, 4), (True, 6)}
    alone = {(2 * t > 64, _waves(2 * t, z, E, "observe")) for t, z, E, _ in rows.TICKS}
    assert alone >= {(False, 1), (False, 2), (True, 2), (True, 4), (True, 6)}
    for call, want in (("scripted_step_observe", {(False, 2), (False, 4), (False, 8), (True, 2), (True, 4), (True, 6)}),
                       ("policy_step_observe", {(False, 1), (False, 2), (True, 2), (True, 4)})):
        assert {(2 * t > 64, _waves(2 * t, z, E, call)) for t, z, E, _ in rows.DECIDING} >= want


def test_divisions_by_multiplication_are_exact():
    """What a workgroup divides (by units per env, zone chunks, rows per pass, chunks of a row's tail), for
    every shape and the largest dividend each occurs with."""
    def exact(n, largest):
        magic = (65536 + n - 1) // n
        return all((x * magic) >> 16 == x // n for x in range(largest + 1))

    for N in range(1, 65):
        G = 64 // N
        assert exact(N, 63)
        for Z in range(17):
            D, ZC = 16 * N + 6 * Z, (6 * Z + 3) // 4
            S = max(1, min(G, 1280 // D))
            assert exact(S, 63)
            assert exact(4 + ZC, max(63, 2 * S * (4 + ZC) - 1))
            if ZC:
                assert exact(ZC, G * ZC - 1)


@pytest.mark.parametrize("call", ["observe", "step_observe", "scripted_step_observe", "policy_step_observe"])
def test_every_shape_fits_a_workgroup(call):
    """Dynamic LDS plus the most a kernel has besides (12 KB) within what a workgroup may take."""
    for N in range(1, 129):
        for Z in (0, 1, 2, 7, 8, 15, 16):
            for E in (1, 300, 700, 3000, 20000):
                for shapes in (0, 1) if Z else (0,):
                    info = _info(N, Z, E, call, zone_shapes=shapes)
                    static = 11648 if N > 64 else 5952
                    assert info["dynamic_lds_bytes"] + static <= info["assumed_lds_per_workgroup_bytes"], (N, Z, E, info)
