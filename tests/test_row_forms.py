"""Which form of the row writers the GPU tests of these forms select (host only): a moved threshold must not leave
a form without its test."""
import ctypes as C

import pytest

from paper_2602_01665_amd import binding as B
from paper_2602_01665_amd import inputs as I
from tests import test_gpu_global_stream as stream
from tests import test_gpu_shared_lines as shared
from tests import test_pace as pace

NONE, OWN, SHARED, CARRIED = -1, 0, 1, 2        # TabxRowForm.lines


def _form(N, Z, E, call="step_observe", **over):
    return B.tabx_row_form(B.make_params(I.custom_params(N, 40.0, 0, Z, num_envs=E, **over)), call)


def test_errors_and_calls_without_rows():
    form = B.TabxRowForm()
    p = B.make_params(I.custom_params(20, 40.0, 0, 8, num_envs=4000))
    assert B._lib.tabx_row_form(C.byref(p), 7, C.byref(form)) == -2
    assert B._lib.tabx_row_form(C.byref(p), 3, None) == -1
    assert B._lib.tabx_row_form(None, 3, C.byref(form)) == -1
    for call in ("reset", "step", "heuristic_actions"):
        assert B.tabx_row_form(p, call) == dict(lines=NONE, pace=0, wavefronts_per_simd=-1, streams_global_state=0), call


SHARED_ONLY = {(20, 3, 1901), (20, 5, 2500), (60, 9, 401), (10, 1, 17003), (4, 7, 56001), (2, 1, 300007)}
IN_REGISTERS = {(72, 2, 700)}


def test_ticks_with_shared_lines():
    for team, Z, E in shared.BIG:
        key = (2 * team, Z, E)
        want = SHARED if key in SHARED_ONLY else NONE if key in IN_REGISTERS else CARRIED
        assert _form(*key)["lines"] == want, key


def test_other_calls_with_shared_lines():
    assert [_form(2 * t, Z, E, "observe")["lines"] for t, Z, E in shared.OBSERVED] == \
        [CARRIED, SHARED, CARRIED, CARRIED, CARRIED]
    assert [_form(2 * t, Z, E, "scripted_step_observe")["lines"] for t, Z, E in shared.SCRIPTED] == \
        [SHARED, CARRIED, CARRIED, CARRIED, CARRIED, CARRIED]
    assert [_form(N, Z, E)["lines"] for N, Z, E in shared.ODD] == \
        [SHARED, SHARED, CARRIED, CARRIED, CARRIED, SHARED, SHARED, SHARED]


def test_policy_ticks_and_rows_off_a_line():
    assert [_form(2 * t, Z, E, "policy_step_observe")["lines"] for t, Z, E in shared.POLICY] == \
        [SHARED, CARRIED, SHARED, SHARED, CARRIED, CARRIED, CARRIED]
    for call, fourth in (("step_observe", OWN), ("scripted_step_observe", SHARED)):
        assert [_form(N, Z, E, call)["lines"] for N, Z, E in shared.OFF_LINES] == \
            [SHARED, CARRIED, SHARED, fourth, OWN, CARRIED, OWN, NONE, SHARED]


@pytest.mark.parametrize("call", ["step_observe", "scripted_step_observe", "policy_step_observe", "observe"])
def test_lines_are_handed_on_only_between_tiles_of_one_wavefront(call):
    """Ticks of odd numbers of units up to 20 deal their tiles in turn, and a wavefront with one tile has nobody to
    hand a line on to."""
    handed_on = 0
    for N in range(1, 65):
        for Z in (0, 1, 3, 7, 8):
            for E in (2001, 5003, 12001, 60001, 300007):
                if 4 * N * (16 * N + 6 * Z) * E > 4e9:
                    continue
                info = B.tabx_launch_info(B.make_params(I.custom_params(N, 40.0, 0, Z, num_envs=E)), call)
                if _form(N, Z, E, call)["lines"] != CARRIED:
                    continue
                handed_on += 1
                assert call == "observe" or N % 2 == 0 or N > 20, (N, Z, E)
                share = info["workgroups"] // (8 * -(-E // (8 * info["envs_per_workgroup"])))   # per env group
                tiles = -(-info["envs_per_workgroup"] * N // info["rows_per_flush"])
                assert -(-tiles // share) > info["wavefronts_per_env_group"], (N, Z, E, info)
    assert handed_on > 50


def test_paced_launches():
    for team, Z, E, over in pace.PACED:
        # (33v33 with 7: rows that end on half a chunk, of two wavefronts, do not reach the pace in tiles)
        assert (_form(2 * team, Z, E, **over)["pace"] > 0) == ((team, Z, E) != (33, 7, 1000)), (team, Z, E)
    for team, Z, E in pace.SCRIPTED:
        assert _form(2 * team, Z, E, "scripted_step_observe")["pace"] > 0, (team, Z, E)


@pytest.mark.parametrize("N,Z,E,paced", [
    (20, 8, 1698, False), (20, 8, 1699, True), (64, 0, 190, False), (64, 0, 191, True),      # 50 MB of rows
    (20, 8, 6144, True), (20, 8, 6145, False), (64, 0, 1280, True), (64, 0, 1281, False),    # one generation
    (32, 0, 1024, False), (32, 0, 1025, True),                   # flushes per wavefront
    (128, 0, 670, False), (128, 0, 671, True)])                  # two wavefronts, units in registers
def test_edges_of_the_pace(N, Z, E, paced):
    assert (_form(N, Z, E)["pace"] > 0) == paced


@pytest.mark.parametrize("N,Z,E,lines,paced", [
    (100, 2, 518, NONE, False), (100, 2, 488, SHARED, False), (100, 2, 489, CARRIED, True), (100, 2, 300, SHARED, False),
    (128, 2, 382, SHARED, False), (128, 2, 383, CARRIED, True),
    (128, 3, 319, CARRIED, False), (80, 1, 300, CARRIED, False), (128, 0, 319, OWN, True)])
def test_tiles_of_two_wavefronts(N, Z, E, lines, paced):
    form = _form(N, Z, E)
    assert (form["lines"], form["pace"] > 0) == (lines, paced), form


@pytest.mark.parametrize("N,Z,E,held", [
    (66, 0, 1280, 4), (66, 0, 1281, 3), (66, 0, 1536, 3), (66, 0, 1537, 4), (66, 0, 2048, 4), (66, 0, 2049, 3),
    (66, 0, 3072, 3), (66, 0, 3073, 4), (128, 0, 1024, 4), (100, 0, 1500, 3)])
def test_units_in_registers_three_or_four_wavefronts_per_simd(N, Z, E, held):
    for call in ("step_observe", "scripted_step_observe", "policy_step_observe"):
        assert _form(N, Z, E, call)["wavefronts_per_simd"] == held, call


def test_units_in_registers_half_a_chunk():
    """Only the plain launches need the kernel with three for such rows."""
    for E, scripted in ((1025, 4), (1281, 3), (2048, 4)):
        forms = [_form(66, 7, E, c)["wavefronts_per_simd"] for c in ("step_observe", "observe", "scripted_step_observe")]
        assert forms == [3, 3, scripted], E


@pytest.mark.parametrize("N,Z,E,lines,paced", [
    # 1.5 us of HBM per tile of each wavefront, whole chunks and more than eight tiles 1.25; one generation
    (20, 4, 2725, SHARED, True), (20, 4, 2726, CARRIED, True), (30, 2, 1219, SHARED, True), (30, 2, 1220, CARRIED, True),
    (20, 5, 3214, SHARED, True), (20, 5, 3215, CARRIED, True), (60, 4, 304, SHARED, True), (60, 4, 305, CARRIED, True),
    (53, 7, 667, SHARED, True), (53, 7, 668, CARRIED, True),
    # several generations
    (22, 2, 7000, CARRIED, False),
    # the pace: 1.2 us, tiles that start on lines 1.0
    (20, 4, 2616, SHARED, False), (20, 4, 2617, SHARED, True), (26, 0, 1802, OWN, False), (26, 0, 1803, OWN, True)])
def test_wavefronts_that_hbm_waits_for(N, Z, E, lines, paced):
    form = _form(N, Z, E)
    assert (form["lines"], form["pace"] > 0) == (lines, paced), form


def test_shared_lines_of_two_wavefronts_are_never_paced():
    """Their kernels leave the pace out."""
    shared_lines = 0
    for N in range(65, 129):
        for Z in (0, 1, 2, 3, 7, 16):
            for E in (200, 300, 400, 512, 513, 700, 1000):
                for call in ("step_observe", "scripted_step_observe", "policy_step_observe", "observe"):
                    form = _form(N, Z, E, call)
                    if form["lines"] == SHARED:
                        shared_lines += 1
                        assert form["pace"] == 0, (N, Z, E, call)
    assert shared_lines > 500


def test_streamed_global_states():
    for team, Z, E, fused, levels in stream.STREAMED:
        over = dict(num_levels=levels) if levels else {}
        call = "step_observe" if fused else "observe"
        assert _form(2 * team, Z, E, call, **over)["streams_global_state"] == 1, (team, Z, E)
    assert _form(20, 8, 14000)["streams_global_state"] == 0
    for call, cases in (("scripted_step_observe", stream.SCRIPTED), ("policy_step_observe", stream.POLICY)):
        for team, Z, E in cases:
            assert _form(2 * team, Z, E, call)["streams_global_state"] == int((team, Z, E) not in stream.STORED), (call, team, Z, E)


def test_a_part_of_a_batch_is_not_held_to_a_pace():
    """Its launch shares the machine with the other parts': a workgroup of it may start late."""
    for team, Z, E, over in pace.PACED:
        p = B.make_params(I.custom_params(2 * team, 40.0, 0, Z, num_envs=2 * E, **over))
        for first, count, part in ((0, E, True), (E, E, True), (0, 2 * E, False)):
            mine = B.tabx_part(p, B.TabxScenario(), B.TabxState(), first, count)[0]
            assert mine.shared_machine == int(part)
            held = B.tabx_row_form(mine, "step_observe")["pace"] > 0
            if part:
                assert held == (2 * team > 64 and (team, Z, E) != (33, 7, 1000)), (team, Z, E)
    p.shared_machine = 1                        # (a part of a part, and a caller's own setting)
    assert B.tabx_part(p, B.TabxScenario(), B.TabxState(), 0, p.num_envs)[0].shared_machine == 1
