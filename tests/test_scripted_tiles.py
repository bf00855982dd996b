"""A scripted tick's rows by four wavefronts, two passes per tile: which batches get the form, and the form at
its edges (the first and last batch of a rule, partial last groups, rows that end on half a chunk, uneven shares)
against the checker."""
import pytest

from tests.test_gpu_policy import _scripted_rollout
from tests.test_gpu_row_forms import _scene
from tests.test_launch_forms import _info


@pytest.mark.parametrize("N,Z,E,waves,rows", [
    (32, 0, 4096, 2, 2), (32, 0, 4097, 4, 4), (40, 0, 2048, 2, 1), (40, 0, 2049, 4, 2), (33, 7, 2049, 4, 2),
    (30, 0, 5000, 2, 2), (64, 16, 3000, 4, 2), (32, 0, 768, 4, 4), (32, 0, 769, 4, 2), (40, 0, 512, 4, 2),
    (40, 0, 513, 4, 1), (64, 0, 384, 4, 2), (64, 0, 385, 4, 1), (22, 0, 500, 4, 2), (20, 8, 16384, 2, 3)])
def test_form(N, Z, E, waves, rows):
    info = _info(N, Z, E, "scripted_step_observe")
    assert (info["wavefronts_per_env_group"], info["rows_per_flush"]) == (waves, rows), info


@pytest.mark.gpu
@pytest.mark.parametrize("team,zones,E,ticks", [(16, 0, 4097, 2), (20, 3, 2049, 2), (16, 3, 767, 3), (20, 8, 300, 3),
                                                (32, 0, 384, 3), (15, 5, 601, 3)])
def test_rows(team, zones, E, ticks):
    w, sc = _scene(team, zones, E)
    print(f"[gpu] scripted tiles N={2 * team} Z={zones} E={E}", flush=True)
    _scripted_rollout(w, E, ticks, "medium", "adversaries", scenario=sc, max_steps=4)
