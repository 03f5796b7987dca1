"""Workspace sizes: what every call needs, and the records' room where they are taken."""
import pytest

import synth
from paper_2206_14735_amd import gosurf as G
from tests.test_record_plan_cpu import records_from


def _up(n):
    return (n + 255) // 256 * 256


@pytest.mark.parametrize("M,total", [(509, 509 * 91), (6144, 6144 * 96), (16384, 16384 * 96)])
def test_batches_without_records_pay_for_none(M, total):
    """32 bytes per sample and 36 per ray, and nothing for the pairs: a workspace
    asked for with fewer pairs serves a batch with more."""
    model = G.make_model(synth.configs.ROOM.layout())
    fixed = G.gosurf_workspace_bytes(model, 0, 0, 0)
    own = 2 * _up(16 * total) + _up(32 * M) + _up(4 * M)
    assert fixed < 60e6
    for S in (0, 16384, 65536):
        assert G.gosurf_workspace_bytes(model, M, total, S) == fixed + own
    assert G.lib().gosurf_workspace_bytes(None, M, total, 16384) == fixed + own


def test_batches_with_records_get_their_room():
    L = synth.configs.SPHERE.layout()
    model = G.make_model(L)
    line = records_from(L)
    M = 1024
    need = G.lib().gosurf_workspace_bytes(None, M, line, 0)
    assert G.gosurf_workspace_bytes(model, M, line - 1, 0) <= need
    assert G.gosurf_workspace_bytes(model, M, line, 0) >= need + 168 * line
    assert G.gosurf_workspace_bytes(model, M, line - 200, 100) >= need + 168 * line
    # the copies' room, which nothing uses, serves the records
    c = G.gosurf_workspace_bytes(G.make_model(L, grad_copies=True), M, line, 0)
    assert c == max(G.gosurf_workspace_bytes(model, M, line, 0),
                    need + G.gosurf_workspace_bytes(G.make_model(L, grad_copies=True), M, 1024, 0)
                    - G.gosurf_workspace_bytes(model, M, 1024, 0))
