"""The segments of a tile that the ring kernel sums by itself (fe_streamk_tile_segments runs the kernel's
code on the host) are those that the plan's workgroups hand to each other (fe_streamk_segments), in the
order in which the finishing workgroup adds them: its own first, then the published ones by workgroup."""
import ctypes
import os

import pytest

from paper_2605_08523_amd import api


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not os.path.exists(api.LIB_PATH):
        pytest.fail("libfe.so is not built (python -m paper_2605_08523_amd.build)")
    api.lib()


@pytest.mark.parametrize("schedule,grid", [(2, 512), (2, 608), (2, 160), (2, 16), (1, 256), (1, 80)])
def test_segments_are_the_plans(schedule, grid):
    tile = 256 if schedule == 1 else 128
    for np_ in list(range(tile, 3072 + 1, tile)) + [4096, 5888]:
        geom, _ = api.streamk_segments(np_, schedule, grid, 0)
        finish, handed = {}, {}
        for w in range(geom["grid"]):
            for ps, t, kb0, kb1, _ in api.streamk_segments(np_, schedule, grid, w)[1].tolist():
                if ps:
                    finish[t] = (kb0, kb1)
                else:
                    handed.setdefault(t, []).append((w // geom["groups"], (kb0, kb1)))
        for t in range(geom["dp_tiles"], geom["ntiles"]):
            want = [finish[t]] + [s for _, s in sorted(handed.get(t, []))]
            assert api.streamk_tile_segments(np_, schedule, grid, t) == want, (np_, t)


def test_argument_errors():
    lib, n = api.lib(), ctypes.c_int32()
    for np_, schedule, grid, t in ((1000, 2, 512, 0), (1024, 3, 512, 0), (1024, 2, 0, 0),
                                   (1024, 2, 512, -1), (1024, 2, 512, 36)):
        rc = lib.fe_streamk_tile_segments(np_, schedule, grid, t, None, 0, ctypes.byref(n))
        assert rc == api.FE_ERR_ARG and n.value == 0
    assert lib.fe_streamk_tile_segments(1024, 2, 512, 0, None, 0, None) == api.FE_ERR_ARG
