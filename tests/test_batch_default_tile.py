"""The tile that an untuned batch plan's kernel runs (fe_batch_default_tile, host only), on both sides of
its lines on 256 compute units: all 64 x 64 tiles of an XCD at once, batches of the staged launches (64 MiB
of operands), and the ratio of work between them."""
import ctypes
import os

import pytest

from paper_2605_08523_amd import api


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not os.path.exists(api.LIB_PATH):
        pytest.fail("libfe.so is not built (python -m paper_2605_08523_amd.build)")
    api.lib()


@pytest.mark.parametrize("sizes,launch,prec,tile", [
    # one matrix per XCD: T (2 T + 1) tiles of 64 in 64 places up to T = 5 (n = 640)
    ([640] * 8, "layers", "fp16x2", 64), ([641] * 8, "layers", "fp16x2", 128),
    ([1], "layers", "fp16x2", 64), ([500] * 9, "layers", "fp16x2", 128),
    ([500] * 9, "layers", "bf16x3", 128), ([384] * 11, "layers", "bf16x3", 64),
    # queue: on average one round of them
    ([500] * 14, "queue", "bf16x3", 64), ([500] * 15, "queue", "bf16x3", 128),
    ([640] + [60] * 11, "queue", "fp16x2", 64), ([641] + [60] * 11, "queue", "fp16x2", 128),
    # the ratio of work: T = 4 up to 1.75 rounds (two parts), T = 3 beyond it for two parts only
    ([500] * 24, "queue", "fp16x2", 64), ([500] * 25, "queue", "fp16x2", 128),
    ([520] * 12, "queue", "fp16x2", 128), ([300] * 100, "queue", "fp16x2", 64),
    ([300] * 42, "queue", "bf16x3", 64), ([300] * 43, "queue", "bf16x3", 128),
    ([200] * 255, "queue", "bf16x3", 64), ([70] * 800, "queue", "bf16x3", 64),
    # 64 MiB of operands: staged
    ([140] * 255, "queue", "fp16x2", 64), ([140] * 256, "queue", "fp16x2", 128),
    ([64] * 1024, "queue", "bf16x3", 128), ([520] * 64, "queue", "fp16x2", 128),
])
def test_lines(sizes, launch, prec, tile):
    assert api.batch_default_tile(sizes, 26, launch, prec) == tile


def test_work_table_bounds_it():
    # 3 tiles x 1023 matrices x layers <= 4 Mi items
    assert api.batch_default_tile([100] * 1023, 1366, "queue") == 64
    assert api.batch_default_tile([100] * 1023, 1367, "queue") == 128


def test_argument_errors():
    lib, n, t = api.lib(), (ctypes.c_int64 * 2)(100, 0), ctypes.c_int32()
    for args in ((0, n, 26, 1, 2, 256), (1, None, 26, 1, 2, 256), (1, n, 0, 1, 2, 256), (1, n, 26, 2, 2, 256),
                 (1, n, 26, 1, 2, 0), (2, n, 26, 1, 2, 256)):
        assert lib.fe_batch_default_tile(*args, ctypes.byref(t)) == api.FE_ERR_ARG
    assert lib.fe_batch_default_tile(1, n, 26, 1, 2, 256, None) == api.FE_ERR_ARG
