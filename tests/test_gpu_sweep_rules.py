"""The one-box sweep (width 0) at the lines where its launch changes with row
length and box size, against the tile kernel, bit for bit: rows of their own
workgroup and the row lengths next to them, small boxes whose workgroups are not
grouped, and the sizes next to those."""
import pytest

from test_gpu_sweep_shapes import _run
from paper_1105_2904_amd import workloads as wl

import numpy as np

ROWS = [("fp32", True, (224, 40, 40)), ("fp32", True, (192, 44, 43)), ("fp32", False, (160, 47, 47)), ("fp32", False, (129, 53, 53)),
        ("fp32", True, (128, 53, 53)), ("fp32", False, (255, 38, 38)), ("fp32", True, (256, 38, 38)), ("fp64", True, (144, 50, 50)),
        ("fp64", True, (240, 39, 39)), ("fp64", False, (208, 42, 42)), ("fp16", True, (192, 52, 52)), ("bf16", True, (192, 52, 52)),
        ("fp32", True, (224, 40, 39)), ("fp16", True, (192, 51, 50))]


@pytest.mark.gpu
@pytest.mark.parametrize("storage,aa,box", ROWS)
def test_rows_of_their_own_workgroup(storage, aa, box):
    w = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
    f0 = wl.random_populations(w, (box[2], box[1], box[0]), 5, 0.01)
    for walls in (0, 7):
        a = _run(19, box, storage, aa, walls, (0, 0, 0), f0)
        b = _run(19, box, storage, aa, walls, (256, 0, 0), f0)
        for x, y in zip(a, b):
            assert np.array_equal(x, y), (storage, aa, box, walls)


@pytest.mark.gpu
@pytest.mark.parametrize("storage,aa,box", [("fp64", False, (70, 71, 70)), ("fp64", False, (71, 71, 70)), ("fp32", False, (70, 71, 70)),
                                            ("fp32", False, (71, 71, 70)), ("fp32", True, (50, 51, 52)), ("fp64", False, (21, 23, 20))])
def test_both_sides_of_a_small_box(storage, aa, box):
    test_rows_of_their_own_workgroup(storage, aa, box)


@pytest.mark.gpu
@pytest.mark.parametrize("storage,box", [("fp32", (88, 89, 89)), ("fp32", (100, 70, 100)), ("fp32", (128, 75, 74)),
                                         ("fp64", (74, 73, 74)), ("fp64", (74, 73, 75))])
def test_default_cap_changes_no_value(storage, box):
    w = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
    f0 = wl.random_populations(w, (box[2], box[1], box[0]), 5, 0.01)
    a = _run(19, box, storage, False, 0, (0, 0, 0), f0)
    for shape in ((0, 0, 8), (0, 0, 2)):
        for x, y in zip(a, _run(19, box, storage, False, 0, shape, f0)):
            assert np.array_equal(x, y), (storage, box, shape)


@pytest.mark.gpu
@pytest.mark.parametrize("storage", ["fp16", "bf16"])
@pytest.mark.parametrize("box", [(224, 47, 47), (240, 50, 50), (250, 45, 45), (100, 71, 72), (416, 29, 30), (200, 42, 41), (200, 42, 42),
                                 (240, 50, 51), (240, 51, 51), (82, 70, 73), (239, 47, 47)])
def test_even_rows_with_two_sites_per_lane(storage, box):
    """Even rows that are not whole cache lines, inside and outside of one round of
    waves and on both sides of 350,000 sites (and an odd row)."""
    test_rows_of_their_own_workgroup(storage, False, box)


@pytest.mark.gpu
@pytest.mark.parametrize("storage,box", [("fp64", (361, 363, 1)), ("fp64", (363, 361, 1)), ("fp64", (365, 364, 1)), ("fp32", (511, 511, 1)),
                                         ("fp32", (517, 516, 1)), ("fp64", (39, 38, 39)), ("fp64", (41, 40, 38)), ("fp32", (49, 50, 50))])
def test_both_sides_of_the_size_that_the_caches_hold(storage, box):
    """Two arrays of FP64 or FP32 below and above 18 MiB, rows that are not whole
    cache lines, against tiles of two widths with a persistent grid or without."""
    q = 9 if box[2] == 1 else 19
    w = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4 if q == 9 else [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
    f0 = wl.random_populations(w, (box[2], box[1], box[0]), 5, 0.01)
    a = _run(q, box, storage, False, 0, (0, 0, 0), f0)
    for shape in ((64, 0, 0), (512, 256, 4)):
        for x, y in zip(a, _run(q, box, storage, False, 0, shape, f0)):
            assert np.array_equal(x, y), (storage, box, shape)


@pytest.mark.gpu
@pytest.mark.parametrize("storage,q,box", [("fp16", 19, (128, 17, 16)), ("bf16", 19, (256, 9, 7)), ("fp16", 9, (192, 61, 1)),
                                           ("fp32", 19, (64, 24, 24)), ("fp64", 9, (61, 60, 1))])
def test_cap_of_one_workgroup(storage, q, box):
    """A cap of 1 reserves all of a compute unit's LDS for one workgroup, the sweep
    with two sites per lane, which has LDS of its own, among them."""
    w = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4 if q == 9 else [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
    f0 = wl.random_populations(w, (box[2], box[1], box[0]), 5, 0.01)
    a = _run(q, box, storage, False, 0, (0, 0, 1), f0)
    for shape in ((0, 0, 0), (64, 0, 1)):
        for x, y in zip(a, _run(q, box, storage, False, 0, shape, f0)):
            assert np.array_equal(x, y), (storage, box, shape)
