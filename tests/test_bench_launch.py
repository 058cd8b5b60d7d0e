"""The launch that bench.py looks up in the counter files: workgroup size and
threads of the one-box kernel, with and without a cap."""
import bench


def test_a_cap_counts_workgroups_of_256_on_small_boxes_too():
    for box in ((31, 31, 31), (180, 180, 1)):
        n = box[0] * box[1] * box[2]
        assert bench.sweep_geometry(box, {"width": 0, "grid": 0, "blocks_per_cu": 0}) == (64, (n + 63) // 64 * 64)
        for cap in (1, 2, 5):
            launch = {"width": 0, "grid": 0, "blocks_per_cu": cap}
            assert bench.sweep_geometry(box, launch) == (256, (n + 255) // 256 * 256)


def test_larger_boxes_and_tiles():
    assert bench.sweep_geometry((64, 32, 16), {"width": 0, "grid": 0, "blocks_per_cu": 0}) == (256, 32768)
    assert bench.sweep_geometry((100, 7, 3), {"width": 128, "grid": 0, "blocks_per_cu": 4}) == (128, 17 * 128)
    assert bench.sweep_geometry((100, 7, 3), {"width": 128, "grid": 8, "blocks_per_cu": 0}) == (128, 1024)
