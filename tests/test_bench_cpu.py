"""The benchmark's byte counts, without a GPU."""
import bench


def test_fields_count_once_per_launch():
    """A launch of several steps reads and writes the state once and writes the
    emitted fields once, at its last step."""
    alg, phys = bench.launch_bytes(1000, 120, 16, 4)
    assert phys == 1000 * (120 + 16)
    assert alg == 1000 * (4 * 120 + 16)
    assert bench.launch_bytes(1000, 120, 16, 1) == (136000, 136000)
    assert bench.launch_bytes(1000, 240, 0, 4) == (960000, 240000)
