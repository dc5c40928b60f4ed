"""The HBM bytes that bench.py reports are those of the passes it times."""
import bench


def test_traffic_is_keyed_to_the_timed_passes():
    assert {(name, fields) for name in bench.PASS_NAMES for fields in (1, 256)} == set(bench.TRAFFIC_BYTES)
