"""CPU check of what bench.py says about the launches it times."""
import bench


def test_launch_names():
    assert bench.launch_names(True, 32, 2048, 0) == ("stand_step_kernel", "one launch")
    assert bench.launch_names(False, 32, 2048, 1) == ("row_pass_kernel", "five launches")
    assert bench.launch_names(False, 1, 32, 0) == ("row_parts_kernel", "three launches")
    assert bench.launch_names(False, 1, 32, 1) == ("row_parts_kernel", "five launches")   # all-nodes updates
    assert bench.launch_names(False, 8, 16 * 8, 0) == ("row_parts_kernel", "five launches")
