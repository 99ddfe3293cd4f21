"""CPU check of what bench.py says about the launches it times."""
import bench
from tests import rowplan


def test_launch_names():
    assert bench.launch_names(True, 32, 64, 152064, 16, 9, 4, 0) == ("stand_step_kernel", "one launch")
    assert bench.launch_names(False, 32, 64, 152064, 16, 9, 4, 0) == ("row_pass_kernel", "two launches")
    assert bench.launch_names(False, 32, 64, 152064, 16, 9, 4, 1) == ("row_pass_kernel", "five launches")   # all-nodes updates
    assert bench.launch_names(False, 1, 32, 152064, 10, 7, 4, 0) == ("row_parts_kernel", "two launches")
    assert bench.launch_names(False, 1, 32, 152064, 10, 7, 4, 1) == ("row_parts_kernel", "five launches")
    assert bench.launch_names(False, 8, 128, 32768, 10, 9, 4, 0) == ("row_parts_kernel", "two launches")     # rows held whole
    assert bench.launch_names(False, 65, 16, 152064, 10, 5, 4, 0)[1] == "five launches"
    assert bench.launch_names(False, 128, 128, 152064, 32, 11, 5, 0) == ("row_pass_kernel", "five launches")


def test_launch_names_follow_the_rules_of_the_library():
    for B in (1, 2, 8, 31, 32, 33, 63, 64, 65, 128):
        for W in (2, 5, 8, 9, 16, 32):
            for orders in (1, 4, 8):
                two = B <= 64 and rowplan.lib().tail_step(B, W, orders)
                assert bench.launch_names(False, B, 64, 152064, 16, W, orders, 0)[1] == ("two launches" if two else "five launches")
    for V in (500, 1000, 1272, 1273, 32761, 32768, 32769, 152064):
        for K in (10, 16, 32):
            whole = rowplan.lib().whole(V, 2, K)
            assert bench.launch_names(False, 32, 64, V, K, 9, 4, 0)[0] == ("row_parts_kernel" if whole else "row_pass_kernel")
