"""CPU tests of the rule that splits few rows over workgroups (csrc/row_plan.hpp)."""
import random

import pytest

from tests import rowplan


@pytest.mark.parametrize("V,dtype,rows,K,split", [
    (152064, "bf16", 32, 10, True), (32000, "f32", 16, 10, True), (128256, "bf16", 256, 10, True), (8000, "bf16", 512, 16, True),
    # too short for a bound: fewer lane groups hold elements than are asked for, or hardly more
    (300, "bf16", 16, 10, False), (1000, "bf16", 256, 32, False), (2000, "bf16", 512, 32, False), (1000, "bf16", 256, 10, True),
    (2600, "bf16", 256, 32, True), (48, "bf16", 64, 16, False),
    # too many workgroups: the streaming kernels are faster
    (262144, "f32", 512, 32, False), (152064, "f32", 512, 16, False), (500000, "f32", 256, 16, False), (1000000, "bf16", 384, 16, False),
    (500000, "f32", 32, 16, True), (262144, "f32", 128, 16, True), (128256, "bf16", 512, 10, False), (63000, "bf16", 512, 10, True),
    (200000, "bf16", 256, 16, False), (152064, "bf16", 256, 16, True), (262144, "bf16", 224, 16, True), (262144, "bf16", 384, 16, False),
    (152064, "bf16", 320, 16, True), (200000, "f32", 192, 16, False),
    # more parts than a row has; more rows than are split
    (32 * 32768 + 8, "bf16", 2, 16, False), (32 * 32768, "bf16", 2, 16, True), (32003, "f32", 576, 20, False), (8000, "bf16", 513, 16, False),
])
def test_split_of_verified_rows(V, dtype, rows, K, split):
    assert (rowplan.row_parts(V, dtype, rows, K) > 0) == split


@pytest.mark.parametrize("V,dtype,B,W,N,R,K,split", [
    (152064, "bf16", 4, 32, 32, 32, 16, True),       # transcript: a chain of 32 nodes, every slot a row
    (50257, "bf16", 6, 7, 40, 7, 10, True),          # accepted paths
    (152064, "bf16", 128, 11, 128, 11, 32, True), (200000, "bf16", 128, 8, 48, 8, 32, True),
    (200000, "bf16", 8, 32, 32, 32, 16, False),      # chains: 256 rows of 7 parts
    (500000, "f32", 128, 9, 64, 9, 32, False),       # 256 rows of 31 parts
    (200000, "f32", 16, 32, 32, 32, 32, False),      # 512 rows of 13
    (1000, "bf16", 64, 9, 64, 9, 32, False),         # no bound
    (32000, "bf16", 32, 9, 64, 64, 16, False),       # all-nodes update: 2048 rows
    (32000, "bf16", 4, 9, 64, 64, 16, True),
    (32000, "bf16", 129, 9, 64, 9, 16, False),
])
def test_split_of_updated_rows(V, dtype, B, W, N, R, K, split):
    assert (rowplan.lib().commit_parts(V, rowplan.element_bytes(dtype), B, W, N, R, K) > 0) == split


def test_waves_of_unsplit_rows():
    assert [rowplan.lib().waves(r) for r in (1, 256, 257, 768, 16384)] == [16, 16, 4, 4, 4]


def test_loads_of_the_exact_sums():
    """Few path rows are cut finer; all drafted rows of a tree are not few, whatever the batch."""
    assert [rowplan.lib().loads(1, 0, b) for b in (1, 16, 17, 128)] == [2, 2, 4, 4]
    assert [rowplan.lib().loads(1, 1, b) for b in (1, 16, 17)] == [4, 4, 4] and rowplan.lib().loads(0, 0, 1) == 4


def test_every_plan_fits_the_kernel():
    """Registers, the most parts, the workgroup limit, parts long enough for a bound, and the memory of the candidates."""
    L, r = rowplan.lib(), random.Random(5)
    for _ in range(20000):
        es = r.choice([2, 4])
        V = int(2 ** r.uniform(5, 22))
        K = r.randint(1, min(32, V))
        rows = r.choice([r.randint(1, 64), r.randint(1, 600)])
        p, vec = L.row_parts(V, es, rows, K), L.vectors(V, es)
        if p:
            per = -(-vec // p)
            last = vec - (p - 1) * per
            assert 1 <= p <= L.parts_max() and per <= L.threads() * L.most_vectors() and rows * p <= L.limit(rows)
            assert last >= 10 * K and (p == 1 or last >= L.threads() - L.parts_max())
        W, N = r.randint(1, 32), r.randint(1, 1024)
        N = max(N, W)
        R = r.choice([W, N])
        B = r.randint(1, 300)
        c = L.commit_parts(V, es, B, W, N, R, K)
        if c:
            assert c <= L.parts_max() and -(-vec // c) <= L.threads() * L.most_vectors()
            assert B * R * c * 64 * 8 <= 28 << 20      # 64 candidate keys per part


def test_rows_held_whole():
    """As many vectors as a workgroup's registers hold, and enough of them for a bound."""
    L = rowplan.lib()
    assert [L.whole(V, 2, 10) for V in (792, 800, 32768, 32769)] == [0, 1, 1, 0]
    assert [L.whole(V, 4, 32) for V in (1276, 1280, 16384, 16385)] == [0, 1, 1, 0]


def test_rows_in_two_parts():
    """More rows than are split otherwise, of more vectors than one workgroup holds and no more than two."""
    L = rowplan.lib()
    assert [L.two_parts(V, 2, 576, 16) for V in (32768, 32769, 65536, 65537)] == [0, 1, 1, 0]
    assert [L.two_parts(32003, 4, r, 20) for r in (512, 513, 640, 641)] == [0, 1, 1, 0]
    assert all(L.row_parts(V, 2, r, 16) == 0 for V in (32769, 65536) for r in (513, 640))
    # beyond 584 rows only parts of more than 7.5 vectors per lane
    assert [L.two_parts(V, 2, r, 16) for V in (34304, 61440, 61441) for r in (584, 585, 640, 641)] == [1, 0, 0, 0, 1, 0, 0, 0, 1, 1, 1, 0]


def test_ranges_of_a_path_row():
    """Whole workgroups of sixteen waves, at most 512 ranges; one vector per lane for few trajectories, four for many, as
    long as not too many workgroups are asked for."""
    L = rowplan.lib()
    assert [L.ranges(V, 2, 1) for V in (13, 8192, 8200, 152064, 10 ** 7)] == [16, 16, 32, 304, 512]
    assert [L.ranges(152064, 2, B) for B in (4, 8, 16, 17, 32, 64)] == [304, 256, 128, 80, 80, 64]
    # all trajectories' rows together: not above 2048 or 4096 unless ranges would be longer than 512 vectors, never above 8192
    assert [L.ranges(300000, 2, B) for B in (1, 16, 32, 64)] == [512, 128, 128, 80]
    assert [L.ranges(10 ** 6, 2, B) for B in (16, 32, 64)] == [256, 256, 128]
    for V in (13, 500, 32003, 128256, 300000, 10 ** 6, 4 * 10 ** 6):
        for B in range(1, 65):
            n, vec = L.ranges(V, 2, B), L.vectors(V, 2)
            assert n % 16 == 0 and 16 <= n <= 512 and B * (n - 16) < 8192
            assert -(-vec // n) <= 64 * 16 or B * n > 4096 or n == 512


def test_path_rows_with_summing_workgroups():
    """As many as 512 workgroups serve, at least three, no more than a path has."""
    s = rowplan.lib().tail_slots
    assert [s(1, 7, 19), s(1, 32, 19), s(1, 32, 32), s(8, 7, 16), s(32, 9, 5), s(24, 32, 1), s(64, 2, 8), s(64, 11, 8)] == [7, 26, 16, 4, 3, 21, 2, 3]


def test_calls_that_end_in_one_launch():
    L = rowplan.lib()
    assert [L.tail_verify(*a) for a in ((32, 32, 32), (64, 8, 5), (64, 9, 5), (33, 32, 2), (33, 32, 3))] == [1, 1, 0, 1, 0]
    assert [L.tail_step(*a) for a in ((1, 32, 8), (64, 8, 4), (64, 9, 4), (8, 32, 8), (9, 32, 8), (37, 11, 5), (38, 11, 5))] == [1, 1, 0, 1, 0, 1, 0]
    assert [L.tail_update(*a) for a in ((5, 8), (10, 4), (6, 7), (12, 3), (13, 1))] == [1, 1, 0, 1, 0]


def test_waiting_workgroups_leave_room():
    """At most an eighth of the places of the compute units that may be used: 256 of two places each, 32 of them, one."""
    assert [rowplan.lib().tail_places(B, 512) for B in (1, 64, 65)] == [1, 1, 0]
    assert [rowplan.lib().tail_places(B, 64) for B in (8, 9)] == [1, 0]
    assert [rowplan.lib().tail_places(1, p) for p in (8, 7, 0)] == [1, 0, 0]


@pytest.mark.parametrize("B,N,V,dtype,two", [
    (16, 64, 152064, "bf16", True), (16, 65, 152064, "bf16", False), (13, 64, 128256, "f32", False),
    (32, 50, 32000, "bf16", True), (32, 51, 32000, "bf16", False), (32, 64, 152064, "bf16", False), (32, 64, 96, "bf16", False),
    (64, 32, 64000, "bf16", True), (64, 33, 32000, "bf16", False), (64, 48, 128256, "bf16", False),
])
def test_two_launches_of_a_small_batch(B, N, V, dtype, two):
    assert bool(rowplan.lib().two_launches(B, B * N, V, rowplan.element_bytes(dtype), 16)) == two
