"""Which partitions of a block take the library's own projections (host only: the rule and the number of
parts are plain functions of sizes)."""
import ctypes

import pytest

MIB = 1 << 20
BUFFER = 32 * MIB  # the partials' buffer of a partition


@pytest.fixture(scope="module")
def rule(native):
    use = native["_ZN4duet10use_skinnyEiimim"]  # use_skinny(rows, cus, weight_bytes, widest, bytes)
    use.argtypes, use.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_size_t, ctypes.c_int, ctypes.c_size_t], ctypes.c_bool
    return use


@pytest.fixture(scope="module")
def splits(native):
    f = native["_ZN4duet13skinny_splitsEiiim"]  # skinny_splits(rows, d_in, d_out, bytes)
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_size_t], ctypes.c_int
    return f


def test_partials_fit_their_buffer(rule, splits):
    """Every accepted shape: heads up to 63 kv heads in groups of 16 give QKV widths up to 145152."""
    refused = 0
    for kv in (1, 8, 32, 56, 57, 60, 63):
        for group in (1, 8, 16):
            d, d_qkv = kv * group * 128, kv * (group + 2) * 128
            for rows in (1, 16, 57, 58, 63, 64):
                if not rule(rows, 256, 1 << 40, max(d, d_qkv), BUFFER):
                    refused += 1
                    continue
                for d_in, d_out in ((d, d_qkv), (d, d), (28672, d)):
                    assert splits(rows, d_in, d_out, BUFFER) * rows * d_out * 4 <= BUFFER, (kv, group, rows)
    assert refused  # 64 rows of 57 kv heads need 33.6 MB


@pytest.mark.parametrize("rows,mb,cus,own", [
    (1, 12, 8, False), (16, 29, 32, True), (16, 50, 32, False), (32, 17, 32, True), (32, 30, 32, False),
    (33, 11, 32, False), (64, 9, 32, True), (16, 50, 64, True), (16, 75, 64, False), (32, 30, 64, True),
    (32, 50, 64, False), (64, 17, 64, True), (64, 30, 64, False), (64, 17, 96, True), (64, 50, 128, False),
    (64, 30, 128, True), (64, 50, 224, False), (32, 500, 96, True), (33, 500, 96, False), (32, 500, 88, False),
    (32, 600, 224, False), (64, 1700, 256, True), (65, 1, 256, False), (0, 1, 256, False)])
def test_both_sides_of_the_rule(rule, rows, mb, cus, own):
    """On a share the own kernels run only where they were measured no slower than the library's."""
    assert rule(rows, cus, mb * 1000000, 1024, BUFFER) == own
