"""Which partitions of a block take the library's own projections (host only: the rule and the number of
parts are plain functions of sizes)."""
import ctypes

import pytest

MIB = 1 << 20
BUFFER = 32 * MIB  # the partials' buffer of a partition


@pytest.fixture(scope="module")
def rule(native):
    use = native["_ZN4duet10use_skinnyEiiiiim"]  # use_skinny(rows, cus, d, d_qkv, m, bytes)
    use.argtypes, use.restype = [ctypes.c_int] * 5 + [ctypes.c_size_t], ctypes.c_bool
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
                if not rule(rows, 256, d, d_qkv, 2 * d, BUFFER):
                    refused += 1
                    continue
                for d_in, d_out in ((d, d_qkv), (d, d), (28672, d)):
                    assert splits(rows, d_in, d_out, BUFFER) * rows * d_out * 4 <= BUFFER, (kv, group, rows)
    assert refused  # 64 rows of 57 kv heads need 33.6 MB


WIDTHS = {  # d, d_qkv, m: 6, 17, 30, 17, 50, 75, 436 MB and 1.7 GB of weights a layer
    "6": (1024, 1280, 256), "17": (1024, 1280, 2048), "30": (1024, 1280, 4096), "17w": (1536, 2560, 512),
    "50": (1536, 2560, 4096), "75": (2048, 4096, 4096), "436": (4096, 6144, 14336), "1711": (8192, 10240, 28672)}


@pytest.mark.parametrize("rows,widths,cus,own", [
    (16, "30", 32, True), (16, "50", 32, False), (32, "17", 32, True), (32, "30", 32, False), (16, "17", 8, False),
    (16, "50", 64, True), (16, "75", 64, False), (32, "30", 64, True), (32, "50", 64, False), (17, "50", 64, False),
    (32, "436", 96, True), (32, "436", 88, False), (32, "1711", 224, False), (32, "1711", 256, True),
    (64, "6", 32, True), (64, "17", 32, False), (64, "17", 64, True), (64, "30", 64, False), (64, "30", 128, True),
    (33, "17w", 128, False), (33, "50", 224, False), (33, "17w", 256, False), (32, "17w", 256, True),
    (64, "50", 256, True), (64, "75", 256, True), (64, "436", 256, True), (64, "436", 224, False), (64, "17", 256, True),
    (65, "17", 256, False), (0, "17", 256, False)])
def test_both_sides_of_the_rule(rule, rows, widths, cus, own):
    """The own kernels run only where they were measured no slower than the library's."""
    assert rule(rows, cus, *WIDTHS[widths], BUFFER) == own
