"""Which kernel the sizes of GPU tests reach on a card of 256 compute units.  Those tests compare bits with another kernel's, and would pass on
that one as well; here the rules are asked, with the sizes that the tests themselves have."""
import ctypes
import itertools

import pytest

import test_gpu_decode_resident as resident
import test_gpu_decode_resident_rows as resident_rows
import test_gpu_decode_resident_sets as resident_sets
import test_gpu_mx_narrow_tiles as mx_narrow
import test_gpu_packed_thin_columns as thin
import test_gpu_packed_wide_tiles as wide
from paper_2310_19102_amd import binding

TILES = {3: "walk128x128", 4: "walk256x128", **wide.TILES}


def rule(name, M, N, *more):
    return getattr(ctypes.CDLL(binding._LIB_PATH), "atom_internal_" + name)(ctypes.c_int64(M), ctypes.c_int64(N), *more, ctypes.c_int64(256))


def set_rows(M, N, K):
    """Rows of a set of the decode kernel that keeps the activations; 0: another kernel runs."""
    return rule("decode_resident_rows", M, N, K)


def sizes(test):
    """The arguments of every case of a test."""
    axes = [[dict(zip(mark.args[0].split(","), v if isinstance(v, tuple) else (v,))) for v in mark.args[1]] for mark in test.pytestmark]
    return [{k: v for part in case for k, v in part.items()} for case in itertools.product(*axes)]


def test_columns_and_stages_of_thin_tiles():
    for c in sizes(thin.test_thin_columns):
        K, columns = 128 * (c["G4"] + 1), c["columns"]
        tile = rule("packed_tile", c["M"], c["N"], K, 128)
        assert tile in (0, 1), c
        stages = 6 if columns == 32 or (columns == 64 and c["G4"] > 46) else 4
        assert divmod(rule("packed_thin_form", c["M"], c["N"], K, tile), 10) == (columns, stages), c


def test_stages_of_narrow_mx_tiles():
    for c in sizes(mx_narrow.test_mx_narrow_tiles):
        assert rule("mx_tile_k", c["M"], c["N"], c["K"]) == 64064, c
        assert {0: "64x64", 6: "64x32, six stages", 8: "64x32, eight stages"}[rule("mx_narrow_stages", c["M"], c["N"], c["K"])] == c["name"], c


def test_rows_of_a_set():
    for c in sizes(resident.test_resident_decode_equals_slices):
        assert set_rows(**c) and not set_rows(c["M"], resident.SLICE, c["K"]), c
    for c in sizes(resident_rows.test_rows_of_a_workgroup):
        assert set_rows(**c) == (32 if c["N"] == 10001 else 48 if c["M"] <= 48 else 64) and not set_rows(c["M"], resident.SLICE, c["K"]), c
    # beyond 64 rows, with K up to 4096 and with K = 8192; between them 32
    few, many = {65: 48, 96: 48, 97: 64, 130: 48, 150: 64, 193: 64, 256: 64}, {65: 48, 96: 48, 130: 48}
    for c in sizes(resident_sets.test_sets_of_rows):
        assert set_rows(**c) == (few[c["M"]] if c["K"] <= 4096 else many.get(c["M"], 32) if c["K"] == 8192 else 32), c
    for c in sizes(resident_sets.test_three_blocks_of_groups):
        assert set_rows(**c) == 32, c
    for c in sizes(resident_sets.test_one_set_of_48_rows):
        assert set_rows(**c) == 48, c
    for test in (resident_sets.test_sets_of_rows, resident_sets.test_three_blocks_of_groups, resident_sets.test_one_set_of_48_rows):
        for c in sizes(test):
            assert not set_rows(c["M"], resident_sets.SLICE, c["K"]), c


@pytest.mark.parametrize("M,K,N,name", [
    (1536, 4096, 11008, "walk128x128"),  # two rounds of two 128 x 128 tiles per compute unit and eight tiles: 256 x 192 is 4 % slower
    (668, 5120, 22016, "walk128x128"),
    (759, 4096, 22016, "walk128x128"),
    (666, 2688, 22016, "walk128x128"),
    (1325, 5120, 22016, "128x384"),      # two rounds and 380 tiles: 128 x 128 is 9 % slower
    (1300, 5120, 13824, "128x384"),      # two and 164
    (2045, 11008, 12288, "256x192"),     # three whole rounds of 256 x 128: 9 % slower
    (1939, 8192, 12288, "256x192"),
    (1096, 8192, 7598, "128x384"),       # one round, nearly full: two of 256 x 192 are 8 % slower
])
def test_tile_is_the_faster_one(M, K, N, name):
    """(As measured.)"""
    assert TILES[rule("packed_tile", M, N, K, 128)] == name
