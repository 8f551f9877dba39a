"""The first sizes past present lines of the rules that choose kernels, checked as the tests of those kernels check theirs."""
import pytest

from test_gpu_decode_resident import test_resident_decode_equals_slices as equals_slices
from test_gpu_decode_resident_sets import _check as equals_slices_of_2048
from test_gpu_gemm_scratch import test_bits_of_the_packed_product as bits_of_the_packed_product
from test_gpu_kv_splits import test_splits as splits_and_oracle
from test_routes_cpu import set_rows

pytestmark = pytest.mark.gpu


# two blocks of groups to a wavefront: up to 24 rows and beyond, two sets
@pytest.mark.parametrize("K", [4352, 4864, 8192])
@pytest.mark.parametrize("M,N", [(17, 8208), (24, 8208), (25, 4112), (64, 4112)])
def test_two_blocks_of_groups(M, N, K):
    assert set_rows(M, N, K) == 32 and not set_rows(M, N - 16, K)
    equals_slices(M, N, K)


@pytest.mark.parametrize("M,N,K", [(20, 12304, 11008), (20, 16400, 9216), (33, 8208, 8448)])
def test_three_blocks_of_groups(M, N, K):
    assert set_rows(M, N, K) == 32 and not set_rows(M, N - 16, K)
    equals_slices_of_2048(M, N, K)


def test_product_on_tiles_of_192_rows():
    bits_of_the_packed_product(300, 13824, 4096)


# one split up to a number of groups that grows with the heads: 136 at 224, 162 at 240, 87 at 195
@pytest.mark.parametrize("B,H,T,splits", [(7, 32, 8704, 1), (7, 32, 8705, 2), (6, 40, 10368, 1), (6, 40, 10369, 2), (13, 15, 5568, 1), (13, 15, 5569, 2)])
def test_splits_of_long_caches(B, H, T, splits):
    splits_and_oracle(B, H, T, splits)
