"""The Chebyshev recurrence with four rows per workgroup where the last workgroup has fewer, and
kept terms in that form."""
import pytest

from test_gpu_foe_mu import test_kept_terms_change_no_bit as _kept
from test_gpu_foe_rows import test_row_recurrence_at_its_size_limits as _rows

pytestmark = pytest.mark.gpu

# more than 512 rows (else fewer share a workgroup), at most 2528 vertices
SIZES = [(1025, 7), (1026, 6), (1027, 5), (2525, 4), (2527, 7)]


@pytest.mark.parametrize("N,order", SIZES)
def test_rows_of_the_last_workgroup(N, order):
    _rows(N, order)


@pytest.mark.parametrize("N,order", SIZES)
def test_kept_terms_of_the_last_workgroup(N, order):
    _kept(N, order)
