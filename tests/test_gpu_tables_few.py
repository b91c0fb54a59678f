"""complex64 V(z) tables of few planes are formed on the host, longer ones on the
device: the same bits on both sides of the line (six planes)."""
import pytest

from test_gpu_tables import test_tables_bitwise_equal_host_records as check_tables

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [2, 5, 6, 7, 8])
@pytest.mark.parametrize("absorb", [False, True])
def test_tables_on_both_sides(nz, absorb):
    check_tables(nz, absorb)
