"""The block adjoint where several frequency rows have a kernel of their own with
eight waves (2804 terms, four for one row), and the complex one where several
rows take it because the one-pass kernel spills (76 terms): against the passes
at the edges of its blocks, as the other solutions."""
import pytest

from test_gpu_block_adjoint import test_block_adjoint_edges as real_edges
from test_gpu_block_adjoint import test_complex_block_adjoint_edges as complex_edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("momentum", [False, True], ids=["energies", "momenta"])
def test_rows_of_their_own(momentum):
    real_edges(6, (5, 6, 2), momentum)


def test_complex_rows_where_one_pass_spills():
    complex_edges(4, (0, 4, 9))
