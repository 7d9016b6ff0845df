"""Carbon atoms at the edges of the lane groups of the crowded walk (8, 16, 32 and 64 lanes): every
atom of a ball has all others as its bonds.  The oracle, as in the crowded shells' test."""
import pytest

from test_gpu_crowded import test_many_bonds as _many_bonds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("bonds,sep", [(5, 0.6), (8, 0.5), (9, 0.5), (15, 0.4), (16, 0.4), (17, 0.4), (31, 0.3), (32, 0.3),
                                       (33, 0.3), (63, 0.2)])
def test_edges_of_the_groups(bonds, sep, fp64):
    _many_bonds(bonds + 1, 1.04, sep, fp64)
