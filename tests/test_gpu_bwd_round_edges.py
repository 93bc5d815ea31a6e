"""The backward walk's rounds at the edges where their pairs stop fitting. All 16 sub-blocks of a
tile list every particle, padded to a multiple of four: 640 pairs hold 40 isotropic entries, and of 41
a round keeps (640 - 48) / 16 = 37; 576 hold 36 anisotropic ones, and of 37 it keeps 33. Counts on
both sides of each, and lists that end at the edge of a cut round, of the second, and one past."""
import pytest

from tests import test_gpu_bwd_rounds as rounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family,n", [("iso", n) for n in (37, 40, 41, 74, 75, 77, 78)] +
                         [("aniso", n) for n in (33, 36, 37, 66, 67, 69, 70)])
def test_round_edges_match_oracle(family, n):
    rounds.test_rounds_match_oracle(family, n, False)
