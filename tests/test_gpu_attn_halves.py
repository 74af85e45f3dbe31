"""The two-pass attention kernel where a query's last tile shows keys to one of its two lanes only, or a few to the second: a lane's own maximum and
sum begin, or do not, in a tile that hides keys."""
import pytest

from paper_2310_17723_amd import binding as HB
from test_gpu_attn_split import test_split_against_block as against_split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("mask", [HB.MASK_NONE, HB.MASK_PADDING, HB.MASK_CAUSAL])
@pytest.mark.parametrize("S", [516, 517, 521, 546, 548, 576])
def test_last_tile(Dh, fp8, mask, S):
    against_split(Dh, fp8, mask, S, S)
