"""Injection on both sides of the line between the small and the full argument tables: four layers and head_dim 128."""
import pytest

from test_gpu_inject import check, make_card

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,G", [(64, 32), (128, 64), (256, 32)])
@pytest.mark.parametrize("count", [3, 4, 5, 9])
@pytest.mark.parametrize("rope", [None, (500000.0, 64)])
def test_layer_counts_around_four(D, G, count, rope):
    desc, rdesc, card, host = make_card(10, 1, 70, D, G, 300 + D + G)
    check(desc, rdesc, card, host, 10 - count, count, 90, 5, rope, "inject %d layers D=%d rope=%s" % (count, D, rope))
