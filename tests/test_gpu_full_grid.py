"""Launches of two-cue pinhole pairs at the line where they take every wave that the chip holds of their kernel
(1024 pixels per wave: 6.29e6 source pixels on 256 CUs), one copy of the pairs below it and above it."""
import pytest

import test_gpu_items
from test_gpu_items import pba  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


# 6 pairs of 64x96: 170 copies are 6.27e6 pixels, 171 are 6.30e6
@pytest.mark.parametrize("copies", [170, 171])
@pytest.mark.parametrize("prec", ["F32", "F64"])
def test_items_at_the_line(pba, copies, prec):  # noqa: F811
    test_gpu_items.test_every_item_is_evaluated_once(pba, 3, 64, 96, copies, prec)
