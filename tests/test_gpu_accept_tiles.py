"""Acceptance on bf16 rows that go through Gram tiles (widths that are multiples of 128): trips of eight k-steps and what is left of them per wave, the
width whose part is in flight at once, tiles of 15 others that are full, just over and nearly empty.  Case and bounds are those of
test_gpu_accept_widths."""
import pytest

import test_gpu_accept_widths as widths

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden", [128, 384, 1024, 1152, 2048, 3968, 4096, 4224, 5120])
@pytest.mark.parametrize("kids", [1, 7, 8, 15, 16, 60])
def test_acceptance_in_tiles(hidden, kids):
    widths.test_acceptance_on_generic_rows("bf16", hidden, kids)
