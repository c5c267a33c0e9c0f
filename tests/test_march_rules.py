"""Which march takes ragged batches of long rows, by the host's dispatch report: no GPU."""
import pytest

import paper_2411_19419_amd as cs

STAGED = 9


# segments of the staged march that are short only because they are counted by XCD: 1.1 to 1.8 times the other march's time
@pytest.mark.parametrize("shape,batch,storage", [
    ((57, 85, 8, 1, 0), 540, 0), ((64, 87, 8, 1, 0), 601, 0), ((43, 47, 8, 1, 4), 1156, 0), ((62, 69, 8, 1, 4), 282, 0),
    ((43, 58, 8, 1, 7), 1026, 1), ((38, 35, 8, 1, 0), 985, 1),
])
def test_ragged_batches_of_long_rows_stay_off_the_staged_march(shape, batch, storage):
    assert cs.conv_dispatch_info(*shape, batch, storage).kernel != STAGED
    # (what would march if items left the product to the marches: the threshold at its default, no items or blocks below it)
    assert cs.conv_dispatch_info(*shape, batch, storage, march_min_jobs=1).kernel != STAGED


# 25 taps at stride 1 that were in blocks before the staged march's segments were counted by XCD: its sums are less exact
@pytest.mark.parametrize("shape,batch,storage", [
    ((288, 426, 5, 1, 4), 40, 0), ((604, 540, 5, 1, 0), 69, 0), ((515, 539, 5, 1, 2), 44, 1), ((403, 445, 5, 1, 4), 38, 1), ((350, 525, 5, 1, 4), 40, 1),
])
def test_25_taps_in_blocks(shape, batch, storage):
    assert cs.conv_dispatch_info(*shape, batch, storage).kernel == 12
