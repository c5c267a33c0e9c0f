"""Which launches of a few workgroups less than compute units march over the rectangles: queried on the host, no GPU."""
import pytest

import paper_2411_19419_amd as cs

RECTANGLES, ROW_GROUPS = 5, 10


@pytest.mark.parametrize("shape,batch,kernel", [
    # strips that are mostly empty, with many blocks of columns: long segments (of a whole small plane) and short ones
    ((32, 20, 7, 2, 6), 1318, ROW_GROUPS), ((39, 25, 7, 2, 3), 1065, ROW_GROUPS), ((53, 32, 5, 2, 2), 1488, ROW_GROUPS),
    ((95, 61, 5, 2, 0), 880, ROW_GROUPS), ((26, 25, 7, 2, 6), 2005, ROW_GROUPS), ((214, 143, 5, 2, 2), 459, RECTANGLES),
    # workgroups enough, but not full ones: few blocks of columns ...
    ((201, 261, 7, 1, 3), 12, ROW_GROUPS), ((447, 386, 7, 2, 6), 12, ROW_GROUPS), ((717, 730, 7, 2, 3), 1, ROW_GROUPS), ((31, 36, 5, 1, 4), 522, ROW_GROUPS),
    # ... and many, or one column of lanes
    ((81, 77, 7, 1, 3), 96, RECTANGLES), ((126, 199, 7, 2, 6), 96, RECTANGLES), ((375, 587, 7, 1, 0), 4, RECTANGLES), ((688, 933, 7, 2, 3), 1, RECTANGLES),
])
def test_rectangles_or_row_groups(shape, batch, kernel):
    assert cs.conv_dispatch_info(*shape, batch, 2).kernel == kernel
