"""The host's dispatch report tells row groups from the kernels that have a lane per row and chunk of columns (same kernel codes)."""
import pytest

import paper_2411_19419_amd as cs


@pytest.mark.parametrize("shape,batch,storage,channels,kernel,chunks", [
    ((1362, 1644, 1, 2, 0), 100, 0, 1, 1, 25), ((909, 1348, 6, 3, 3), 131, 0, 1, 1, 33), ((30, 31, 9, 3, 8), 2, 0, 136, 0, 2), ((2388, 1551, 3, 3, 1), 64, 1, 1, 1, 16),
    ((85, 92, 4, 1, 2), 204, 2, 1, 10, 51), ((360, 306, 8, 1, 7), 3, 2, 1, 10, 3),
    ((32, 32, 3, 1, 1), 1, 0, 1, 0, 0), ((32, 32, 3, 1, 1), 16, 0, 1, 1, 0), ((32, 32, 3, 1, 1), 16, 2, 1, 10, 0), ((224, 224, 3, 1, 1), 16, 0, 4, 1, 0),
])
def test_chunks_of_a_row(shape, batch, storage, channels, kernel, chunks):
    d = cs.conv_dispatch_info(*shape, batch, storage, channels)
    assert (d.kernel, d.strip) == (kernel, chunks)
    if chunks:
        assert d.columns_per_lane == (4 if batch >= 4 else 1) and chunks == -(-batch // d.columns_per_lane)
        assert d.lanes_per_row * d.strip * (cs.conv_out_shape(*shape)[0] if storage != 1 else shape[0]) <= d.workgroups * d.threads
