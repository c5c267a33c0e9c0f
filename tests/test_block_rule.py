"""Which products the block kernel (batch on the lanes) takes: queried on the host, no GPU."""
import pytest

import paper_2411_19419_amd as cs


@pytest.mark.parametrize("shape,batch,storage,blocks", [
    ((224, 224, 3, 1, 1), 256, 0, True), ((224, 224, 3, 1, 1), 33, 0, True), ((224, 224, 3, 1, 1), 32, 0, False),
    ((224, 224, 3, 1, 1), 256, 1, True), ((256, 256, 5, 2, 2), 64, 0, True), ((256, 256, 5, 2, 2), 64, 1, True),
    ((246, 246, 4, 1, 2), 96, 0, True), ((329, 300, 6, 2, 5), 100, 1, True), ((300, 300, 12, 4, 5), 64, 1, True),
    ((224, 224, 5, 3, 0), 256, 0, True), ((224, 224, 4, 1, 1), 256, 1, True), ((224, 224, 9, 2, 4), 256, 1, True),
    # not compiled: 1 and 6 taps a side, strides above 4, T^T of more than 5 taps per axis and result (4 at strides 3 and 4)
    ((224, 224, 1, 1, 0), 256, 0, False), ((224, 224, 6, 1, 0), 256, 0, False), ((224, 224, 5, 5, 0), 256, 0, False),
    ((224, 224, 6, 1, 1), 256, 1, False), ((224, 224, 11, 2, 3), 256, 1, False), ((224, 224, 13, 3, 3), 256, 1, False),
    ((224, 224, 3, 3, 1), 256, 1, False),
    # a long start for little work, at any batch
    ((24, 25, 5, 1, 4), 131, 0, False), ((39, 40, 11, 4, 0), 128, 1, False), ((37, 48, 12, 3, 6), 178, 1, False),
    ((59, 62, 11, 3, 10), 168, 1, False), ((85, 52, 11, 4, 10), 180, 1, False), ((89, 104, 12, 4, 6), 108, 1, False),
    # ... but for short starts none
    ((64, 90, 3, 1, 1), 131, 0, True), ((40, 40, 3, 2, 1), 72, 1, True),
    # 25 taps, and 16 of T^T at stride 3: not in place of tiles; 25 taps at stride 1: marches that are full, lanes that are not
    ((182, 111, 5, 1, 2), 144, 0, False), ((475, 679, 5, 1, 2), 80, 0, False), ((180, 170, 5, 1, 2), 128, 1, True),
    ((93, 124, 5, 1, 0), 160, 1, False), ((84, 74, 5, 1, 0), 64, 0, False), ((128, 128, 5, 1, 2), 128, 0, True),
    ((124, 120, 12, 3, 6), 64, 1, False), ((124, 120, 12, 3, 6), 72, 1, True), ((191, 180, 5, 1, 4), 36, 1, False),
    # T^T of mostly single entries: idle lanes or none, every batch
    ((340, 367, 3, 2, 1), 160, 1, True), ((340, 367, 3, 2, 1), 168, 1, True), ((340, 367, 3, 2, 1), 192, 1, True),
    ((340, 367, 3, 2, 1), 72, 1, True), ((881, 1143, 5, 4, 2), 40, 1, True),
    # byte offsets of 32 bits: operands of 4 GiB and more
    ((4000, 4000, 3, 1, 1), 68, 0, False), ((3900, 4000, 3, 1, 1), 68, 0, True),
])
def test_block_rule(shape, batch, storage, blocks):
    d = cs.conv_dispatch_info(*shape, batch, storage)
    assert (d.kernel == 12) == blocks, (shape, batch, d.kernel)
    if blocks:
        m, n, k, s, p = shape
        mo, no = cs.conv_out_shape(*shape)
        assert d.columns_per_lane == 4 and d.lanes_per_row in (16, 32, 64)
        sums = d.workgroups * d.threads * d.strip * d.segment * d.columns_per_lane
        assert sums >= (m * n if storage else mo * no) * batch
        taps = (-k // s) ** 2 if storage else k * k          # the weights of every group's outputs, a float each
        assert 4 * d.threads // d.lanes_per_row * d.strip * d.segment * taps <= d.lds_bytes <= 16384
