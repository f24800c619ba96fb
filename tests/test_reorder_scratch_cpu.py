"""Scratch sizes of the reorder (host code only): a program allocates the
scratch of its largest cloud once and uses it for every smaller one."""
import pytest

from paper_2104_07526_amd import pcr

ORDERS = [pcr.ORDER_MORTON, pcr.ORDER_MORTON_SHUFFLE, pcr.ORDER_SHUFFLE]


@pytest.mark.parametrize("order", ORDERS)
@pytest.mark.parametrize("batch", [1, 3, 128])
def test_scratch_of_a_cloud_serves_smaller_ones(order, batch):
    step = 3 << 20                     # the sort's tiles change size here (and at step * batch for the batches)
    around = [s + d for s in (step, step * batch, 4 * step) for d in range(-3, 4)]
    sizes = sorted({1, 2, 127, 128, 129, 2047, 2048, 2049, 65_536, 65_537, 3_050_144, 10_000_000, 100_000_000,
                    796_000_000, (1 << 32) - 1, *around})
    need = [pcr.reorder_scratch_bytes(n, order, batch) for n in sizes]
    assert need[0] > 0
    for (n, a), b in zip(zip(sizes, need), need[1:]):
        assert a <= b, n
