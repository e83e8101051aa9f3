"""GPU: the merge kernel takes groups of rows XCD by XCD, the last ones first; every group is taken once, whatever their number beyond a multiple of the
8 XCDs.  The whole round of clustering bit for bit against numpy, the packer against the host's."""
import numpy as np
import pytest

import paper_2506_12038_amd as lcd
from gpu_common import to_dev

pytestmark = pytest.mark.gpu


# fewer groups of 8 rows than XCDs, as many, and several rounds without and with a rest; rows shorter and longer than a step of
# a workgroup, in one part and in several of the assignment
@pytest.mark.parametrize("tiles", [1, 3, 4, 5, 8, 31])
@pytest.mark.parametrize("K", [256, 1024, 3072, 4096, 4352, 9216])
@pytest.mark.parametrize("bits", [2, 3, 4])
def test_every_row_tile_is_taken_once(tiles, K, bits):
    N, slots = 16 * tiles, 1 << bits
    rng = np.random.default_rng(100 * tiles + K + bits)
    # centroids i + row: every row has boundaries of its own, the weights are the centroids themselves
    codebook = (np.arange(slots)[None, :] * 2 + np.arange(N)[:, None] % 61).astype(np.float16)
    idx = rng.integers(0, slots, size=(N, K), dtype=np.uint8)
    w = np.take_along_axis(codebook, idx.astype(np.int64), axis=1)
    got = lcd.lcd_assign_indices(to_dev(w), to_dev(codebook), slots, bits)
    assert np.array_equal(got.cpu().numpy(), idx)
    counts = lcd.lcd_cluster_counts(got, bits)
    expect = np.stack([(idx == b).sum(axis=1) for b in range(slots)], axis=1)
    assert np.array_equal(counts.cpu().numpy(), expect)
    _, out, merged = lcd.lcd_merge_closest(to_dev(codebook), counts, got, slots, bits)      # (equal gaps: the lowest pair)
    assert np.array_equal(merged.cpu().numpy(), np.zeros(N, dtype=np.uint8))
    renumbered = idx - (idx > 0)
    assert np.array_equal(out.cpu().numpy(), renumbered)
    packed = lcd.lcd_pack_indices(out, bits)
    assert np.array_equal(packed.cpu().numpy(), lcd.lcd_pack_indices_host(renumbered.astype(np.uint8), bits))


def test_beyond_the_size_that_is_merged_backwards():
    N, K, bits, slots = 8208, 8192, 2, 4
    idx = np.random.default_rng(5).integers(0, slots, size=(N, K), dtype=np.uint8)
    codebook = np.tile(np.array([0, 2, 3, 9], dtype=np.float16), (N, 1))     # entries 1 and 2 merge
    device = to_dev(idx)
    counts = lcd.lcd_cluster_counts(device, bits)
    assert np.array_equal(counts.cpu().numpy(), np.stack([(idx == b).sum(axis=1) for b in range(slots)], axis=1))
    _, out, merged = lcd.lcd_merge_closest(to_dev(codebook), counts, device, slots, bits)
    assert np.array_equal(merged.cpu().numpy(), np.ones(N, dtype=np.uint8))
    assert np.array_equal(out.cpu().numpy(), idx - (idx > 1))
