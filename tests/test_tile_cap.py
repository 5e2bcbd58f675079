"""Range of vqe_set_tile_cap (no GPU): 0 and 16 to 8192 entries."""
import pytest

import paper_2311_01242_amd as vq


@pytest.mark.parametrize("batched", [False, True])
def test_tile_cap_range(batched):
    try:
        for entries in (16, 17, 4096, 8190, 8191, 8192, 0):
            vq.set_tile_cap(20, batched, entries)
        for entries in (-1, 1, 15, 8193, 1 << 20):
            with pytest.raises(vq.VQEError) as e:
                vq.set_tile_cap(20, batched, entries)
            assert e.value.code == vq.VQE_ERANGE
    finally:
        vq.set_tile_cap(20, batched)
