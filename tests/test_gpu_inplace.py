"""Restore and verify read the host image where it lies (needs an MI355X):
images of fewer tiles than the launch has workgroups, of as many and of more,
in every mode, and bytes that the host changes between two calls."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import garbage_fill, host_bytes, random_byte_fragments, snapshot_and_check

pytestmark = pytest.mark.gpu

TILE = 8192


@pytest.mark.parametrize("mode", [dict(), dict(staging=8 * TILE), dict(direct=True), dict(bounce=8 * TILE)])
@pytest.mark.parametrize("tiles", [1, 23, 24, 25, 160, 161, 500])
def test_host_changes_between_calls_are_seen(tiles, mode):
    chunk = 4 * TILE
    tensors, host = random_byte_fragments([tiles * TILE - 5 * TILE // 3] * (tiles > 1) + [5 * TILE // 3 - 7], seed=tiles)
    ck, snap = snapshot_and_check(tensors, host, chunk, 256, group=chunk, **mode)
    img, sums = ck.host_image(snap)
    before = img.copy()
    for _ in range(2):
        at = img.size - 9
        img[at] ^= 0x10
        c = at // chunk
        assert ck.verify() == [c]
        garbage_fill(tensors)
        assert ck.restore() == [c]
        got = O.pack([host_bytes(t) for t in tensors], 256, chunk)[0]
        pad = got != img  # every byte is written back, padding aside
        assert not pad.any() or at >= int(ck.offsets[-1]) + tensors[-1].numel()
        img[at] ^= 0x10
        assert ck.verify() == []
        garbage_fill(tensors)
        assert ck.restore() == []
        assert all(np.array_equal(host_bytes(t), h) for t, h in zip(tensors, host))
    assert np.array_equal(img, before)
    ck.close()
