"""Tiles against fragments that start and end anywhere (needs an MI355X):
whole tiles inside an unaligned fragment, tiles cut by a fragment's end, and
neighbouring bytes that no kernel may touch, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import host_bytes, snapshot_and_check

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2607_01646_amd as P

TILE = 8192
SIZES = [TILE - 1, TILE, TILE + 1, 2 * TILE, 2 * TILE + 15, 5 * TILE + 17, 16, 1, 3 * TILE + 8]


def shifted_views(shift, seed):
    """Byte views at address = shift mod 16, with guard bytes between them."""
    rng = np.random.default_rng(seed)
    starts, at = [], shift
    for n in SIZES:
        starts.append(at)
        at += -(-(n + 16) // 16) * 16
    flat = torch.from_numpy(rng.integers(0, 256, at + 64, dtype=np.uint8)).cuda()
    return flat, [flat[a:a + n] for a, n in zip(starts, SIZES)]


@pytest.mark.parametrize("shift", [0, 1, 2, 4, 7, 8, 15])
@pytest.mark.parametrize("chunk,align,direct", [
    (2 * TILE, 16, False),   # tile edges fall anywhere in the fragments
    (64 * TILE, 4096, False),
    (3 * TILE, 256, True),   # odd tiles per chunk: the sums kernel's two-tile runs cross chunks
])
def test_unaligned_fragments(shift, chunk, align, direct):
    flat, views = shifted_views(shift, shift + chunk)
    before = host_bytes(flat)
    ck, _ = snapshot_and_check(views, [host_bytes(v) for v in views], chunk, align, direct=direct)
    ck.close()
    assert np.array_equal(host_bytes(flat), before)  # the guard bytes too


@pytest.mark.parametrize("shift", [0, 3, 8, 14])
def test_unaligned_fragments_without_allocation(shift):
    _, views = shifted_views(shift, 77 + shift)
    want, _, nc = O.pack([host_bytes(v) for v in views], 16, 4 * TILE)
    image = torch.full((want.size + 64,), 0xC3, dtype=torch.uint8, device="cuda")
    sums = torch.full((nc,), -1, dtype=torch.int64, device="cuda")
    P.ckpt_pack_noalloc(views, image, sums, chunk_bytes=4 * TILE, align_bytes=16)
    got = image.cpu().numpy()
    assert np.array_equal(got[:want.size], want) and np.all(got[want.size:] == 0xC3)
    assert np.array_equal(sums.cpu().numpy().view(np.uint64), O.chunk_sums(want, 0, want.size, 4 * TILE))
