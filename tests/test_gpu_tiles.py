"""Tiles against fragments that start and end anywhere (needs an MI355X):
whole tiles inside an unaligned fragment, tiles cut by a fragment's end, and
neighbouring bytes that no kernel may touch, against the CPU oracle."""
import time

import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import host_bytes, random_byte_fragments, snapshot_and_check

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


@pytest.mark.parametrize("tile", [16, 32, 256, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("size,kw", [
    (200_003, dict()), (1_900_001, dict(direct=True)),          # written by the pack kernel
    (2_500_007, dict()), (2_500_007, dict(grid=3)),
    (17_000_003, dict(direct=True)), (2_500_007, dict(bounce=1)),
])
def test_small_tiles(tile, size, kw):
    """Chunk sizes that leave tiles of less than 8 KiB, in runs that end inside
    a chunk and past the image, over fragments that start and end anywhere."""
    chunk = tile * (2 * (70_000 // tile // 2) + 1)
    assert P.ckpt_debug_tile_plan([size], chunk, 16)[0] == tile
    if "bounce" in kw:
        kw = dict(bounce=4 * chunk, group=2 * chunk)
    rng = np.random.default_rng(tile + size)
    cuts = np.sort(rng.integers(0, size + 1, 37))
    sizes = [int(n) for n in np.diff(np.concatenate([[0], cuts, [size]]))] + [0, 5, 16, 33]
    flat = torch.from_numpy(rng.integers(0, 256, sum(sizes) + 3 * len(sizes) + 1, dtype=np.uint8)).cuda()
    before, views, at = host_bytes(flat), [], 1
    for n in sizes:
        views.append(flat[at:at + n])
        at += n + 3
    ck, _ = snapshot_and_check(views, [host_bytes(v) for v in views], chunk, 16, **kw)
    assert np.array_equal(host_bytes(flat), before)  # and no byte beside a fragment
    ck.close()


@pytest.mark.parametrize("chunk", [(1 << 20) + 16, (1 << 20) + 256, 65536 - 16])
def test_small_tiles_cost_no_latency_each(chunk):
    """What one workgroup per tile, or a few that stride over small tiles,
    would take ten times as long for."""
    tensors, _ = random_byte_fragments([2 << 20] * (7 if chunk < 1 << 20 else 16), seed=chunk)

    def seconds(C):
        best = []
        with P.Checkpointer(tensors, chunk_bytes=C, align_bytes=16, direct=C < 1 << 20) as ck:
            for _ in range(5):
                t = time.perf_counter()
                ck.wait_committed(ck.snapshot(step=1))
                ck.restore()
                best.append(time.perf_counter() - t)
        return min(best)

    assert seconds(chunk) < 3 * seconds(-(-chunk // 8192) * 8192)


@pytest.mark.parametrize("direct", [False, True])
def test_more_tiles_than_a_dispatch_has_workgroups(direct):
    """16-byte tiles of an image just past 128 MiB: one workgroup per tile
    would be more lanes than a dispatch can count."""
    n = (1 << 32) // 512 * 16 + 48
    tensors, host = random_byte_fragments([n // 3, n - n // 3 - 21], seed=n)
    ck, _ = snapshot_and_check(tensors, host, 16 * 65537, 16, direct=direct)
    assert ck.image_bytes > (1 << 32) // 512 * 16
    ck.close()


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_fragments_inside_a_word_are_read_at_the_rate_of_words(shift):
    """One unaligned load per vector took a quarter longer than a fragment that
    starts at a 4-byte word."""
    flat = torch.zeros((1 << 30) + 64, dtype=torch.uint8, device="cuda")

    def sums_ms(at):
        with P.Checkpointer([flat[at:at + (1 << 30)]], chunk_bytes=1 << 20, direct=True) as ck:
            P.ckpt_set_timing(ck.ctx, 1)
            ms = []
            for k in range(5):
                ck.wait_committed(ck.snapshot(step=k))
                ms.append(P.ckpt_last_timing(ck.ctx, P.CKPT_OP_SNAPSHOT)["kernel_ms"])
            return min(ms)

    assert sums_ms(4 + shift) < 1.12 * sums_ms(4)


@pytest.mark.parametrize("grid", [0, 5])
@pytest.mark.parametrize("n,size,align,empty", [(700, 16384 - 256, 256, 0), (700, 16384 + 16, 16, 0), (900, 9001, 16, 9),
                                                (6000, 333, 256, 0), (20000, 17, 16, 3)])
def test_layouts_around_a_fragment_for_two_tiles(n, size, align, empty, grid):
    """Both shapes of the pack, on either side of their line and among empty
    fragments, at any alignment."""
    rng = np.random.default_rng(n)
    flat = torch.from_numpy(rng.integers(0, 256, n * (size + 1) + 1, dtype=np.uint8)).cuda()
    views = [flat[1 + k * (size + 1):1 + k * (size + 1) + size] for k in range(n)]
    for k in range(empty):
        views.insert(k * 7, flat[:0])
    host = [host_bytes(v) for v in views]
    ck, _ = snapshot_and_check(views, host, 1 << 16, align, grid=grid)
    ck.close()
    want, _, nc = O.pack(host, align, 1 << 16)
    image, sums = torch.empty(want.size, dtype=torch.uint8, device="cuda"), torch.empty(nc, dtype=torch.int64, device="cuda")
    P.ckpt_pack_noalloc(views, image, sums, chunk_bytes=1 << 16, align_bytes=align)
    assert np.array_equal(host_bytes(image), want)
    assert np.array_equal(host_bytes(sums).view(np.uint64), O.chunk_sums(want, 0, want.size, 1 << 16))


def test_shared_tiles_are_packed_at_the_rate_of_whole_ones():
    """Most tiles hold the ends of fragments: the pack took a third longer than
    of one fragment of as many bytes with 512 lanes for each such tile."""
    def pack_ms(n, size):
        flat = torch.zeros(n * size, dtype=torch.uint8, device="cuda")
        with P.Checkpointer([flat[k * size:(k + 1) * size] for k in range(n)], chunk_bytes=1 << 20) as ck:
            P.ckpt_set_timing(ck.ctx, 1)
            ms = []
            for k in range(5):
                ck.wait_committed(ck.snapshot(step=k))
                ms.append(P.ckpt_last_timing(ck.ctx, P.CKPT_OP_SNAPSHOT)["kernel_ms"])
            return min(ms)

    assert pack_ms(65536, 9216) < 1.25 * pack_ms(1, 65536 * 9216)


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


@pytest.mark.parametrize("n,total,chunk,align", [
    (1, 1, 65536, 16),                     # one byte
    (64, 1 << 20, 65536, 256),             # one workgroup a chunk
    (248, 64 << 20, 65536, 256),           # ... the most fragments, about the largest image
    (249, 1 << 20, 65536, 256),            # one fragment more than a batch of descriptors
    (248, 3 << 20, 4112, 16),              # chunks of an odd number of vectors
    (200, 16 << 20, 65536 + 8192, 16),     # tiles, about the largest such image
    (200, (16 << 20) + 99999, 1 << 20, 16),  # just past it: the tile table from the arguments
    (250, 10 << 20, 16 * 4099, 16),        # 16-byte tiles: several scratch groups, two batches
    (20, 10 << 20, 16 * 4099, 16),         # ... from the arguments
    (700, 5 << 20, 1 << 20, 4096),         # three batches
    (4097, 48 << 20, 1 << 20, 256),        # the tile table's wave search takes three steps
    (3000, 1 << 20, 1 << 20, 16),          # more fragments than the table's LDS holds
    (65536, 4 << 20, 1 << 20, 16),         # the most fragments
])
def test_allocation_free_paths(n, total, chunk, align):
    """Each way the allocation-free pack takes by size and fragment count."""
    rng = np.random.default_rng(n + total + chunk)
    cuts = np.sort(rng.integers(0, total + 1, n - 1))
    sizes = np.diff(np.concatenate([[0], cuts, [total]])).astype(np.int64)
    if n > 4:
        sizes[[0, n // 2, n - 1]] = 0  # empty at both ends and inside
    flat = torch.from_numpy(rng.integers(0, 256, int(sizes.sum()), dtype=np.uint8)).cuda()
    at = np.concatenate([[0], np.cumsum(sizes)])
    views = [flat[int(a):int(a + s)] for a, s in zip(at, sizes)]
    want, _, nc = O.pack([host_bytes(v) for v in views], align, chunk)
    image = torch.full((want.size + 64,), 0xC3, dtype=torch.uint8, device="cuda")
    sums = torch.full((nc + 1,), -1, dtype=torch.int64, device="cuda")
    for _ in range(2):  # again over the first call's tables
        assert P.ckpt_pack_noalloc(views, image, sums, chunk_bytes=chunk, align_bytes=align) == (want.size, nc)
    got = image.cpu().numpy()
    assert np.array_equal(got[:want.size], want) and np.all(got[want.size:] == 0xC3)
    assert np.array_equal(sums.cpu().numpy().view(np.uint64)[:nc], O.chunk_sums(want, 0, want.size, chunk))
    assert int(sums[nc]) == -1


def test_binding_reads_tensors_alike_on_both_paths():
    """The native reading of plain tensors and the Python one of everything
    else: the same results, and the same errors for what is refused."""
    class Sub(torch.Tensor):
        pass

    base = [torch.arange(5000, device="cuda", dtype=torch.int32), torch.empty(0, device="cuda"),
            torch.rand(3, 1001, device="cuda", dtype=torch.float64), torch.rand(777, device="cuda").to(torch.bfloat16)]
    want, _, nc = O.pack([host_bytes(t) for t in base], 256, 65536)
    image = torch.zeros(want.size, dtype=torch.uint8, device="cuda")
    sums = torch.zeros(nc, dtype=torch.int64, device="cuda")
    for tensors in (base, tuple(base), [base[0], base[1], torch.nn.Parameter(base[2]), base[3].detach()],
                    [t.as_subclass(Sub) for t in base]):
        for chunk in (65536, np.int64(65536)):
            image.zero_()
            sums.zero_()
            assert P.ckpt_pack_noalloc(tensors, image, sums, chunk_bytes=chunk) == (want.size, nc)
            assert np.array_equal(image.cpu().numpy(), want)
            assert np.array_equal(sums.cpu().numpy().view(np.uint64), O.chunk_sums(want, 0, want.size, 65536))
    with pytest.raises(ValueError, match="contiguous"):
        P.ckpt_pack_noalloc([base[2].t()], image, sums)
    with pytest.raises(ValueError, match="fragment 1 is not a device tensor"):
        P.ckpt_pack_noalloc([base[0], base[0].cpu()], image, sums)
    for bad in (dict(tensors=[]), dict(tensors=base, chunk_bytes=100), dict(tensors=base, image=image[:-16]),
                dict(tensors=base, image=torch.zeros(want.size, dtype=torch.uint8))):
        with pytest.raises(P.CkptError) as e:
            P.ckpt_pack_noalloc(**dict(dict(image=image, sums=sums, chunk_bytes=65536), **bad))
        assert e.value.code == P.CKPT_EINVAL and len(str(e.value)) > 20
