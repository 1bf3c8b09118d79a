"""Kernels that read or write the host image where it lies (needs an MI355X):
restore with fewer tiles than the launch has workgroups, as many and more, in
every mode, and bytes that the host changes between two calls; small images
and small pieces written by the kernel; and verify, which does neither."""
import time

import numpy as np
import pytest
import torch

import oracle as O

from gpu_util import garbage_fill, host_bytes, random_byte_fragments, snapshot_and_check

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2607_01646_amd as P

TILE = 8192


@pytest.mark.parametrize("mode", [dict(), dict(staging=8 * TILE), dict(direct=True), dict(bounce=8 * TILE)])
@pytest.mark.parametrize("tiles", [1, 23, 24, 25, 160, 161, 500])
def test_host_changes_between_calls_are_seen(tiles, mode):
    """A changed byte of a fragment is found and restored as it is now; one of
    the padding behind the last fragment is found and reaches no fragment."""
    chunk = 4 * TILE
    last = 2 * TILE // 3 - 7  # and 178 bytes of padding
    tensors, host = random_byte_fragments([tiles * TILE - (last + 178), last], seed=tiles)
    ck, snap = snapshot_and_check(tensors, host, chunk, 256, group=chunk, **mode)
    img, sums = ck.host_image(snap)
    assert img.size == tiles * TILE and int(ck.offsets[-1]) + last == img.size - 178
    before = img.copy()
    for at in (img.size - 9, img.size - 179, 0):
        img[at] ^= 0x10
        c = at // chunk
        assert ck.verify() == [c]
        garbage_fill(tensors)
        assert ck.restore() == [c]
        got = O.pack([host_bytes(t) for t in tensors], 256, chunk)[0]
        assert np.array_equal(got[:-178], img[:-178]) and not got[-178:].any()
        img[at] ^= 0x10
        assert ck.verify() == []
        garbage_fill(tensors)
        assert ck.restore() == []
        assert all(np.array_equal(host_bytes(t), h) for t, h in zip(tensors, host))
    assert np.array_equal(img, before)
    ck.close()


@pytest.mark.parametrize("bounce", [False, True])
@pytest.mark.parametrize("size,chunk", [((700 << 20) - 77, 1 << 20), ((100 << 20) - 77, 3 * 4096 * 11),
                                        ((70 << 20) + 1, 40 << 20), (5000, 4096), (1, 1 << 20)])
def test_verify_goes_through_its_ring(size, chunk, bounce):
    """Verify over fewer spans than its ring has slots and over more, with
    several wrong chunks; its kernels run for a small part of the transfer, so
    that training beside it keeps the compute units.  (A launch lasts 6 to 20 us
    by its events whatever it reads, 4 MiB are 70 us on the link.)"""
    group = max(chunk, (4 << 20) // chunk * chunk) if bounce else 0
    tensors, host = random_byte_fragments([size // 3, size - size // 3], seed=size)
    ck, snap = snapshot_and_check(tensors, host, chunk, 16, group=group, bounce=4 * group)
    P.ckpt_set_timing(ck.ctx, 1)
    img, sums = ck.host_image(snap)
    at = sorted({x // chunk: x for x in (0, img.size // 2, img.size - 1)}.values())  # one byte in a chunk
    for x in at:
        img[x] ^= 0x80
    assert ck.verify() == [x // chunk for x in at]
    for x in at:
        img[x] ^= 0x80
    assert ck.verify() == []
    assert np.array_equal(P.ckpt_last_sums(ck.ctx), sums)
    t = P.ckpt_last_timing(ck.ctx, P.CKPT_OP_VERIFY)
    assert t["copies"] == t["kernels"] > 0 and t["copy_bytes"] == img.size
    assert size < 1 << 20 or t["kernel_ms"] < 0.3 * t["copy_ms"]
    ck.close()


@pytest.mark.parametrize("direct", [False, True])
@pytest.mark.parametrize("size,chunk", [
    (1, 65536), (65536, 65536), (100_000, 16), (1_000_000, 48), (1 << 20, 4096), (1 << 20, 65536 + 16),
    (2 << 20, 65536), ((2 << 20) + 1, 65536), (2 << 20, 1 << 20),  # about the largest staged image
    (16 << 20, 65536), ((16 << 20) - 5, 1 << 20), ((16 << 20) + 1, 1 << 20),  # ... and direct one
    (64 * 4096, 4096),                       # the most chunks whose pack releases the commit itself
    (64 * 4096 + 16, 4096),                  # one more
    (64 * 65536, 65536),
])
def test_small_images_written_by_the_kernel(size, chunk, direct):
    """Images on both sides of the sizes that the pack writes straight into
    host memory: image and sums against the oracle, the gate before an
    overwrite, and such snapshots before and after one that was interrupted."""
    tensors, host = random_byte_fragments([size // 3, 0, size - size // 3], seed=size + chunk)
    ck, _ = snapshot_and_check(tensors, host, chunk, 16, direct=direct)
    for step in range(3):
        before = [host_bytes(t) for t in tensors]
        if step == 1:
            P.ckpt_debug_interrupt_next(ck.ctx, 0)
        s = ck.snapshot(step=step)
        ck.wait_captured(s)
        garbage_fill(tensors, 17 + step)  # behind the gate
        if step == 1:
            torch.cuda.synchronize()
            assert ck.state(s) == P.CKPT_SNAP_ABORTED
            continue
        ck.wait_committed(s)
        img, sums = ck.host_image(s)
        want, _, _ = O.pack(before, 16, chunk)
        assert np.array_equal(img, want)
        assert np.array_equal(sums, O.chunk_sums(want, 0, want.size, chunk))
    ck.close()


@pytest.mark.parametrize("size,chunk,direct", [(2 << 20, 65536, False), (2 << 20, 1 << 20, False),
                                               (2 << 20, 65536, True), (16 << 20, 65536, True),
                                               (16 << 20, 1 << 20, True)])
def test_small_image_behind_an_interrupted_copy(size, chunk, direct):
    """A small image written by the kernel right after a snapshot that was
    interrupted once its copies were issued: the same host image, which must
    hold the new bytes whenever those copies land."""
    tensors, host = random_byte_fragments([size // 8] * 8, seed=size)
    ck, _ = snapshot_and_check(tensors, host, chunk, 16, direct=direct)
    for k in range(8):
        P.ckpt_debug_interrupt_next(ck.ctx, 1)
        s = ck.snapshot(step=2 * k)
        if not direct:  # there the gate waits for the copies themselves
            ck.wait_captured(s)
        garbage_fill(tensors, 40 + k)
        s2 = ck.snapshot(step=2 * k + 1)
        ck.wait_committed(s2)
        assert ck.state(s) == P.CKPT_SNAP_ABORTED
        torch.cuda.synchronize()
        img, sums = ck.host_image(s2)
        assert np.all(img == 40 + k)
        assert np.array_equal(sums, O.chunk_sums(img, 0, img.size, chunk))
        assert ck.verify(s2) == []
    ck.close()


@pytest.mark.parametrize("align,shift", [(16, 1), (256, 0), (4096, 6)])
def test_direct_pieces_around_the_kernel_size(align, shift):
    """Direct D2H over several groups: pieces that the kernel copies and
    pieces that the engines copy side by side, from unaligned fragments, and
    groups whose only piece is a small one."""
    k = 512 << 10
    sizes = [k - 1, 3, k, 0, k + 1, 5 * k + 7, 16, 1, 1000, 2 * k, 4097, 40 * k + 11, 17, 255]
    flat = torch.from_numpy(np.random.default_rng(align).integers(0, 256, sum(sizes) + 64 * len(sizes), dtype=np.uint8))
    flat, at, views = flat.cuda(), shift, []
    for n in sizes:
        views.append(flat[at:at + n])
        at += n + 3
    before = host_bytes(flat)
    for chunk, group in [(1 << 20, 4 << 20), (1 << 19, 1 << 19), (1 << 20, 0)]:
        ck, _ = snapshot_and_check(views, [host_bytes(v) for v in views], chunk, align, group=group, direct=True)
        ck.close()
        assert np.array_equal(host_bytes(flat), before)


@pytest.mark.parametrize("size,chunk,group,launch", [
    ((64 << 20) - 16, 1 << 20, 0, 0),                 # just under a led group
    (64 << 20, 1 << 20, 0, 0),                        # the lead and the rest, in one group
    ((64 << 20) + 777, 3 * 4096, 0, 0),               # 4 KiB tiles; the lead ends inside a chunk
    (150 << 20, 5 << 20, 70 << 20, 0),                # the first of three groups is led
    (200 << 20, 1 << 20, 64 << 20, 128 << 20),        # two groups per launch
    (30 << 20, 1 << 20, 8 << 20, 0),                  # halves without a lead, the last group smaller
])
def test_led_and_halved_groups(size, chunk, group, launch):
    """Full staging: the first group's lead, copies in two halves, and the
    same after a snapshot that was interrupted behind its first group."""
    tensors, host = random_byte_fragments([size // 7, size - size // 7 - 5, 5], seed=size)
    ck, _ = snapshot_and_check(tensors, host, chunk, 16, group=group, launch=launch)
    for step in range(3):
        before = [host_bytes(t) for t in tensors]
        if step == 1:
            P.ckpt_debug_interrupt_next(ck.ctx, 1)
        s = ck.snapshot(step=step)
        ck.wait_captured(s)
        garbage_fill(tensors, 17 + step)  # behind the gate
        torch.cuda.synchronize()
        if step == 1:
            assert ck.state(s) == P.CKPT_SNAP_ABORTED
            continue
        ck.wait_committed(s)
        img, sums = ck.host_image(s)
        want, _, _ = O.pack(before, 16, chunk)
        assert np.array_equal(img, want)
        assert np.array_equal(sums, O.chunk_sums(want, 0, want.size, chunk))
    ck.close()


@pytest.mark.parametrize("level", [1, 2])
def test_timing_counts_the_pieces_a_kernel_copies(level):
    """Direct D2H of a group of small pieces and one large one: the kernel's
    copies are part of the copy and of the whole, so that the rate from them is
    one that the link has."""
    tensors, _ = random_byte_fragments([32 << 10] * 2000 + [1 << 20], seed=level)
    with P.Checkpointer(tensors, direct=True) as ck:
        P.ckpt_set_timing(ck.ctx, level)
        for k in range(3):
            ck.wait_committed(ck.snapshot(step=k))
            t = P.ckpt_last_timing(ck.ctx, P.CKPT_OP_SNAPSHOT)
            # 66.6 MB; 16 lanes of PCIe 5.0 carry 63 GB/s
            assert t["copy_bytes"] / 64e6 < t["copy_ms"] < t["total_ms"] < 100, t


@pytest.mark.parametrize("chunk", [65536, 1 << 20])  # packed by chunks, by tiles
def test_grid_blocks_bounds_what_writes_the_image(chunk):
    """grid_blocks caps these kernels too: one workgroup has 8 KiB on the
    link, which wants 200, and takes several times as long."""
    tensors, host = random_byte_fragments([2 << 20], seed=chunk)

    def seconds(grid):
        best = []
        ck, _ = snapshot_and_check(tensors, host, chunk, 256, grid=grid)
        for _ in range(5):
            t = time.perf_counter()
            ck.wait_committed(ck.snapshot(step=1))
            best.append(time.perf_counter() - t)
        ck.close()
        return min(best)

    assert seconds(1) > 2 * seconds(0)


def test_more_pieces_than_a_group_has_requests():
    """Direct D2H of 6000 pieces of 40 KiB in one group: 4096 copies by the
    engines, the rest by the kernel."""
    sizes = [(40 << 10) + 16 * (k % 7) - k % 3 for k in range(6000)]
    assert P.ckpt_debug_kernel_pieces(sizes).sum() == 6000 - 4096
    tensors, host = random_byte_fragments(sizes, seed=6)
    ck, _ = snapshot_and_check(tensors, host, 1 << 20, direct=True)
    ck.close()
