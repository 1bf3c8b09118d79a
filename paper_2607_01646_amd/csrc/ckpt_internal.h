// Internal interface between the libckpt runtime and its gfx950 kernels.
// Not installed; the public ABI is include/ckpt.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ckpt {

// One registered fragment as the kernels see it (32 bytes).
struct FragDev {
    uint64_t ptr;    // device address of the fragment's first byte (any alignment)
    uint64_t nbytes; // fragment bytes
    uint64_t off;    // image offset, a multiple of the alignment (>= 16)
    uint64_t end;    // image offset where the next fragment starts (or the image end)
};

// Tiling of the image.  Tile t covers image bytes [t*T, min((t+1)*T, I)),
// T = 1 << tile_shift divides the chunk size, so no tile crosses a chunk.
struct Geometry {
    uint64_t image_bytes;
    uint64_t n_tiles;
    uint64_t n_chunks;
    uint32_t tile_shift;
    uint32_t tiles_per_chunk; // chunk_bytes >> tile_shift
    bool dense = false;       // at least one non-empty fragment for two tiles: most are shared by several
};

// Where tile t's bytes are, one 64-bit word per tile: the device address of
// its first byte (any alignment; below 2^63) when the whole tile lies in one
// fragment, else kTileSlow with the first fragment holding one of its bytes
// and how many follow it up to the last one.  The tile kernels are bound by
// the loads they have in flight, and every dependent load ahead of them
// shortens that: one word replaces the chain tile -> fragment index ->
// fragment record.
constexpr uint64_t kTileSlow = 1ull << 63;
constexpr uint32_t kMaxFrags = 0x80000000u; // a tile's fragment span fits 31 bits

__host__ __device__ inline uint64_t tile_entry(const FragDev& f, uint32_t first, uint32_t last, uint64_t lo,
                                               uint64_t hi)
{
    if (first == last && hi - f.off <= f.nbytes) return f.ptr + (lo - f.off);
    return kTileSlow | ((uint64_t)(last - first) << 32) | first;
}
__host__ __device__ inline uint32_t tile_first(uint64_t e) { return (uint32_t)e; }
__host__ __device__ inline uint32_t tile_last(uint64_t e) { return (uint32_t)e + (uint32_t)((e & ~kTileSlow) >> 32); }

// Tiles are at most 1 << kMaxTileShift = 8 KiB: each wave's slice of a tile
// is at most one batch of one 16-byte vector per lane.
constexpr uint32_t kMaxTileShift = 13;

// The tile kernels.  Each covers tiles [t_lo, t_hi) and writes tile t's
// word-sum to partials[t] (one entry per tile of the image); launches cover
// whole chunks.  grid_cap bounds the workgroups (one per tile when the cap is
// larger).  Non-null t0/t1 are timing events recorded around the dispatch
// itself.
//   pack:     fragment bytes -> image window; image byte x goes to dst + (x - dst_origin);
//             a non-null release is an HSA signal value the launch sets to 0
//             once workgroup 0 has done its work: a tile, a run of small ones, or
//             with a capped grid its share of all (so the stream's previous
//             kernel has finished)
//   sums:     the sums the pack would compute, from the fragments alone (no image
//             window is written); release as for the pack
//   scatter:  image window -> fragment bytes (image byte x read at src + (x - src_origin))
//   checksum: image window only
hipError_t launch_pack(const FragDev* frags, const uint64_t* tile_src,
                       const Geometry& g, uint64_t t_lo, uint64_t t_hi, uint8_t* dst, uint64_t dst_origin,
                       unsigned long long* partials, uint32_t grid_cap, hipStream_t s, hipEvent_t t0 = nullptr,
                       hipEvent_t t1 = nullptr, int64_t* release = nullptr);
// pack_chunks: the whole image by one workgroup per chunk, with the chunk
// sums; for small images.  A non-null release is set to 0 once the image and
// the sums are written; ticket is then 4 bytes of device memory holding 0, and
// does again when the launch has ended.  For images of at most kReleaseChunks
// chunks.  A one-lane kernel behind the pack costs the commit a launch: trigger
// to commit with it / with the pack's own release, medians of 1200, 17 chunks
// of 64 KiB 60.7 / 58.4 us, 30 chunks 78.3 / 75.9.  The line is not a
// measured crossing: every workgroup pays an L2 write-back, and past 64 chunks
// a launch is a small share of an image's time on the link.
constexpr uint64_t kReleaseChunks = 64;
hipError_t launch_pack_chunks(const FragDev* frags, const uint64_t* tile_src, const Geometry& g, uint8_t* dst,
                              unsigned long long* sums_out, hipStream_t s, int64_t* release = nullptr,
                              uint32_t* ticket = nullptr);
hipError_t launch_sums(const FragDev* frags, const uint64_t* tile_src,
                       const Geometry& g, uint64_t t_lo, uint64_t t_hi, unsigned long long* partials,
                       uint32_t grid_cap, hipStream_t s, hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr,
                       int64_t* release = nullptr);
hipError_t launch_scatter(const FragDev* frags, const uint64_t* tile_src,
                          const Geometry& g, uint64_t t_lo, uint64_t t_hi, const uint8_t* src, uint64_t src_origin,
                          unsigned long long* partials, uint32_t grid_cap, hipStream_t s, hipEvent_t t0 = nullptr,
                          hipEvent_t t1 = nullptr);
hipError_t launch_checksum(const Geometry& g, uint64_t t_lo, uint64_t t_hi, const uint8_t* src, uint64_t src_origin,
                           unsigned long long* partials, uint32_t grid_cap, hipStream_t s, hipEvent_t t0 = nullptr,
                           hipEvent_t t1 = nullptr);

// grid_cap of a scatter that reads pinned host memory.  The link needs ~200
// KiB of loads in flight, and a restore, beside which nothing runs, enough to
// cover its stores too.  GB/s over a 1.5 GB image by grid: 12 44.5, 16 55.8,
// 24 57.0, 32 56.4, 48 53.0, 64 55.0, 96 56.9, 160 57.0, 256 57.0, 512 57.3
// (windows of 320 to 640 KiB are slow on the link itself: a plain copy kernel
// shows the same).
constexpr uint32_t kRestoreGrid = 160;

// grid_cap of a pack that writes pinned host memory: 16 to 256 workgroups
// write at 57 GB/s; a 2 MiB image's snapshot took 74 us with 32, 70 with 64,
// 78 with 128 or one per tile.
constexpr uint32_t kHostPackGrid = 64;

// Chunk sums of the chunks covered by tiles [t_lo, t_hi): sums_out[c] is the
// sum of the partial sums of the chunk's tiles.  With expected non-null, bad[c] is set to 1
// where sums_out[c] != expected[c] (and to 0 elsewhere).  A non-null release
// is set to 0 as the launch starts, as for the pack.
hipError_t launch_chunk_reduce(const Geometry& g, uint64_t t_lo, uint64_t t_hi, const unsigned long long* partials,
                               unsigned long long* sums_out, const unsigned long long* expected, uint8_t* bad,
                               hipStream_t s, int64_t* release = nullptr);

// Direct D2H: the bytes of one fragment inside one chunk group, or one run of
// image padding inside a group (zeroed on the host before the group's copies).
struct Piece {
    uint64_t src; // device address (pieces); unused for padding
    uint64_t off; // image offset
    uint64_t n;
};

// Copy pieces[0, n_pieces) (device memory) into the pinned host image img:
// the smallest pieces of a group, which the DMA engines would spend more time
// taking up than copying (a request costs its engine ~9 us, in which the link
// moves 512 KiB).  The kernel holds compute units while it writes over the
// link, and a GEMM with one workgroup for every unit loses about as long as it
// runs, so past kKernelPiece bytes a piece, where that loss is a tenth of what
// the snapshot gains, it gets at most 1 / kKernelShare of a group's bytes.
// Snapshot in ms / what 4096^3 bf16 products beside it lost by it: nothing by
// the kernel; every piece of up to 512 KiB; those up to 32 KiB and a share of
// 1/16, 1/32, 1/64 (this):
//   1500 x 512 KiB            20.7/0.7  14.6/13.5  20.1/1.8  20.3/1.5  20.4/1.1
//   2000 x 128 KiB            13.6/0.1   4.9/4.5   12.8/0.8  13.2/0.6  13.4/0.4
//   2000 x 32 KiB             10.4/0.3   1.3/1.2        as every piece
//   512 MiB in 1024 ragged    12.6/0.44 10.0/1.54  10.1/1.2  10.1/0.8  10.3/0.40
//   100 MiB in 300 ragged      3.0/0.08  2.0/0.24   2.1/0.17  2.1/0.07  2.2/0.04
//   1.5 GB of a GPT in 400    27.6/1.3  27.3/1.3        as every piece
constexpr uint64_t kKernelPiece = 32ull << 10;
constexpr uint64_t kKernelPieceMax = 512ull << 10;
constexpr uint64_t kKernelShare = 64;
constexpr uint32_t kPieceGrid = 64;
hipError_t launch_copy_pieces(const Piece* pieces, uint64_t n_pieces, uint8_t* img, uint32_t grid_cap, hipStream_t s);

// Store 0 into *signal_value (an HSA signal's value) once the work enqueued
// on s before this call has completed.
hipError_t launch_release(int64_t* signal_value, hipStream_t s);

// Fill [p, p + n) (p 16-byte aligned, n a multiple of 16) with the 16-byte
// pattern w (the staging canary of ckpt_config.poison).
hipError_t launch_fill16(uint8_t* p, uint64_t n, const uint32_t w[4], hipStream_t s);

// ---- The allocation-free pack (ckpt_pack_noalloc) ----
// Its tables and partial sums live in a fixed device array of the kernel
// file (one per GPU, held until the process ends), laid out as: the fragment
// table (at most kNoallocMaxFrags entries), then the tile table of one group
// of at most kNoallocGroupTiles tiles, then that group's partial sums.  Groups are whole chunks and are packed one
// after another on the caller's stream, reusing the tables.
constexpr uint32_t kNoallocMaxFrags = 65536;
constexpr uint64_t kNoallocGroupTiles = 262144; // 2 GiB of 8 KiB tiles
constexpr uint64_t kNoallocMaxChunkTiles = 131072; // a chunk of at most 1 GiB
constexpr uint64_t kNoallocFragsOff = 0;
constexpr uint64_t kNoallocTilesOff = kNoallocFragsOff + (uint64_t)kNoallocMaxFrags * sizeof(FragDev);
constexpr uint64_t kNoallocPartialsOff = kNoallocTilesOff + kNoallocGroupTiles * 8;
constexpr uint64_t kNoallocScratchBytes = kNoallocPartialsOff + kNoallocGroupTiles * 8; // 6 MiB
// Fragment descriptors travel as kernel arguments, so the caller's array has
// been read when the call returns and nothing is allocated for it.  A batch
// is the most that fits 4 KiB of arguments beside a kernel's others: pointer
// and size only, the image offsets being a scan of the padded sizes.
constexpr uint32_t kArgFrags = 248;
struct FragArgs {
    uint32_t count, align;
    uint64_t off; // image offset of the batch's first fragment
    struct {
        uint64_t ptr, nbytes;
    } f[kArgFrags];
};
// Without a tile table, for at most kArgFrags fragments (launch_pack_small):
// images of up to kSmallChunksImage whose chunks are at most kSmallSpan, one
// workgroup and one launch for each chunk's bytes and sum; and images of up
// to kSmallImage in 8 KiB tiles, the chunk reduce following.  The lines lie
// where the table's launches stop costing more.  Time a call in a row of calls,
// in us, with tables -> without (8 fragments): 64 KiB chunks, image of 1 MiB
// 13.0 -> 7.4, 16 MiB 12.0 -> 9.3, 64 MiB 30.5 -> 22.3 (128 KiB chunks by one
// workgroup each: 13.0 -> 12.1 at 1 MiB, 11.5 -> 15.4 at 16 MiB); 1 MiB chunks
// in tiles, image of 1 MiB 12.4 -> 9.6, 16 MiB 11.6 -> 10.7, 64 MiB 28.7 -> 28.3.
// There is no lower line: every workgroup's scan weighs more the smaller the
// chunks are, but so does the table path's reduce, one workgroup per chunk.
// 64 MiB with 8 / 248 fragments: 4 KiB chunks 72.8 -> 44.0 / 75.4 -> 53.7, 1 KiB
// 187 -> 156 / 190 -> 192, 256 bytes 650 -> 613 / 654 -> 735, 16 bytes 10164 ->
// 9750 / 10182 -> 11756.
constexpr uint64_t kSmallSpan = 64ull << 10;
constexpr uint64_t kSmallChunksImage = 64ull << 20;
constexpr uint64_t kSmallImage = 16ull << 20;

// Device address of the current device's scratch array, looked up once per
// device with that device current (the array's host-side name is only a
// handle, never a device address).
hipError_t noalloc_scratch(uint8_t** ptr);

// Write the batch's fragment records to dst[0, b.count) on the device.
hipError_t launch_frag_upload(FragDev* dst, const FragArgs& b, hipStream_t s);

// The tile table (see launch_tile_table) and the records of a fragment list
// that is one batch, in one launch.
hipError_t launch_tile_table_args(const FragArgs& b, FragDev* frags, const Geometry& g, uint64_t t_lo, uint64_t t_hi,
                                  uint64_t* tile_src, hipStream_t s);

// Pack an image of one batch of fragments into img with no tables: out[k] is
// the word-sum of image bytes [k * span, (k + 1) * span), span a multiple of 16.
hipError_t launch_pack_small(const FragArgs& b, uint8_t* img, uint64_t image_bytes, uint64_t span,
                             unsigned long long* out, hipStream_t s);

// Tile table of tiles [t_lo, t_hi) over the n fragments in frags (device):
// tile_src[t - t_lo] = tile_entry() of the first and last fragment holding a
// byte of tile t (the first fragment whose padded span ends past the tile's
// first / last byte; the last fragment when none does), as the runtime's host
// planner computes it.
hipError_t launch_tile_table(const FragDev* frags, uint32_t n, const Geometry& g, uint64_t t_lo, uint64_t t_hi,
                             uint64_t* tile_src, hipStream_t s);

// Tile size rule shared by the planners: the largest power of two no larger
// than 1 << kMaxTileShift (and at least 16) that divides the chunk size.
inline uint32_t tile_shift_for(uint64_t chunk_bytes)
{
    uint32_t ts = 4;
    while (ts < kMaxTileShift && chunk_bytes % (1ull << (ts + 1)) == 0) ++ts;
    return ts;
}

} // namespace ckpt
