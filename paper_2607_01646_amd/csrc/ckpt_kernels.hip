// ckpt_kernels.hip -- gfx950 kernels of libckpt.
//
// Four bandwidth-bound tile kernels over the snapshot image (the contiguous
// buffer of the D2H phase, paper Sec. V-B):
//   PACK     gather fragment bytes into the image window and sum each chunk,
//   SCATTER  write an image window back into the fragments (recovery, paper
//            Sec. VI-E) while re-summing and checking each chunk,
//   VERIFY   re-sum and check an image window only,
//   SUMS     sum each chunk of the image the fragments would make, reading
//            the fragments only (direct D2H: the DMA engines gather the
//            fragments into the host image themselves).
// The chunk sum is the sum of the chunk's 8-byte little-endian words modulo
// 2^64 (padding included).  Bytes are moved as opaque 128-bit words: no
// floating-point instruction touches them, so NaN payloads, -0 and
// subnormals pass unchanged.
//
// Work split.  The image is cut into power-of-two tiles of at most 8 KiB
// that never cross a chunk.  A workgroup of 512 lanes (8 wave64) takes one
// tile (a separate instantiation strides over tiles when the grid is
// capped): wave w owns the tile's 1 KiB slice w and each lane moves one
// 16-byte vector.  Where the chunk size leaves smaller tiles, a workgroup
// takes the 8 KiB run of tiles that such a tile's workgroup would (run_kernel).
// Consecutive tiles go to consecutive workgroups, which the hardware deals
// out round-robin over the 8 XCDs (measured faster than giving each XCD a
// contiguous range).
// What bounds it: HBM, and how soon a wave's load goes out.  A copy of 8 GiB
// with no lookup ahead of it runs at 6.6-6.8 TB/s with one vector per lane
// and 6.1 with two, 5.0 with eight (the fewer bytes a workgroup holds, the
// closer together the reads and writes in flight are).  With two dependent
// lookups ahead of the load (tile -> fragment index -> fragment record) one
// vector per lane fell to 5.3-5.6 TB/s, so each tile's table entry is the
// address of its bytes itself.  The whole pack of a 14.2 GB shard: 4478 us
// with 256 lanes x 2 vectors and the two lookups, 4460 with the entry alone,
// 4385 with 512 lanes x 1.
// A tile inside one fragment takes an unrolled non-temporal stream; when the
// fragment is not 16-byte aligned its side reads the 4-byte words that hold
// each vector (ld_any) and stores unaligned vectors.  Otherwise each vector finds its fragment (binary search
// over the tile's fragment offsets in LDS), loads aligned 16-byte blocks and
// funnel-shifts them when the fragment is misaligned, masks the fragment
// tail and writes zeros for padding.
// Sum reduction: per lane in 64 bits, across the wave with lane shuffles,
// across the workgroup in LDS; one partial sum per tile (one per wave instead
// costs 1.4% of the pack: 32 bytes written per 8 KiB, from four waves).  A
// small second kernel adds the partial sums of each chunk (and, when
// checking, compares with the stored sum).  The hot kernel thus has no
// atomics and no device-scope fence: on gfx950 such a fence writes back and
// invalidates the XCD's L2, which per tile would cost more than the tile's
// own traffic.
// Addition modulo 2^64 is associative and commutative, so any order of
// tiles gives the same bits.
#include <hip/hip_ext.h>

#include <algorithm>
#include <mutex>

#include "ckpt_internal.h"

namespace ckpt {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBlock = 512;      // lanes per workgroup (8 wave64)
constexpr int kLdsFrags = 256;  // fragment records cached per tile (an 8 KiB tile holds at most 33 non-empty ones)
constexpr int kUnroll = 1;      // 16-byte vectors per lane per batch: one batch covers an 8 KiB tile
// The pack of layouts in which most tiles are shared by fragments
// (Geometry::dense).  Such a tile has a chain of dependent loads ahead of its
// data, and twice the tiles are under way with half the lanes each.  Pack in
// us, 256 lanes x 2 with two table lookups / 512 x 1 / 512 x 1 with the
// fragments' records in LDS / this, records too: 65536 fragments of 9000 bytes
// 210 / 278 / 250 / 206, of 4097 102 / 110 / 102 / 93, 262144 of 1 KiB 99 / 122
// / 108 / 92 (large aligned fragments: 4 GiB 1367 / 1317 / 1320 / 1380).
constexpr int kDenseBlock = 256, kDenseUnroll = 2;

enum Mode { PACK = 0, SCATTER = 1, VERIFY = 2, SUMS = 3 };

struct Args {
    const FragDev* frags;
    const uint64_t* tile_src; // per tile: where its bytes are (tile_entry)
    Geometry g;
    uint64_t t_lo, t_hi;
    uint8_t* img; // PACK: destination window; SCATTER/VERIFY: source window; SUMS: unused
    uint64_t origin;
    unsigned long long* partials; // one sum per tile
    int64_t* release;             // PACK, SUMS: an HSA signal value to set to 0 (or null)
};

struct ReduceArgs {
    const unsigned long long* partials;
    uint64_t c_lo, c_hi; // chunks of this launch
    uint64_t n_tiles;
    uint32_t tiles_per_chunk;
    unsigned long long* sums_out; // PACK: chunk sums; SCATTER/VERIFY: recomputed sums
    const unsigned long long* expected; // null when only summing
    uint8_t* bad;
    int64_t* release; // an HSA signal value to set to 0 at the start (or null)
};

// Lane 0 of workgroup 0 stores 0 into *release: a system-scope release of
// "the kernels before this one on the stream have finished".  A kernel
// starts only once the previous kernel of its stream has completed, and a
// kernel's completion releases its writes at device scope (on a multi-XCD
// part that writes the L2 back), so a DMA engine waiting for the signal
// reads that kernel's bytes.  Carried by the next launch, it saves a
// one-lane kernel and a dispatch gap per chunk group.  The tile kernel does
// it after workgroup 0's tile: ahead of the tile, the test of the pointer
// put a second dependent argument load in front of every workgroup's work.
__device__ __forceinline__ void release_signal(int64_t* release)
{
    if (release && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(release, (int64_t)0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ unsigned long long vsum(u32x4 v)
{
    const unsigned long long w0 = (unsigned long long)v.x | ((unsigned long long)v.y << 32);
    const unsigned long long w1 = (unsigned long long)v.z | ((unsigned long long)v.w << 32);
    return w0 + w1;
}

__device__ __forceinline__ u32x4 load16(uint64_t a) { return *reinterpret_cast<const u32x4*>(a); }

__device__ __forceinline__ u32x4 make4(uint64_t r0, uint64_t r1)
{
    u32x4 v;
    v.x = (unsigned)r0;
    v.y = (unsigned)(r0 >> 32);
    v.z = (unsigned)r1;
    v.w = (unsigned)(r1 >> 32);
    return v;
}

// Bytes [p, p+16) of a fragment (ptr, nbytes), p a multiple of 16; bytes at
// or past nbytes read as zero.  Only aligned 16-byte blocks that contain at
// least one byte of the fragment are loaded.
__device__ u32x4 fetch_general(uint64_t ptr, uint64_t nbytes, uint64_t p)
{
    u32x4 r = {0u, 0u, 0u, 0u};
    if (p >= nbytes) return r;
    const uint64_t left = nbytes - p;
    const uint64_t a = ptr + p;
    uint32_t s = (uint32_t)(a & 15);
    if (s == 0 && left >= 16) return load16(a);
    const uint64_t a0 = a - s;
    const u32x4 lo = load16(a0); // holds byte a, a fragment byte
    u32x4 hi = r;
    if (s != 0 && a0 + 16 < ptr + nbytes) hi = load16(a0 + 16); // first byte is a fragment byte
    uint64_t w0 = (uint64_t)lo.x | ((uint64_t)lo.y << 32);
    uint64_t w1 = (uint64_t)lo.z | ((uint64_t)lo.w << 32);
    uint64_t w2 = (uint64_t)hi.x | ((uint64_t)hi.y << 32);
    const uint64_t w3 = (uint64_t)hi.z | ((uint64_t)hi.w << 32);
    if (s >= 8) {
        w0 = w1;
        w1 = w2;
        w2 = w3;
        s -= 8;
    }
    uint64_t r0 = w0, r1 = w1;
    if (s != 0) {
        r0 = (w0 >> (8 * s)) | (w1 << (64 - 8 * s));
        r1 = (w1 >> (8 * s)) | (w2 << (64 - 8 * s));
    }
    if (left < 16) {
        if (left < 8) {
            r0 &= (1ull << (8 * left)) - 1;
            r1 = 0;
        } else if (left == 8) {
            r1 = 0;
        } else {
            r1 &= (1ull << (8 * (left - 8))) - 1;
        }
    }
    return make4(r0, r1);
}

// Write the fragment bytes among [p, p+16) from v; p a multiple of 16.
// Stores never touch a byte outside the fragment.
__device__ void store_general(uint64_t ptr, uint64_t nbytes, uint64_t p, u32x4 v)
{
    if (p >= nbytes) return;
    const uint64_t left = nbytes - p;
    const uint64_t d = ptr + p;
    if ((d & 15) == 0 && left >= 16) {
        *reinterpret_cast<u32x4*>(d) = v;
        return;
    }
    const uint32_t nb = left < 16 ? (uint32_t)left : 16u;
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
    if ((d & 3) == 0 && (nb & 3) == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (4u * k < nb) reinterpret_cast<unsigned*>(d)[k] = w[k];
    } else if ((d & 1) == 0 && (nb & 1) == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (2u * k < nb) reinterpret_cast<unsigned short*>(d)[k] = (unsigned short)(w[k >> 1] >> (16 * (k & 1)));
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if ((uint32_t)k < nb) reinterpret_cast<unsigned char*>(d)[k] = (unsigned char)(w[k >> 2] >> (8 * (k & 3)));
    }
}

template <bool NT>
__device__ __forceinline__ u32x4 ld(const u32x4* p)
{
    if (NT) return __builtin_nontemporal_load(p);
    return *p;
}

// Streaming 16-byte store: non-temporal and device scope (sc1).  The device
// scope sends the line past the XCD's L2 at once; on the 1.3B shard's pack
// this measured ~1% faster than the non-temporal store alone (same bytes and
// sums; sc1 on the loads was slower).  The address is a device pointer into
// global memory (fragments or the image), so the global form applies.
// A store of more than 8 bytes reads its data registers after issue: on the
// gfx940 family a VALU write to them needs two wait states first.  The
// compiler keeps that distance for its own stores but cannot see into this
// one, so the two wait states (s_nop 1) come with it.
__device__ __forceinline__ void st_stream(u32x4 v, u32x4* p)
{
    asm volatile("global_store_dwordx4 %0, %1, off nt sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}

template <bool NT>
__device__ __forceinline__ void st(u32x4 v, u32x4* p)
{
    if (NT) st_stream(v, p);
    else *p = v;
}

// Vector accesses at any address are one instruction on gfx950; the memory
// pipe splits those that cross a cache line, and takes loads that start inside
// a 4-byte word more slowly.
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
typedef unsigned int u32x4_words __attribute__((ext_vector_type(4), aligned(4)));

// 16 bytes at any address, from the 4-byte words that hold them: no word
// without one of these bytes is read.  Cached, since neighbouring lanes share
// words and lines.  Pack of one fragment of 100 MiB / 1 GiB, in us, that
// starts at an odd or odd half word: one unaligned non-temporal load 45.2 /
// 368, aligned pairs of vectors 39.0 / 352, this 39.1 / 351; at a word: 41.7 /
// 335, 38.3 / 350, 38.5 / 341 (a multiple of 16, which does not come here:
// 43.5 / 332).  Sums of 1 GiB 203, 189, 182; 164, 250, 176 (163).
__device__ __forceinline__ u32x4 ld_any(const uint8_t* p)
{
    const uint32_t sh = (uint32_t)(uintptr_t)p & 3;
    const u32x4 v = *reinterpret_cast<const u32x4_words*>(p - sh);
    if (sh == 0) return v;
    const uint32_t w = *reinterpret_cast<const uint32_t*>(p - sh + 16);
    u32x4 r;
    r.x = __builtin_amdgcn_alignbyte(v.y, v.x, sh);
    r.y = __builtin_amdgcn_alignbyte(v.z, v.y, sh);
    r.z = __builtin_amdgcn_alignbyte(v.w, v.z, sh);
    r.w = __builtin_amdgcn_alignbyte(w, v.w, sh);
    return r;
}

// One wave's slice of a tile: the n <= 64 * UNROLL vectors at s (copied to d
// unless STORE is false) and their sum.  Lane l takes vectors l, l + 64, ...;
// every guarded load is issued before the first store, each a contiguous
// 1 KiB run per wave.  SRC_ANY / DST_ANY: that side is at any address, not
// only a multiple of 16.  Written out without a loop: a runtime trip count
// here measured ~1.5% slower.
template <int UNROLL, bool NTL, bool NTS, bool STORE, bool SRC_ANY = false, bool DST_ANY = false>
__device__ __forceinline__ unsigned long long slice_stream(const uint8_t* s, uint8_t* d, uint32_t n, uint32_t lane)
{
    u32x4 r[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u)
        if (lane + u * 64 < n)
            r[u] = SRC_ANY ? ld_any(s + 16 * (lane + u * 64))
                           : ld<NTL>(reinterpret_cast<const u32x4*>(s) + lane + u * 64);
    unsigned long long acc = 0;
#pragma unroll
    for (int u = 0; u < UNROLL; ++u)
        if (lane + u * 64 < n) {
            if (STORE && DST_ANY) *reinterpret_cast<u32x4_any*>(d + 16 * (lane + u * 64)) = r[u];
            else if (STORE) st<NTS>(r[u], reinterpret_cast<u32x4*>(d) + lane + u * 64);
            acc += vsum(r[u]);
        }
    return acc;
}

__device__ __forceinline__ unsigned long long shfl_xor64(unsigned long long v, int m)
{
    const unsigned lo = __shfl_xor((unsigned)v, m);
    const unsigned hi = __shfl_xor((unsigned)(v >> 32), m);
    return ((unsigned long long)hi << 32) | lo;
}

// Sum over one wave; every lane gets the result.
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v)
{
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += shfl_xor64(v, m);
    return v;
}

// Sum over the workgroup; the result is valid in thread 0.
template <int BLOCK>
__device__ __forceinline__ unsigned long long block_sum(unsigned long long v, unsigned long long* s_red)
{
    v = wave_sum(v);
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) s_red[wave] = v;
    __syncthreads();
    unsigned long long r = 0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < BLOCK / 64; ++w) r += s_red[w];
    }
    __syncthreads();
    return r;
}

// Index (relative to f0) of the fragment holding image byte x: the largest k
// with s_off[k] <= x.  Empty fragments share their offset with the next
// fragment, so the largest such k is never an empty one.
__device__ __forceinline__ uint32_t find_frag_lds(const uint64_t* s_off, uint32_t n, uint64_t x)
{
    uint32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (s_off[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ uint32_t find_frag_global(const FragDev* frags, uint32_t f0, uint32_t f1, uint64_t x)
{
    uint32_t lo = f0, hi = f1;
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo + 1) >> 1);
        if (frags[mid].off <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The fragments of a tile that several share: records in LDS, so that no vector
// waits for its fragment's record behind the search.
struct TileFrags {
    uint64_t off[kLdsFrags], ptr[kLdsFrags], nbytes[kLdsFrags];
};

// One tile: wave w owns vectors [w * slice, (w + 1) * slice) of it.  Returns
// the sum of the vectors this lane moved.
template <int MODE, int BLOCK, int UNROLL, bool NTL, bool NTS>
__device__ __forceinline__ unsigned long long move_tile(const Args& a, uint64_t t, TileFrags& s)
{
    static_assert(BLOCK * UNROLL * 16 == (1u << kMaxTileShift), "one batch per lane covers the largest tile");
    constexpr uint32_t kSlice = 64 * UNROLL; // vectors per wave slice
    const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint64_t base = t << a.g.tile_shift;
    uint64_t end = base + (1ull << a.g.tile_shift);
    if (end > a.g.image_bytes) end = a.g.image_bytes;
    const uint32_t nvec = (uint32_t)((end - base) >> 4);
    // Wave w owns vectors [v0, v1) of the tile (empty past a short tile's end).
    const uint32_t v0 = w * kSlice;
    const uint32_t v1 = v0 + kSlice < nvec ? v0 + kSlice : (nvec > v0 ? nvec : v0);
    uint8_t* win = MODE == SUMS ? nullptr : a.img + (base - a.origin);
    unsigned long long acc = 0;
    if (MODE == VERIFY) {
        acc = slice_stream<UNROLL, NTL, NTS, false>(win + 16 * v0, nullptr, v1 - v0, lane);
    } else {
        const uint64_t e = a.tile_src[t];
        if (!(e & kTileSlow)) {
            uint8_t* fr = reinterpret_cast<uint8_t*>(e) + 16 * v0;
            uint8_t* im = win + 16 * v0;
            const uint32_t n = v1 - v0;
            const bool aligned = (e & 15) == 0;
            if (MODE == SUMS)
                acc = aligned ? slice_stream<UNROLL, NTL, NTS, false>(fr, nullptr, n, lane)
                              : slice_stream<UNROLL, NTL, NTS, false, true>(fr, nullptr, n, lane);
            else if (MODE == PACK)
                acc = aligned ? slice_stream<UNROLL, NTL, NTS, true>(fr, im, n, lane)
                              : slice_stream<UNROLL, NTL, NTS, true, true>(fr, im, n, lane);
            else
                acc = aligned ? slice_stream<UNROLL, NTL, NTS, true>(im, fr, n, lane)
                              : slice_stream<UNROLL, NTL, NTS, true, false, true>(im, fr, n, lane);
        } else {
            const uint32_t f0 = tile_first(e), f1 = tile_last(e), nf = f1 - f0 + 1;
            const bool in_lds = f0 != f1 && nf <= (uint32_t)kLdsFrags;
            FragDev F;
            if (in_lds) {
                // Several fragments: their records go to LDS for the search.
                // Both barriers are workgroup-uniform (e depends on t only);
                // the first keeps the previous tile's readers ahead of the refill.
                __syncthreads();
                for (uint32_t k = tid; k < nf; k += BLOCK) {
                    const FragDev r = a.frags[f0 + k];
                    s.off[k] = r.off;
                    s.ptr[k] = r.ptr;
                    s.nbytes[k] = r.nbytes;
                }
                __syncthreads();
            } else {
                F = a.frags[f0];
            }
            for (uint32_t v = v0 + lane; v < v1; v += 64) {
                const uint64_t x = base + 16ull * v;
                if (in_lds) {
                    const uint32_t k = find_frag_lds(s.off, nf, x);
                    F.off = s.off[k];
                    F.ptr = s.ptr[k];
                    F.nbytes = s.nbytes[k];
                } else if (f0 != f1) {
                    F = a.frags[find_frag_global(a.frags, f0, f1, x)];
                }
                const uint64_t p = x - F.off;
                if (MODE == SUMS) {
                    acc += vsum(fetch_general(F.ptr, F.nbytes, p));
                } else if (MODE == PACK) {
                    const u32x4 r = fetch_general(F.ptr, F.nbytes, p);
                    st_stream(r, reinterpret_cast<u32x4*>(win) + v);
                    acc += vsum(r);
                } else {
                    u32x4* wv = reinterpret_cast<u32x4*>(win) + v;
                    const u32x4 r = __builtin_nontemporal_load(wv);
                    store_general(F.ptr, F.nbytes, p, r);
                    acc += vsum(r);
                }
            }
        }
    }
    return acc;
}

// One tile and its sum, stored by lane 0 of the workgroup to partials[t].
template <int MODE, int BLOCK, int UNROLL, bool NTL, bool NTS>
__device__ __forceinline__ void do_tile(const Args& a, uint64_t t, TileFrags& s_frags, unsigned long long* s_red)
{
    const unsigned long long acc = wave_sum(move_tile<MODE, BLOCK, UNROLL, NTL, NTS>(a, t, s_frags));
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long sum = 0;
#pragma unroll
        for (uint32_t k = 0; k < BLOCK / 64; ++k) sum += s_red[k];
        a.partials[t] = sum;
    }
}

// Without LOOP the grid has one workgroup per tile and each takes exactly
// one (a grid-stride loop around the same body measured ~3% slower on the
// default launch); with LOOP a capped grid strides over the tiles.
template <int MODE, bool LOOP, int BLOCK = kBlock, int UNROLL = kUnroll, bool NTL = true, bool NTS = true>
__global__ __launch_bounds__(BLOCK) void tile_kernel(Args a)
{
    __shared__ TileFrags s_frags;
    __shared__ unsigned long long s_red[BLOCK / 64];
    const uint64_t first = blockIdx.x;
    if (LOOP) {
        for (uint64_t t = a.t_lo + first; t < a.t_hi; t += gridDim.x) {
            do_tile<MODE, BLOCK, UNROLL, NTL, NTS>(a, t, s_frags, s_red);
            __syncthreads(); // s_red is read before the next tile writes it
        }
    } else {
        do_tile<MODE, BLOCK, UNROLL, NTL, NTS>(a, a.t_lo + first, s_frags, s_red);
    }
    if (MODE == PACK || MODE == SUMS) release_signal(a.release);
}

// One 16-byte vector at image byte x by one lane, which looks its tile up
// itself.  Returns the vector's sum.
template <int MODE>
__device__ __forceinline__ unsigned long long move_vector(const Args& a, uint64_t x)
{
    u32x4* win = MODE == SUMS ? nullptr : reinterpret_cast<u32x4*>(a.img + (x - a.origin));
    u32x4 r;
    if (MODE == VERIFY) return vsum(__builtin_nontemporal_load(win));
    const uint64_t e = a.tile_src[x >> a.g.tile_shift];
    if (!(e & kTileSlow)) {
        uint8_t* fr = reinterpret_cast<uint8_t*>(e + (x & ((1ull << a.g.tile_shift) - 1)));
        if (MODE == SCATTER) {
            r = __builtin_nontemporal_load(win);
            if ((e & 15) == 0) st_stream(r, reinterpret_cast<u32x4*>(fr));
            else *reinterpret_cast<u32x4_any*>(fr) = r;
        } else {
            r = ld_any(fr);
            if (MODE == PACK) st_stream(r, win);
        }
    } else {
        const FragDev F = a.frags[find_frag_global(a.frags, tile_first(e), tile_last(e), x)];
        if (MODE == SCATTER) {
            r = __builtin_nontemporal_load(win);
            store_general(F.ptr, F.nbytes, x - F.off, r);
        } else {
            r = fetch_general(F.ptr, F.nbytes, x - F.off);
            if (MODE == PACK) st_stream(r, win);
        }
    }
    return vsum(r);
}

// Tiles of less than 8 KiB: workgroup b takes 8 KiB of the image, a run of
// whole tiles, one vector per lane, and strides over runs.  The tile size is
// the largest power of two that divides the chunk size, so an odd chunk size
// makes tiles of a few lanes; one workgroup for each of them (or a few that
// stride over them, where the other side of the link wants 200 KiB in flight)
// would be bound by dispatches and by one latency per tile.  256 MiB in 100
// fragments, a workgroup per tile of 512 / of 256 lanes / this: tiles of 4 KiB
// 159 / 174 / 146 us, of 1 KiB 446 / 357 / 144, of 256 bytes 1545 / 1100 / 185,
// of 16 bytes 24600 / 24150 / 1650.
template <int MODE>
__global__ __launch_bounds__(kBlock) void run_kernel(Args a)
{
    __shared__ unsigned long long s_red[kBlock / 64];
    const uint32_t tid = threadIdx.x, shift = a.g.tile_shift;
    const uint32_t lpt = 1u << (shift - 4); // lanes per tile: 1 to 256
    const uint64_t lo = a.t_lo << shift;
    const uint64_t end = (a.t_hi << shift) < a.g.image_bytes ? a.t_hi << shift : a.g.image_bytes;
    const uint64_t runs = (end - lo + (1u << kMaxTileShift) - 1) >> kMaxTileShift;
    for (uint64_t b = blockIdx.x; b < runs; b += gridDim.x) {
        const uint64_t x = lo + (b << kMaxTileShift) + 16 * tid;
        unsigned long long acc = x < end ? move_vector<MODE>(a, x) : 0;
        for (uint32_t m = 1; m < lpt && m < 64; m <<= 1) acc += shfl_xor64(acc, m);
        if (lpt <= 64) {
            if (x < end && (tid & (lpt - 1)) == 0) a.partials[x >> shift] = acc;
        } else { // a tile is two or four waves; uniform over the workgroup
            const uint32_t wpt = lpt >> 6;
            if ((tid & 63) == 0) s_red[tid >> 6] = acc;
            __syncthreads();
            const uint64_t t = ((lo + (b << kMaxTileShift)) >> shift) + tid;
            if (tid < kBlock / 64 / wpt && t < a.t_hi) {
                unsigned long long sum = 0;
                for (uint32_t k = 0; k < wpt; ++k) sum += s_red[tid * wpt + k];
                a.partials[t] = sum;
            }
            __syncthreads(); // s_red is read before the next run writes it
        }
    }
    if (MODE == PACK || MODE == SUMS) release_signal(a.release);
}

// SUMS over runs of kSumsTiles tiles: workgroup b takes tiles
// [t_lo + kSumsTiles * b, t_lo + kSumsTiles * (b + 1)), of 8 KiB.  When they
// are all full tiles inside one 16-byte-aligned fragment, the workgroup streams
// them in one batch: wave w owns a quarter of the run (four vectors per lane,
// all loads issued first), and two waves make up a tile's sum.  Otherwise
// each tile takes the per-tile path.  A read-only stream has no stores to keep the
// memory busy while a workgroup waits for its table lookups, so it needs
// more bytes per workgroup than the pack.  Measured on the 1.3B shard's
// layout: one 8 KiB tile per workgroup ~6.15 TB/s, two ~6.6 TB/s, four
// ~6.4 TB/s, eight ~6.0 TB/s.
constexpr uint32_t kSumsTiles = 2;
constexpr int kSumsBlock = 256;

__global__ __launch_bounds__(kSumsBlock) void sums_run_kernel(Args a)
{
    __shared__ TileFrags s_frags;
    __shared__ unsigned long long s_red[kSumsBlock / 64];
    constexpr uint32_t kTileVecs = 1u << (kMaxTileShift - 4);
    const uint64_t t = a.t_lo + (uint64_t)kSumsTiles * blockIdx.x; // < t_hi (grid: ceil(tiles / kSumsTiles))
    uint64_t e = kTileSlow;
    if (t + kSumsTiles <= a.t_hi && ((t + kSumsTiles) << kMaxTileShift) <= a.g.image_bytes) {
        e = a.tile_src[t];
        if ((e & 15) || a.tile_src[t + 1] != e + (1u << kMaxTileShift)) e = kTileSlow;
    }
    if (!(e & kTileSlow)) { // both tiles full, in one aligned span
        const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        const u32x4* src = reinterpret_cast<const u32x4*>(e) + w * (kTileVecs / 2); // waves 0, 1: tile t; 2, 3: t + 1
        u32x4 r[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) r[u] = __builtin_nontemporal_load(src + lane + u * 64);
        unsigned long long acc = 0;
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) acc += vsum(r[u]);
        acc = wave_sum(acc);
        if (lane == 0) s_red[w] = acc;
        __syncthreads();
        if (threadIdx.x < kSumsTiles) a.partials[t + threadIdx.x] = s_red[2 * threadIdx.x] + s_red[2 * threadIdx.x + 1];
    } else {
        for (uint32_t k = 0; k < kSumsTiles && t + k < a.t_hi; ++k) {
            do_tile<SUMS, kSumsBlock, 2, true, true>(a, t + k, s_frags, s_red);
            __syncthreads(); // s_red is read before the next tile writes it
        }
    }
    release_signal(a.release);
}

// One workgroup per chunk: add the chunk's tile sums; when expected is given,
// also flag a mismatch.  A 64 MiB chunk has 8192 partial sums; each lane
// keeps eight independent loads in flight (with four partial sums per tile,
// a plain strided loop with one load at a time took ~70 us per 1 GiB of
// chunks; now 5 us).
constexpr int kReduceBlock = 1024;
constexpr int kReduceUnroll = 8;

__global__ __launch_bounds__(kReduceBlock) void chunk_reduce_kernel(ReduceArgs r)
{
    __shared__ unsigned long long s_red[kReduceBlock / 64];
    release_signal(r.release);
    const uint64_t c = r.c_lo + blockIdx.x;
    const uint64_t t0 = c * r.tiles_per_chunk;
    uint64_t t1 = t0 + r.tiles_per_chunk;
    if (t1 > r.n_tiles) t1 = r.n_tiles;
    const uint64_t end = t1;
    uint64_t k = t0 + threadIdx.x;
    unsigned long long acc = 0;
    for (; k + (kReduceUnroll - 1) * kReduceBlock < end; k += kReduceUnroll * kReduceBlock) {
        unsigned long long v[kReduceUnroll];
#pragma unroll
        for (int u = 0; u < kReduceUnroll; ++u) v[u] = r.partials[k + u * kReduceBlock];
#pragma unroll
        for (int u = 0; u < kReduceUnroll; ++u) acc += v[u];
    }
    for (; k < end; k += kReduceBlock) acc += r.partials[k];
    const unsigned long long s = block_sum<kReduceBlock>(acc, s_red);
    if (threadIdx.x == 0) {
        r.sums_out[c] = s;
        if (r.expected) r.bad[c] = (s != r.expected[c]) ? 1 : 0;
    }
}

// The pack of one workgroup per chunk: its tiles one after another, and the
// chunk's sum to sums_out, so that no reduce has to follow.  For images small
// enough that their time is launches and not bytes.  With a ticket (0 between
// launches) the workgroup that ends last stores the release itself; every
// workgroup then needs a system-scope release of its own writes, a write-back
// of its XCD's L2, so this is for few workgroups (kReleaseChunks).
__global__ __launch_bounds__(kBlock) void pack_chunks_kernel(Args a, unsigned long long* sums_out, uint32_t* ticket)
{
    __shared__ TileFrags s_frags;
    __shared__ unsigned long long s_red[kBlock / 64];
    const uint64_t t0 = (uint64_t)blockIdx.x * a.g.tiles_per_chunk;
    const uint64_t t1 = t0 + a.g.tiles_per_chunk < a.g.n_tiles ? t0 + a.g.tiles_per_chunk : a.g.n_tiles;
    unsigned long long acc = 0;
    if (a.g.tile_shift < kMaxTileShift) {
        const uint64_t lo = t0 << a.g.tile_shift;
        const uint64_t end = (t1 << a.g.tile_shift) < a.g.image_bytes ? t1 << a.g.tile_shift : a.g.image_bytes;
        for (uint64_t x = lo + 16 * threadIdx.x; x < end; x += 16 * kBlock) acc += move_vector<PACK>(a, x);
    } else {
        for (uint64_t t = t0; t < t1; ++t) acc += move_tile<PACK, kBlock, kUnroll, true, true>(a, t, s_frags);
    }
    acc = block_sum<kBlock>(acc, s_red);
    if (threadIdx.x == 0) sums_out[blockIdx.x] = acc;
    if (ticket) {
        // The compiler does not count st_stream's stores as outstanding.
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        __threadfence_system();
        __syncthreads();
        if (threadIdx.x == 0 &&
            __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) {
            __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.release, (int64_t)0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Most workgroups of a launch: a dispatch counts its lanes in 32 bits.
constexpr uint32_t max_grid(uint32_t block) { return 0xffffffffu / block; }

// A grid of one workgroup per tile (per 8 KiB run of smaller ones), or of as
// many as the cap and the dispatch allow, each striding over the rest: 64 GiB
// are past the dispatch.
// With timing events, the launch records them around the dispatch itself
// (the same interval a kernel trace reports).
template <int MODE>
hipError_t launch_tiles(const Args& a, uint32_t grid_cap, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    if (a.t_hi <= a.t_lo) return hipSuccess;
    const uint32_t per_run = kMaxTileShift - a.g.tile_shift; // log2 of the tiles in 8 KiB
    const uint64_t n = (a.t_hi - a.t_lo + (1ull << per_run) - 1) >> per_run;
    uint32_t block = kBlock, grid = (uint32_t)std::min<uint64_t>(n, std::min(grid_cap, max_grid(kBlock)));
    void (*kern)(Args) = per_run ? run_kernel<MODE> : grid == n ? tile_kernel<MODE, false> : tile_kernel<MODE, true>;
    if (MODE == PACK && !per_run && a.g.dense) {
        block = kDenseBlock;
        grid = (uint32_t)std::min<uint64_t>(n, std::min(grid_cap, max_grid(kDenseBlock)));
        kern = grid == n ? tile_kernel<PACK, false, kDenseBlock, kDenseUnroll>
                         : tile_kernel<PACK, true, kDenseBlock, kDenseUnroll>;
    }
    if (t0 && t1)
        hipExtLaunchKernelGGL(kern, dim3(grid), dim3(block), 0, s, t0, t1, 0, a);
    else
        hipLaunchKernelGGL(kern, dim3(grid), dim3(block), 0, s, a);
    return hipGetLastError();
}

// Bytes [src, src + n) to img + off for each of a list of small pieces (see
// launch_copy_pieces): workgroups stride over the pieces, each lane moves 16
// bytes at a time, and no byte outside a piece is written.
__global__ __launch_bounds__(256) void copy_pieces_kernel(const Piece* pieces, uint64_t n_pieces, uint8_t* img)
{
    for (uint64_t k = blockIdx.x; k < n_pieces; k += gridDim.x) {
        const Piece pc = pieces[k];
        for (uint64_t x = 16 * threadIdx.x; x < pc.n; x += 16 * 256)
            store_general((uint64_t)(uintptr_t)img + pc.off, pc.n, x, fetch_general(pc.src, pc.n, x));
    }
}

// One lane: publish "this point of the stream has been reached" to a DMA
// engine by storing 0 into an HSA signal value it polls.  The store is a
// system-scope release; the kernels before it on the stream have finished
// and their writes are past the L2 (the stream's kernel boundaries release
// at device scope, which on a multi-XCD part writes the L2 back).
__global__ void release_signal_kernel(int64_t* value)
{
    __hip_atomic_store(value, (int64_t)0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(256) void fill16_kernel(u32x4* p, uint64_t n16, u32x4 w)
{
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n16; k += (uint64_t)gridDim.x * blockDim.x)
        p[k] = w;
}

// ---- allocation-free pack: scratch, fragment and tile tables, small images ----

// Image offsets of the batch's fragments, by a scan of their padded sizes:
// s_off[k] for k < b.count.  Called by all lanes of a workgroup of at least
// kArgFrags lanes; ends with a barrier.  s_wave holds one value per wave.
static_assert(kArgFrags <= 256, "the scan covers four waves");
__device__ __forceinline__ void scan_offsets(const FragArgs& b, uint64_t* s_off, uint64_t* s_wave)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint64_t mask = b.align - 1;
    const uint64_t size = tid < b.count ? (b.f[tid].nbytes + mask) & ~mask : 0;
    uint64_t v = size; // inclusive scan over the wave
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned lo = __shfl_up((unsigned)v, d), hi = __shfl_up((unsigned)(v >> 32), d);
        if (lane >= (uint32_t)d) v += ((uint64_t)hi << 32) | lo;
    }
    if (lane == 63 && w < 4) s_wave[w] = v;
    __syncthreads();
    if (tid < b.count) {
        uint64_t off = b.off + v - size;
        for (uint32_t k = 0; k < w; ++k) off += s_wave[k];
        s_off[tid] = off;
    }
    __syncthreads();
}

__device__ __forceinline__ FragDev arg_frag(const FragArgs& b, const uint64_t* s_off, uint32_t k)
{
    FragDev f;
    f.ptr = b.f[k].ptr;
    f.nbytes = b.f[k].nbytes;
    f.off = s_off[k];
    f.end = f.off + ((f.nbytes + b.align - 1) & ~(uint64_t)(b.align - 1));
    return f;
}

// The batch's fragment records, at dst.
__global__ __launch_bounds__(256) void frag_upload_kernel(FragDev* dst, FragArgs b)
{
    __shared__ uint64_t s_off[kArgFrags], s_wave[4];
    scan_offsets(b, s_off, s_wave);
    if (threadIdx.x < b.count) dst[threadIdx.x] = arg_frag(b, s_off, threadIdx.x);
}

// Tile table of tiles [t_lo, t_hi) when every fragment fits one batch: the
// offsets are scanned into LDS and searched there, and workgroup 0 stores the
// records (the pack reads them for tiles that no single fragment covers).
// One launch instead of an upload and a table kernel that searches memory.
__global__ __launch_bounds__(256) void tile_table_args_kernel(FragArgs b, FragDev* frags, Geometry g, uint64_t t_lo,
                                                              uint64_t t_hi, uint64_t* tile_src)
{
    __shared__ uint64_t s_off[kArgFrags], s_wave[4];
    scan_offsets(b, s_off, s_wave);
    if (blockIdx.x == 0 && threadIdx.x < b.count) frags[threadIdx.x] = arg_frag(b, s_off, threadIdx.x);
    const uint64_t t = t_lo + 256ull * blockIdx.x + threadIdx.x;
    if (t >= t_hi) return;
    const uint64_t x0 = t << g.tile_shift;
    uint64_t x1 = x0 + (1ull << g.tile_shift);
    if (x1 > g.image_bytes) x1 = g.image_bytes;
    const uint32_t f0 = find_frag_lds(s_off, b.count, x0), f1 = find_frag_lds(s_off, b.count, x1 - 1);
    tile_src[t - t_lo] = tile_entry(arg_frag(b, s_off, f0), f0, f1, x0, x1);
}

// A small image in one pass over the fragments, with no table: workgroup k
// packs image bytes [k * span, (k + 1) * span) and stores their word-sum in
// out[k].  With span the chunk size these are the chunk sums and the pack is
// one launch; else span is the tile size and the chunk reduce follows.  Every
// workgroup scans the fragment sizes for itself (about 2 us), which costs
// less than the launches that the tables need (3-6 us each, the gap between
// them included).  Four vectors per lane are under way at a time: a 64 KiB
// chunk is two rounds.
constexpr int kSmallBlock = 512;
constexpr int kSmallUnroll = 4;
__global__ __launch_bounds__(kSmallBlock) void pack_small_kernel(FragArgs b, uint8_t* img, uint64_t image_bytes,
                                                                 uint64_t span, unsigned long long* out)
{
    __shared__ uint64_t s_off[kArgFrags], s_wave[4];
    __shared__ unsigned long long s_red[kSmallBlock / 64];
    scan_offsets(b, s_off, s_wave);
    const uint64_t lo = (uint64_t)blockIdx.x * span;
    const uint64_t hi = lo + span < image_bytes ? lo + span : image_bytes;
    unsigned long long acc = 0;
    for (uint64_t x0 = lo + 16 * threadIdx.x; x0 < hi; x0 += 16 * kSmallBlock * kSmallUnroll) {
        u32x4 r[kSmallUnroll];
#pragma unroll
        for (int u = 0; u < kSmallUnroll; ++u) {
            const uint64_t x = x0 + 16 * kSmallBlock * u;
            if (x < hi) {
                const uint32_t k = find_frag_lds(s_off, b.count, x);
                r[u] = fetch_general(b.f[k].ptr, b.f[k].nbytes, x - s_off[k]);
            }
        }
#pragma unroll
        for (int u = 0; u < kSmallUnroll; ++u) {
            const uint64_t x = x0 + 16 * kSmallBlock * u;
            if (x < hi) {
                st_stream(r[u], reinterpret_cast<u32x4*>(img + x));
                acc += vsum(r[u]);
            }
        }
    }
    acc = block_sum<kSmallBlock>(acc, s_red);
    if (threadIdx.x == 0) out[blockIdx.x] = acc;
}

// First fragment whose padded span ends past x, by one wave: 64 ends a step, so
// that 4096 fragments take two dependent loads and not twelve.  end[] never
// decreases; n - 1 when no span ends past x.
__device__ __forceinline__ uint32_t find_end_wave(const FragDev* frags, uint32_t n, uint64_t x)
{
    const uint32_t lane = threadIdx.x & 63;
    uint32_t lo = 0, m = n; // the answer lies in [lo, lo + m)
    while (m > 1) {
        const uint32_t step = (m + 63) / 64, k = lane * step + step - 1; // the last of the lane's run
        const uint32_t skip = step * (uint32_t)__popcll(__ballot(k < m && frags[lo + k].end <= x));
        lo += skip;
        m = step < m - skip ? step : m - skip;
    }
    return lo < n ? lo : n - 1;
}

// One lane per tile: the first fragment whose padded span [off, end) ends past
// the tile's first byte, and the first one ending past its last byte (empty
// fragments have empty spans).  Bound by the chain of dependent loads: two
// waves find the fragments at the ends of the workgroup's tiles, the ends
// between them go to LDS, and the lanes search there (memory is the fallback
// when more than kTableFrags lie in the workgroup's 2 MiB).
constexpr uint32_t kTableFrags = 1024;
__global__ __launch_bounds__(256) void tile_table_kernel(const FragDev* frags, uint32_t n, Geometry g, uint64_t t_lo,
                                                         uint64_t t_hi, uint64_t* tile_src)
{
    __shared__ uint64_t s_end[kTableFrags];
    __shared__ uint32_t s_f[2];
    const uint32_t tid = threadIdx.x;
    const uint64_t b_lo = t_lo + 256ull * blockIdx.x, b_hi = b_lo + 256 < t_hi ? b_lo + 256 : t_hi;
    if (tid < 128) { // waves 0 and 1
        uint64_t x = b_lo << g.tile_shift;
        if (tid >= 64) {
            x = b_hi << g.tile_shift;
            x = (x < g.image_bytes ? x : g.image_bytes) - 1;
        }
        const uint32_t f = find_end_wave(frags, n, x);
        if ((tid & 63) == 0) s_f[tid >> 6] = f;
    }
    __syncthreads();
    const uint32_t f0 = s_f[0], f1 = s_f[1];
    const bool in_lds = f1 - f0 < kTableFrags;
    if (in_lds)
        for (uint32_t k = tid; k <= f1 - f0; k += 256) s_end[k] = frags[f0 + k].end;
    __syncthreads();
    const uint64_t t = b_lo + tid;
    if (t >= b_hi) return;
    const uint64_t x0 = t << g.tile_shift;
    uint64_t x1 = x0 + (1ull << g.tile_shift);
    if (x1 > g.image_bytes) x1 = g.image_bytes;
    uint32_t r[2];
    const uint64_t xs[2] = {x0, x1 - 1};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        uint32_t lo = k ? r[0] : f0, hi = f1; // the answer lies in [lo, hi]
        while (lo < hi) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            if ((in_lds ? s_end[mid - f0] : frags[mid].end) > xs[k]) hi = mid;
            else lo = mid + 1;
        }
        r[k] = lo;
    }
    tile_src[t - t_lo] = tile_entry(frags[r[0]], r[0], r[1], x0, x1);
}

// The scratch of ckpt_pack_noalloc (layout in ckpt_internal.h).  Host code
// reaches it only through the address noalloc_scratch() looks up.
static __device__ __align__(256) uint8_t scratch[kNoallocScratchBytes];

} // namespace

hipError_t noalloc_scratch(uint8_t** ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex m;
    static uint8_t* addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> l(m);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = (uint8_t*)p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t launch_fill16(uint8_t* p, uint64_t n, const uint32_t w[4], hipStream_t s)
{
    if (n == 0) return hipSuccess;
    if (((uintptr_t)p & 15) || (n & 15)) return hipErrorInvalidValue;
    u32x4 v;
    v.x = w[0];
    v.y = w[1];
    v.z = w[2];
    v.w = w[3];
    const uint64_t n16 = n >> 4;
    const uint64_t blocks = std::min<uint64_t>((n16 + 255) / 256, 8192);
    hipLaunchKernelGGL(fill16_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, reinterpret_cast<u32x4*>(p), n16, v);
    return hipGetLastError();
}

hipError_t launch_frag_upload(FragDev* dst, const FragArgs& b, hipStream_t s)
{
    if (b.count == 0 || b.count > kArgFrags) return hipErrorInvalidValue;
    hipLaunchKernelGGL(frag_upload_kernel, dim3(1), dim3(256), 0, s, dst, b);
    return hipGetLastError();
}

hipError_t launch_tile_table_args(const FragArgs& b, FragDev* frags, const Geometry& g, uint64_t t_lo, uint64_t t_hi,
                                  uint64_t* tile_src, hipStream_t s)
{
    if (t_hi <= t_lo) return hipSuccess;
    if (b.count == 0 || b.count > kArgFrags || b.off != 0) return hipErrorInvalidValue;
    const uint64_t nt = t_hi - t_lo;
    hipLaunchKernelGGL(tile_table_args_kernel, dim3((uint32_t)((nt + 255) / 256)), dim3(256), 0, s, b, frags, g, t_lo,
                       t_hi, tile_src);
    return hipGetLastError();
}

hipError_t launch_pack_small(const FragArgs& b, uint8_t* img, uint64_t image_bytes, uint64_t span,
                             unsigned long long* out, hipStream_t s)
{
    if (b.count == 0 || b.count > kArgFrags || b.off != 0 || image_bytes == 0 || span % 16) return hipErrorInvalidValue;
    const uint64_t n = (image_bytes + span - 1) / span;
    hipLaunchKernelGGL(pack_small_kernel, dim3((uint32_t)n), dim3(kSmallBlock), 0, s, b, img, image_bytes, span, out);
    return hipGetLastError();
}

hipError_t launch_tile_table(const FragDev* frags, uint32_t n, const Geometry& g, uint64_t t_lo, uint64_t t_hi,
                             uint64_t* tile_src, hipStream_t s)
{
    if (t_hi <= t_lo || n == 0) return hipSuccess;
    const uint64_t nt = t_hi - t_lo;
    hipLaunchKernelGGL(tile_table_kernel, dim3((uint32_t)((nt + 255) / 256)), dim3(256), 0, s, frags, n, g, t_lo, t_hi,
                       tile_src);
    return hipGetLastError();
}

hipError_t launch_copy_pieces(const Piece* pieces, uint64_t n_pieces, uint8_t* img, uint32_t grid_cap, hipStream_t s)
{
    if (n_pieces == 0) return hipSuccess;
    const uint32_t grid = (uint32_t)std::min<uint64_t>(n_pieces, std::min(grid_cap, kPieceGrid));
    hipLaunchKernelGGL(copy_pieces_kernel, dim3(grid), dim3(256), 0, s, pieces, n_pieces, img);
    return hipGetLastError();
}

hipError_t launch_release(int64_t* signal_value, hipStream_t s)
{
    hipLaunchKernelGGL(release_signal_kernel, dim3(1), dim3(1), 0, s, signal_value);
    return hipGetLastError();
}

hipError_t launch_pack(const FragDev* frags, const uint64_t* tile_src,
                       const Geometry& g, uint64_t t_lo, uint64_t t_hi, uint8_t* dst, uint64_t dst_origin,
                       unsigned long long* partials, uint32_t grid_cap, hipStream_t s, hipEvent_t t0, hipEvent_t t1,
                       int64_t* release)
{
    Args a{frags, tile_src, g, t_lo, t_hi, dst, dst_origin, partials, release};
    return launch_tiles<PACK>(a, grid_cap, s, t0, t1);
}

hipError_t launch_pack_chunks(const FragDev* frags, const uint64_t* tile_src, const Geometry& g, uint8_t* dst,
                              unsigned long long* sums_out, hipStream_t s, int64_t* release, uint32_t* ticket)
{
    if (!release != !ticket) return hipErrorInvalidValue;
    Args a{frags, tile_src, g, 0, g.n_tiles, dst, 0, nullptr, release};
    hipLaunchKernelGGL(pack_chunks_kernel, dim3((uint32_t)g.n_chunks), dim3(kBlock), 0, s, a, sums_out, ticket);
    return hipGetLastError();
}

hipError_t launch_sums(const FragDev* frags, const uint64_t* tile_src,
                       const Geometry& g, uint64_t t_lo, uint64_t t_hi, unsigned long long* partials,
                       uint32_t grid_cap, hipStream_t s, hipEvent_t t0, hipEvent_t t1, int64_t* release)
{
    Args a{frags, tile_src, g, t_lo, t_hi, nullptr, 0, partials, release};
    if (t_hi <= t_lo) return hipSuccess;
    const uint64_t runs = (t_hi - t_lo + kSumsTiles - 1) / kSumsTiles;
    // Smaller tiles, and a capped grid, which strides over tiles.
    if (g.tile_shift < kMaxTileShift || runs > std::min(grid_cap, max_grid(kSumsBlock)))
        return launch_tiles<SUMS>(a, grid_cap, s, t0, t1);
    if (t0 && t1)
        hipExtLaunchKernelGGL(sums_run_kernel, dim3((uint32_t)runs), dim3(kSumsBlock), 0, s, t0, t1, 0, a);
    else
        hipLaunchKernelGGL(sums_run_kernel, dim3((uint32_t)runs), dim3(kSumsBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_scatter(const FragDev* frags, const uint64_t* tile_src,
                          const Geometry& g, uint64_t t_lo, uint64_t t_hi, const uint8_t* src, uint64_t src_origin,
                          unsigned long long* partials, uint32_t grid_cap, hipStream_t s, hipEvent_t t0,
                          hipEvent_t t1)
{
    Args a{frags, tile_src, g, t_lo, t_hi, const_cast<uint8_t*>(src), src_origin, partials, nullptr};
    return launch_tiles<SCATTER>(a, grid_cap, s, t0, t1);
}

hipError_t launch_checksum(const Geometry& g, uint64_t t_lo, uint64_t t_hi, const uint8_t* src, uint64_t src_origin,
                           unsigned long long* partials, uint32_t grid_cap, hipStream_t s, hipEvent_t t0,
                           hipEvent_t t1)
{
    Args a{nullptr, nullptr, g, t_lo, t_hi, const_cast<uint8_t*>(src), src_origin, partials, nullptr};
    return launch_tiles<VERIFY>(a, grid_cap, s, t0, t1);
}

hipError_t launch_chunk_reduce(const Geometry& g, uint64_t t_lo, uint64_t t_hi, const unsigned long long* partials,
                               unsigned long long* sums_out, const unsigned long long* expected, uint8_t* bad,
                               hipStream_t s, int64_t* release)
{
    if (t_hi <= t_lo) return hipSuccess;
    ReduceArgs r;
    r.partials = partials;
    r.c_lo = t_lo / g.tiles_per_chunk;
    r.c_hi = (t_hi + g.tiles_per_chunk - 1) / g.tiles_per_chunk;
    r.n_tiles = g.n_tiles;
    r.tiles_per_chunk = g.tiles_per_chunk;
    r.sums_out = sums_out;
    r.expected = expected;
    r.bad = bad;
    r.release = release;
    hipLaunchKernelGGL(chunk_reduce_kernel, dim3((uint32_t)(r.c_hi - r.c_lo)), dim3(kReduceBlock), 0, s, r);
    return hipGetLastError();
}

} // namespace ckpt
