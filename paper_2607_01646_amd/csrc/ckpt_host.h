// ckpt_host.h -- internal to libckpt's host side: the context, the records
// of snapshots in flight, the bounce-mode pump, the replication worker and
// the image file, shared by ckpt_runtime.cpp (core path), ckpt_bounce.cpp
// (pageable images behind pinned rings), ckpt_h2h.cpp (replication to a ring
// peer) and ckpt_file.cpp (crash-surviving images).  Not installed.
#pragma once

#include <hip/hip_runtime.h>
#include <hsa/hsa.h>
#include <hsa/hsa_ext_amd.h>

#include <fcntl.h>
#include <sys/mman.h>
#include <sys/stat.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "../../include/ckpt.h"
#include "ckpt_internal.h"
#include "ckpt_wire.h"

namespace ckpt {

constexpr uint64_t kDefaultChunk = 64ull << 20;
constexpr uint32_t kDefaultAlign = 256;
constexpr uint64_t kDefaultGroup = 1ull << 30;
constexpr uint64_t kDefaultLaunch = 0; // full-image staging: bytes per pack launch (0 = one group)
constexpr uint32_t kMaxMeta = 1u << 20;
constexpr uint32_t kDefaultGrid = 0x7fffffff; // one workgroup per tile unless capped
constexpr int kMaxEngines = 2;
// Group copies of at least this many bytes are dealt to both engines.
// What an engine alone moves depends on the machine (29 to 57 GB/s seen, and
// not the same for the two), both together fill the link on each; below, a
// second request costs more than it gives.
constexpr uint64_t kSplitCopy = 8ull << 20;
// Of several pinned groups smaller than this, alternate ones already keep both
// engines busy, and a second request for each costs more.  Whole / in halves, us:
// 64 MiB in groups of 8 MiB 1295 / 1335, of 16 1280 / 1295, 120 in 24 2320 /
// 2355-2560, 128 in 32 2460 / 2500-2680, 96 in 48 1885 / 1885.  (Pageable
// images drain group by group: 64 MiB in groups of 16 MiB 1700 / 1580.)
constexpr uint64_t kSplitGroup = 48ull << 20;
inline bool split_copy(uint64_t n, int engines, uint64_t pinned_groups, uint64_t group_bytes)
{
    return engines > 1 && n >= kSplitCopy && (pinned_groups <= 1 || group_bytes >= kSplitGroup);
}
// The lead: 16 MiB keep the link busy for 290 us, in which the rest of a group
// of 1 GiB is packed (330 us); groups of less than four leads gain nothing.
// It is part of its engine's share, so that the other still has its own.
// Snapshot to commit without / with it, where each engine alone
// fills the link: 65 MiB 1336 / 1322 us, 120 MiB 2362 / 2329, 239 MB 4389 /
// 4284, 1.5 GB 26744 / 26410, 2.8 GB 49514 / 49133.  (With all of the group
// behind the lead on the other engine 239 MB took 4288 us there, and 7710
// where that engine alone moves 29 GB/s.)
constexpr uint64_t kLead = 16ull << 20;
// Bytes of an n-byte group that its first engine moves when both do: half of
// one of several groups, whose first engines alternate, and three quarters of an
// only one.  There engine 0 alone nearly fills the link on every machine but
// the first (41 GB/s), and engine 1 on some does not: 239 MB took 4400 us whole
// on engine 0, 5323 in halves and 7707 mostly on engine 1 where that moves 29
// GB/s.  A quarter is done in time from 14 GB/s on.  Where both fill the link,
// whole / halves / this: 4380 / 4280 / 4315.
inline uint64_t first_share(uint64_t n, uint64_t groups)
{
    return ((groups > 1 ? n / 2 : n / 4 * 3) + 4095) & ~4095ull;
}
// The requests of a staged group's copy of n bytes, in the order in which
// they are issued: the lead if any, the (rest of the) first `cut` bytes on the
// group's first engine (0), what is left of n on its other one.  Returns how many.
struct CopySpan {
    uint64_t lo, n;
    int engine;
};
inline int copy_spans(uint64_t n, uint64_t cut, uint64_t lead, CopySpan out[3])
{
    int k = 0;
    if (lead) out[k++] = CopySpan{0, lead, 0};
    out[k++] = CopySpan{lead, cut - lead, 0};
    if (cut < n) out[k++] = CopySpan{cut, n - cut, 1};
    return k;
}
// Verify's device ring: slots of up to 64 MiB of whole chunks (at least one),
// with pageable images 16 MiB; as many as fit 256 MiB, two to eight.  A slot's
// checksum takes ~1% of the time of its copy, so only the last one's adds to a
// verify.  By slot, 8 / 16 / 32 / 64 MiB: 239 MB 4300 / 4290 / 4308 / 4276 us,
// 1.5 GB 26640 / 26625 / 26650 / 26440 (one copy of each chunk group, a ring of
// two groups: 4295 and 26460); pageable 239 MB 4590 / 4574 / 4658 / 4720 (4900).
constexpr uint64_t kVerifySlot = 64ull << 20;
constexpr uint64_t kVerifySlotBounce = 16ull << 20;
constexpr uint64_t kVerifyRing = 256ull << 20;
constexpr uint32_t kDefaultHostThreads = 12; // bounce mode: host copy threads (measured: 8 do not keep up with the link)

struct Frag {
    uint64_t ptr, nbytes, off;
    uint32_t dtype, cls;
};

constexpr uint64_t kMaxDirectPieces = 65536;
// Direct D2H into pinned images: most copies of one group.  They wait in the
// engines' queues for a release that a launch behind them stores, so a call
// that blocked on a full queue would never end: 16384 on one engine have run,
// 65536 had not come back after 90 s.  4096 leave each at least 256 bytes of a 1 MiB queue.
constexpr size_t kMaxRequests = 4096;

// Images up to these sizes (one chunk group, pinned) are packed straight into
// host memory: the kernels write over the link at its full rate (57 GB/s), and
// a DMA request costs ~10 us before its first byte.  Trigger to commit in us,
// DMA -> kernel, 64 KiB and 1 MiB chunks: staged, 64 KiB 53 -> 46, 1 MiB
// 72 -> 50/57, 2 MiB 90 -> 71/76, 4 MiB 130 -> 113/123, 8 MiB 204 -> 236; the
// gate waits for the kernel, so the line lies where that is still less than a
// DMA snapshot of nothing.  In direct mode, where each fragment is a request of
// ~9 us and the gate waits for the copies either way, larger images too when
// their pieces are at most kInKernelPiece on average: the kernel holds compute
// units, and GEMMs beside it lose half as long as it runs.  Snapshot / what
// 4096^3 bf16 products lost by it, in us, DMA -> kernel: 2 MiB in 8 fragments
// 116/2 -> 82/23, 4 MiB in 8 156/4 -> 117/53, in 64 420/3 -> 117/53, 8 MiB in 8
// 235/5 -> 218/110, 16 MiB in 8 400/4 -> 363/178, in 64 650/33 -> 362/177, in 240
// 1460/10 -> 358/182.  (Staged, 1 MiB 74/2 -> 63/9, 2 MiB 97/0 -> 80/21.)
constexpr uint64_t kInKernelImage = 2ull << 20;
constexpr uint64_t kInKernelDirect = 16ull << 20;
constexpr uint64_t kInKernelPiece = 80ull << 10;
// Whether a pinned image of one group is written by the pack kernel; pieces:
// fragment pieces of direct D2H, 0 = full staging.
inline bool in_kernel_size(uint64_t image_bytes, uint64_t pieces)
{
    return image_bytes <= kInKernelImage ||
           (image_bytes <= kInKernelDirect && image_bytes <= pieces * kInKernelPiece);
}

// GPU-side resources of one snapshot record, recycled between snapshots.
struct RecRes {
    std::vector<hipEvent_t> captured;   // per group, on the pack stream
    std::vector<hsa_signal_t> dep;      // per group: set to 0 by the GPU once g is packed
    std::vector<int64_t*> dep_val;      // value addresses of dep
    std::vector<hsa_signal_t> copied;   // per group: the group's image copy finished
    std::vector<hsa_signal_t> flagged;  // per group: the area-done copy after it finished
    std::vector<hsa_signal_t> piece_done; // direct D2H, per piece but each group's last (whose copy
                                          // signals `copied`): the piece's copy finished;
                                          // else per group: the copy of its second share (issue_halves)
    hsa_signal_t dep_lead{0};           // the first group's lead (lead_bytes) packed
    hsa_signal_t lead_done{0};          // ... and copied
    int64_t* dep_lead_val = nullptr;
    hsa_signal_t dep_sums{0}, done{0};  // sums packed; sums copied (the last copy issued)
    int64_t* dep_sums_val = nullptr;
    uint64_t* h_seq = nullptr;          // pinned, per group: area use number, source of the area-done copy
    unsigned long long* d_sums = nullptr;
    std::vector<hipEvent_t> k0, k1;     // timing: around each pack launch
    hipEvent_t t0 = nullptr;
    hipEvent_t t_pieces = nullptr;      // timing: after the kernel copy of the first group's small pieces
    hipEvent_t t_red = nullptr;         // timing: after the chunk-sum reduce and its release
    bool in_kernel = false;             // this snapshot's kernels write the host image themselves (no copies):
                                        // it is done when dep_sums is 0
    std::atomic<uint32_t> landed{0};    // bounce mode: groups moved from the ring into the image
    std::atomic<bool> failed{false};    // bounce mode: a copy of this record could not be completed
    std::atomic<bool> recorded{false};  // image file: the commit record has been written
    // Timing, in the HSA system timestamp domain (that of the DMA engines'
    // copy timestamps): when the last group landed in the pageable image,
    // and when the commit record was written (0 = not yet).
    std::atomic<uint64_t> landed_ts{0};
    std::atomic<uint64_t> recorded_ts{0};
};

struct SnapRec {
    uint64_t id = 0, step = 0;
    int buf = -1;
    bool bounce = false;    // the image is pageable; groups land through the bounce ring
    bool file = false;      // the image lives in the image file: committed once its record is written
    bool aborted = false;
    bool committed = false; // cached once `done` has reached 0
    bool timed = false;
    bool per_launch = false; // timed with events around every pack launch (else around the first only)
    uint32_t groups_copied = 0;
    std::vector<uint8_t> meta;
    RecRes* res = nullptr;
};

struct OpTiming {
    bool valid = false;
    ckpt_timing t{};
};

// Host threads that copy between host buffers in parallel (bounce mode).
// copy() cuts one copy into parts, queues all but the first, runs the
// first itself, and returns when every part is done; several threads may
// call it at once.
class CopyPool {
public:
    explicit CopyPool(unsigned n) : n_(std::max(1u, n))
    {
        for (unsigned k = 0; k + 1 < n_; ++k) th_.emplace_back([this] { work(); });
    }
    ~CopyPool()
    {
        {
            std::lock_guard<std::mutex> l(m_);
            stop_ = true;
        }
        cv_.notify_all();
        for (auto& t : th_) t.join();
    }
    void copy(uint8_t* dst, const uint8_t* src, uint64_t n)
    {
        const uint64_t min_part = 4ull << 20;
        uint64_t parts = std::min<uint64_t>(n_, std::max<uint64_t>(1, n / min_part));
        if (parts <= 1) {
            std::memcpy(dst, src, n);
            return;
        }
        const uint64_t per = (n / parts + 4095) & ~4095ull;
        Batch b;
        b.left = 0;
        {
            std::lock_guard<std::mutex> l(m_);
            for (uint64_t k = 1; k < parts; ++k) {
                const uint64_t lo = std::min(k * per, n), hi = std::min(lo + per, n);
                if (hi <= lo) continue;
                q_.push_back(Part{dst + lo, src + lo, hi - lo, &b});
                ++b.left;
            }
        }
        cv_.notify_all();
        std::memcpy(dst, src, std::min(per, n));
        std::unique_lock<std::mutex> l(b.m);
        b.cv.wait(l, [&] { return b.left == 0; });
    }

private:
    struct Batch {
        unsigned left;
        std::mutex m;
        std::condition_variable cv;
    };
    struct Part {
        uint8_t* dst;
        const uint8_t* src;
        uint64_t n;
        Batch* b;
    };
    void work()
    {
        for (;;) {
            Part p;
            {
                std::unique_lock<std::mutex> l(m_);
                cv_.wait(l, [&] { return stop_ || !q_.empty(); });
                if (q_.empty()) return;
                p = q_.front();
                q_.pop_front();
            }
            std::memcpy(p.dst, p.src, p.n);
            std::lock_guard<std::mutex> l(p.b->m);
            if (--p.b->left == 0) p.b->cv.notify_all();
        }
    }
    unsigned n_;
    std::mutex m_;
    std::condition_variable cv_;
    std::deque<Part> q_;
    bool stop_ = false;
    std::vector<std::thread> th_;
};

// One group of a snapshot on its way through the bounce ring, or (sums)
// the snapshot's chunk-sum copy, which follows its groups.
struct PumpItem {
    RecRes* res = nullptr;
    uint32_t g = 0;
    bool sums = false;               // the chunk sums: device -> pinned sums array, no ring slot
    uint8_t* image = nullptr;        // destination: pageable host image (group) or pinned sums array
    const uint8_t* staging = nullptr; // source in device memory (null in direct mode: the pieces)
    uint64_t lo = 0;                 // group: image offset of its first byte
    uint64_t n = 0;
    uint64_t* area_done = nullptr;   // group: device counter bumped once the staging area has been read
    const uint64_t* seq = nullptr;   // group: pinned, the value it is set to
    hsa_amd_sdma_engine_id_t engine{};
    uint32_t groups = 0;             // record: the snapshot's group copies
    int buf = 0;                     // host image written
    bool record = false;             // image file: write the snapshot's commit record (no copy)
    uint64_t need_rec = 0;           // sums: records of image buf that must be written before its sums array is reused
    uint64_t snap_id = 0, step = 0;
    std::shared_ptr<const std::vector<uint8_t>> meta;
};

// Image file (ckpt_image_file): the two images, their sums and commit
// records in one shared mapping.  Layout: FileHead at 0, FileRec b at
// kRecOff + 512 * b, then per image its sums, its caller blob area and (2 MiB
// aligned) its bytes.
struct FileHead {
    char magic[8]; // "CKPTFIL1"
    uint32_t version, align;
    uint64_t chunk, image_bytes, n_chunks;
    uint32_t n_frag, pad;
    uint64_t table_sum; // word-sum of the fragment table (offset, bytes, dtype, class per fragment)
    uint64_t image_off[2], sums_off[2], meta_off[2];
    uint64_t file_bytes;
};
struct FileRec {
    uint64_t state;   // 1 = committed; stored last, 0 before the image is rewritten
    uint64_t seq;     // commit number: of two valid records the larger is the newest
    uint64_t snap_id, step, meta_len;
    uint64_t rec_sum; // word-sum of seq, snap_id, step, meta_len, the chunk sums and the zero-padded blob
};
constexpr uint64_t kRecOff = 4096;

// Bounce-mode D2H (one per context).  The issuer takes snapshot groups in
// order, waits for a free ring slot, and starts the DMA staging -> slot
// (after the group's pack, through its dependency signal) followed by the
// staging area's use-counter copy.  The drainer takes them in the same
// order, waits for each DMA, copies slot -> image on the copy pool, frees
// the slot and counts the group as landed.
//
// Every DMA of bounce mode is issued by the issuer, in snapshot and group
// order.  Each engine runs its requests in order, and a request waiting for
// a pack blocks the requests behind it; issuing the chunk-sum copy (which
// waits for the last pack) ahead of group copies that earlier packs depend
// on -- through the staging counters -- would stall the engine for good.
struct Pump {
    std::mutex m;
    std::condition_variable cv;
    std::deque<PumpItem> issue_q;
    std::deque<std::pair<PumpItem, uint64_t>> drain_q;
    std::vector<uint8_t> busy; // per ring slot
    uint64_t next_slot = 0;
    uint64_t rec_pushed[2] = {0, 0}, rec_done[2] = {0, 0}; // image-file commit records per host image
    bool stop = false;
    bool failed = false;
    std::string err;
    std::thread issuer, drainer;
};

// H2H replication (paper Sec. V-B, "Host-to-host"): one job per snapshot,
// handed to the worker when the snapshot is issued.  The worker waits for
// the local commit, sends the replicated chunks with their sums and the
// envelope, and waits for the peer's acknowledgement.
struct RepJob {
    uint64_t id = 0, step = 0;
    int buf = 0;
    RecRes* res = nullptr;
    uint32_t groups_copied = 0;
    bool bounce = false;
    std::vector<uint8_t> meta;
};

enum { REP_PENDING = 0, REP_OK = 1, REP_CORRUPT = 2, REP_FAILED = 3 };

struct RepStatus {
    int state = REP_PENDING;
    std::vector<uint64_t> bad; // sender chunk ids the peer found corrupt
    std::string err;
};

struct Replicator {
    int fd = -1;
    uint64_t first_id = 0; // the first snapshot this peer receives (peers may be added later)
    uint64_t cls_mask = 0;
    std::vector<uint64_t> ids; // replicated chunks, increasing
    uint64_t bytes = 0;        // replica bytes per snapshot
    std::mutex m;
    std::condition_variable cv;
    std::deque<RepJob> q;
    std::map<uint64_t, RepStatus> status;
    bool busy[2] = {false, false}; // a replication still reads host image b
    bool stop = false;
    bool broken = false; // the connection failed: later jobs fail at once
    std::string err;
    int fault_kind = 0;  // debug: 1 = flip one bit of the next stream, 2 = cut the next stream
    uint64_t fault_a = 0, fault_b = 0;
    double last_send_ms = 0, last_ack_ms = 0; // commit -> last byte sent, commit -> acknowledgement
    std::thread worker;
};

// What the last ckpt_restore_from_peer fetched.
struct PeerRestore {
    bool valid = false;
    uint64_t snap_id = 0, step = 0;
    std::vector<uint64_t> ids; // chunks written
    std::vector<uint8_t> envelope;
    double fetch_ms = 0, check_ms = 0;
};

} // namespace ckpt

using namespace ckpt;

struct ckpt_ctx {
    // configuration
    int device = 0;
    uint64_t C = kDefaultChunk;
    uint32_t A = kDefaultAlign;
    uint64_t staging_cap = 0; // 0 = full image
    uint64_t group_cfg = kDefaultGroup;
    bool group_set = false; // group_bytes given explicitly (ring mode: slots of that many bytes)
    uint32_t grid_cap = kDefaultGrid;
    bool timing = false;
    bool timing_span = false; // timing level 2: a snapshot's first launch and pack-stream end only

    // layout
    bool registered = false;
    std::vector<Frag> frags;
    uint64_t I = 0, n_chunks = 0, payload = 0;
    Geometry geo{};
    uint64_t G = 1;        // chunks per group
    uint64_t n_groups = 0; // groups
    uint64_t launch_cfg = kDefaultLaunch;
    uint64_t LG = 1;         // groups per pack launch (1 in ring mode)
    uint64_t n_launches = 0; // pack launches per snapshot
    bool ring = false;
    uint64_t n_slots = 0;  // ring slots of G chunks each (ring mode)
    bool direct = false;   // direct D2H: no snapshot staging, the engines copy the fragments
    std::vector<Piece> pieces, gaps;              // direct D2H, by group (CSR below)
    std::vector<uint64_t> piece_first, gap_first; // [n_groups + 1]
    std::vector<uint8_t> piece_chain;             // per piece: which of its group's two chains of copies it is in
    std::vector<uint64_t> other_last;             // per group: last piece of the chain that does not end with the
                                                  // group's last piece (UINT64_MAX: a single chain)
    std::vector<uint64_t> small_first;            // [n_groups + 1]: the pieces that a kernel copies instead

    // device memory
    FragDev* d_frags = nullptr;
    Piece* d_small = nullptr;                 // direct D2H: the small pieces, by group
    uint64_t* d_tile_src = nullptr;           // per tile: tile_entry()
    uint8_t* d_staging = nullptr;
    unsigned long long* d_partials = nullptr; // [2][n_tiles] tile partial sums: pack, check
    uint32_t* d_ticket = nullptr;             // launch_pack_chunks' (behind the counters)
    uint64_t* d_area_done = nullptr;          // per staging area (direct D2H: per group): number of
                                              // finished copies out of it

    // pinned host memory
    uint8_t* h_img[2] = {nullptr, nullptr};
    uint64_t* h_sums[2] = {nullptr, nullptr};
    uint64_t holder[2] = {0, 0}; // snapshot id whose bytes each image holds (0 = none)
    uint8_t* h_bad = nullptr;                   // written by the chunk-sum compare
    unsigned long long* h_recomputed = nullptr; // "

    // HSA agents and DMA engines
    hsa_agent_t gpu_agent{0}, img_agent[2] = {{0}, {0}};
    hsa_amd_sdma_engine_id_t d2h_engine[kMaxEngines];
    int n_d2h_engines = 0;
    uint32_t d2h_engines_cfg = 0; // 0 = all available (up to kMaxEngines)
    bool poison = false;          // fill each staging area with the canary before it is packed again
    hsa_amd_sdma_engine_id_t h2d_engine{};
    uint64_t ts_freq = 1;

    // streams and events
    hipStream_t s_pack = nullptr;
    bool own_pack = true; // false: s_pack is the caller's side stream (never destroyed here)
    hipEvent_t ev_trigger = nullptr, ev_done = nullptr;
    std::vector<uint64_t> area_seq;     // per staging area: copies issued out of it
    std::vector<hsa_signal_t> area_flag; // per staging area: completion signal of its latest counter copy
                                         // (0 once that copy, and the image copy before it, are done)
    std::vector<RecRes*> free_res;
    std::map<uint64_t, SnapRec> recs;
    uint64_t next_id = 1;
    int32_t interrupt_next = -1;

    // results of the last restore / verify
    bool have_last_sums = false;
    std::vector<uint64_t> last_sums;
    OpTiming op_timing[3];
    std::vector<hipEvent_t> tk0, tk1; // restore timing
    hipEvent_t tt0 = nullptr;

    // bounce mode: pageable images behind two pinned rings of chunk groups
    bool bounce = false;
    uint64_t bounce_cfg = 0;
    uint32_t host_threads = kDefaultHostThreads;
    uint64_t n_bslots = 0;            // slots per ring
    uint64_t img_map_bytes = 0;       // mapped length of each pageable image
    uint8_t* h_bout = nullptr;        // device -> host ring
    uint8_t* h_bin = nullptr;         // host -> device ring
    std::vector<hipEvent_t> bin_done; // per host -> device slot: the kernel or copy that last read it has finished
    CopyPool* pool = nullptr;
    Pump* pump = nullptr;

    // H2H replication to ring peers (k distinct peers, in the order they were added)
    std::vector<Replicator*> reps;

    // the last restore from a ring peer's replica
    PeerRestore peer_restore;

    // image file (crash-surviving images; bounce mode only)
    std::string file_path;
    int file_mode = -1; // -1 none, else CKPT_FILE_CREATE / CKPT_FILE_ADOPT
    int file_fd = -1;
    uint8_t* file_map = nullptr;
    FileHead fhead{};
    uint64_t file_seq = 0; // last commit number written (drainer thread after registration)

    // verify: its own device ring and streams
    uint8_t* d_vring = nullptr;
    uint64_t vslot_chunks = 1, n_vslots = 0;
    hipStream_t s_vcopy[2] = {nullptr, nullptr}, s_vker = nullptr;
    hipEvent_t ev_vdone = nullptr, vt0 = nullptr, vc1 = nullptr;
    std::vector<hipEvent_t> vfree, vloaded; // per slot: read by the kernel, filled
    std::vector<hipEvent_t> vk0, vk1;       // per launch, timing

    std::string err;
};

namespace ckpt {

// Record `fmt` as the context's last error and return `code`.
ckpt_status fail(ckpt_ctx* c, ckpt_status code, const char* fmt, ...);
const char* hsa_text(hsa_status_t s);

#define HIPCHK(ctx, expr)                                                                                    \
    do {                                                                                                     \
        hipError_t e_ = (expr);                                                                              \
        if (e_ != hipSuccess)                                                                                \
            return fail((ctx), CKPT_EHIP, "%s failed: %s (%d)", #expr, hipGetErrorString(e_), (int)e_);       \
    } while (0)

#define HSACHK(ctx, expr)                                                                                    \
    do {                                                                                                     \
        hsa_status_t s_ = (expr);                                                                            \
        if (s_ != HSA_STATUS_SUCCESS)                                                                        \
            return fail((ctx), CKPT_EHIP, "%s failed: %s (%d)", #expr, hsa_text(s_), (int)s_);               \
    } while (0)

uint64_t round_up(uint64_t x, uint64_t a);
bool geometry_ok(uint64_t C, uint32_t A);

// Chunk group g: image bytes [group_lo, group_hi), tiles [tiles_lo,
// tiles_hi), its staging area (a ring slot, or its own place in the full
// device image) and where that area starts.
inline uint64_t group_lo(const ckpt_ctx* c, uint64_t g) { return g * c->G * c->C; }
inline uint64_t group_hi(const ckpt_ctx* c, uint64_t g) { return std::min((g + 1) * c->G * c->C, c->I); }
// Whether group g's staged copy is dealt to two engines.
inline bool in_halves(const ckpt_ctx* c, uint64_t g)
{
    return split_copy(group_hi(c, g) - group_lo(c, g), c->n_d2h_engines, c->bounce ? 0 : c->n_groups, c->G * c->C);
}
// Bytes of the first group that a launch of their own packs ahead of the rest
// (0: none), whole tiles; full-image staging only.
inline uint64_t lead_bytes(const ckpt_ctx* c)
{
    return !c->ring && !c->direct && !c->poison && group_hi(c, 0) >= 4 * kLead ? kLead : 0;
}
inline uint64_t tiles_lo(const ckpt_ctx* c, uint64_t g) { return group_lo(c, g) >> c->geo.tile_shift; }
inline uint64_t tiles_hi(const ckpt_ctx* c, uint64_t g)
{
    return (group_hi(c, g) + (1ull << c->geo.tile_shift) - 1) >> c->geo.tile_shift;
}
inline uint64_t area_of(const ckpt_ctx* c, uint64_t g) { return c->ring ? g % c->n_slots : g; }
inline uint8_t* staging_of(const ckpt_ctx* c, uint64_t g)
{
    return c->ring ? c->d_staging + (g % c->n_slots) * c->G * c->C : c->d_staging + group_lo(c, g);
}

ckpt_status make_event(ckpt_ctx* c, hipEvent_t* e, bool timed);
// Milliseconds between two recorded timing events (-1 when unavailable).
float elapsed(hipEvent_t a, hipEvent_t b);
// Issue one SDMA copy of n bytes on `engine`, after the n_dep signals at dep
// (when non-null), completing into `completion`.
ckpt_status dma(ckpt_ctx* c, void* dst, hsa_agent_t dst_agent, const void* src, hsa_agent_t src_agent, uint64_t n,
                const hsa_signal_t* dep, hsa_signal_t completion, hsa_amd_sdma_engine_id_t engine,
                uint32_t n_dep = 1);
// Text of this thread's last failed ckpt_pack_noalloc ("" if none).
const char* noalloc_error();

// Snapshot records (ckpt_runtime.cpp)
ckpt_status get_res(ckpt_ctx* c, RecRes** out);
// Wait until every snapshot's copies have finished and the library's
// streams are idle.
ckpt_status drain(ckpt_ctx* c);
// The host image the next snapshot would fill (EBUSY while a snapshot is
// uncommitted or that image is being sent to the peer).
ckpt_status pick_target_image(ckpt_ctx* c, int* out);
// Restore (scatter) or verify host image b against h_sums[b] (ckpt_check.cpp): all chunks,
// or only `ids` (increasing).  Fills the bad list like ckpt_restore.  With
// `fill`, each span [lo, hi) of image bytes is first handed to fill, which
// puts them in place (the host -> device work of earlier spans runs
// meanwhile); false from fill ends the operation with EHIP once the work
// already issued has finished (the caller records the error text).
ckpt_status check_image(ckpt_ctx* c, int b, hipStream_t stream, bool scatter, const std::vector<uint64_t>* ids,
                        uint32_t* bad_chunks, uint32_t cap, uint32_t* n_bad,
                        const std::function<bool(uint64_t, uint64_t)>& fill = nullptr);
bool res_done(const RecRes* res, uint32_t groups_copied, bool bounce);
void parallel_zero(uint8_t* p, uint64_t n);
std::vector<uint8_t> build_envelope(const ckpt_ctx* c, uint64_t step, const std::vector<uint8_t>& meta,
                                    const uint64_t* sums);

// Issue snapshot r (ckpt_snapshot.cpp): its kernels on the pack stream after
// the work already on `after`, and its copies; groups from n_copy on stay on
// the device, and stop >= 0 marks the snapshot interrupted (never committed).
ckpt_status issue_snapshot(ckpt_ctx* c, SnapRec& r, hipStream_t after, uint64_t n_copy, int32_t stop);

// Direct D2H: zero group g's padding runs in `dst` (host memory holding the
// group's first image byte at dst), then copy its fragment pieces into place,
// those of chain e on engine[e], each after the previous one of its chain
// (the first after first_dep); the group's last piece signals
// res->copied[g].  Returns the pieces issued: fewer than the group's means a
// copy could not be issued (ckpt_snapshot.cpp).
uint64_t issue_pieces(ckpt_ctx* c, RecRes* res, uint64_t g, uint8_t* dst, hsa_agent_t dst_agent,
                      const hsa_signal_t* first_dep, const hsa_amd_sdma_engine_id_t engine[2]);
// Copy group g, n bytes at src (device staging) to dst (pinned), after *dep:
// its shares on the two engines, or in one request when it is small or there is
// one engine; with lead > 0 (two engines, less than a share) the first `lead`
// bytes of the first share go ahead, after res->dep_lead.  Returns the signals
// of group_signals() that will be lowered: fewer means that a request could not
// be issued (the signals of what was not issued are 0).
int issue_halves(ckpt_ctx* c, RecRes* res, uint64_t g, uint8_t* dst, hsa_agent_t dst_agent, const uint8_t* src,
                 uint64_t n, const hsa_signal_t* dep, uint64_t lead = 0);
// Wait (bounded) until the first `got` pieces of group g have been copied.
void wait_pieces(ckpt_ctx* c, RecRes* res, uint64_t g, uint64_t got);
// The signals that reach 0 once group g's image copies have finished: `copied`,
// and the end of the group's other chain or its second half.  Returns how many.
int group_signals(const ckpt_ctx* c, const RecRes* res, uint64_t g, hsa_signal_t out[2]);

// Bounce mode (ckpt_bounce.cpp)
bool poll_zero(hsa_signal_t sig, int seconds);
void pump_issue(ckpt_ctx* c);
void pump_drain(ckpt_ctx* c);
void stop_pump(ckpt_ctx* c);

// Image file (ckpt_file.cpp)
ckpt_status open_image_file(ckpt_ctx* c);
ckpt_status adopt_image_file(ckpt_ctx* c);
void file_invalidate(ckpt_ctx* c, int b);
void file_commit(ckpt_ctx* c, const PumpItem& it);

// Replication to ring peers (ckpt_h2h.cpp)
constexpr size_t kMaxPeers = 8;
void rep_stop(ckpt_ctx* c);
// Whether a replication still reads host image b.
bool rep_busy(ckpt_ctx* c, int b);

} // namespace ckpt
