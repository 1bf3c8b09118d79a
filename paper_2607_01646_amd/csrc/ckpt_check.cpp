// ckpt_check.cpp -- restore and verify of a committed host image (paper
// Sec. V-C third stage, Sec. VI-E).  Restore's scatter kernel reads the image
// where it lies in pinned host memory, over the host link: nothing is staged
// on the device, and the bytes' way over the link, the writes into the
// fragments and the sums run at the same time.  Verify runs beside training,
// so there a DMA engine brings the image to a small device ring and the
// checksum kernel reads it from there: a kernel that reads over the link
// holds its compute units for the whole transfer, and a GEMM with one
// workgroup for every unit then takes two rounds (4096^3 in bf16 beside
// verifies of 1.5 GB: +62% with 24 workgroups on the link, 27.5 ms a verify;
// +3% with the ring, 28.0 ms).  The chunk-sum compare of both reads the
// stored sums and writes its results in host memory.
#include "ckpt_host.h"

namespace ckpt {

// Restore (scatter=true) or verify (scatter=false) the chunks of host image
// b against the sums in h_sums[b]: every chunk, or only the chunks `ids`
// (increasing) when given.  The caller has checked the arguments and, for a
// restore, drained every snapshot.
ckpt_status check_image(ckpt_ctx* c, int b, hipStream_t stream, bool scatter, const std::vector<uint64_t>* ids,
                        uint32_t* bad_chunks, uint32_t cap, uint32_t* n_bad,
                        const std::function<bool(uint64_t, uint64_t)>& fill)
{
    const int op = scatter ? CKPT_OP_RESTORE : CKPT_OP_VERIFY;
    hipStream_t s = scatter ? c->s_pack : c->s_vker;
    const hipEvent_t done = scatter ? c->ev_done : c->ev_vdone, t0 = scatter ? c->tt0 : c->vt0;
    const std::vector<hipEvent_t>&k0 = scatter ? c->tk0 : c->vk0, &k1 = scatter ? c->tk1 : c->vk1;
    // Byte spans, one launch each: runs of consecutive chunks, cut at the
    // size of a chunk group when the host puts the bytes in place span by span
    // (bounce slots, bytes arriving from a peer), and of a ring slot for verify.
    uint64_t most = c->bounce || fill ? c->G : c->n_chunks;
    if (!scatter) most = std::min(most, c->vslot_chunks);
    std::vector<std::pair<uint64_t, uint64_t>> spans;
    if (!ids) {
        for (uint64_t k = 0; k < c->n_chunks; k += most)
            spans.emplace_back(k * c->C, std::min((k + most) * c->C, c->I));
    } else {
        for (size_t j = 0; j < ids->size();) {
            size_t k = j + 1;
            while (k < ids->size() && (*ids)[k] == (*ids)[k - 1] + 1 && k - j < most) ++k;
            spans.emplace_back((*ids)[j] * c->C, std::min(((*ids)[k - 1] + 1) * c->C, c->I));
            j = k;
        }
    }
    const uint64_t n_spans = spans.size(), slot_bytes = c->G * c->C;
    const bool timed = c->timing && !ids; // timing is kept for whole-image operations only
    unsigned long long* partials = c->d_partials + c->geo.n_tiles;
    const uint32_t grid = scatter ? std::min(c->grid_cap, kRestoreGrid) : c->grid_cap;
    const uint64_t vslot_bytes = c->vslot_chunks * c->C;
    if (scatter) {
        HIPCHK(c, hipEventRecord(c->ev_trigger, stream));
        HIPCHK(c, hipStreamWaitEvent(s, c->ev_trigger, 0));
    }
    if (timed) HIPCHK(c, hipEventRecord(t0, scatter ? s : c->s_vcopy[0]));
    for (uint64_t u = 0; u < n_spans; ++u) {
        const uint64_t lo = spans[u].first, hi = spans[u].second;
        if (fill && !fill(lo, hi)) { // the span's bytes did not arrive: let the issued work finish, then fail
            (void)hipStreamSynchronize(s);
            return CKPT_EHIP;
        }
        const uint8_t* src = c->h_img[b] + lo;
        if (c->bounce) { // pageable image: through a pinned ring slot, free once what read it has finished
            const uint64_t slot = u % c->n_bslots;
            if (u >= c->n_bslots) HIPCHK(c, hipEventSynchronize(c->bin_done[slot]));
            c->pool->copy(c->h_bin + slot * slot_bytes, src, hi - lo);
            src = c->h_bin + slot * slot_bytes;
        }
        if (!scatter) {
            // The host paces the ring: it waits for the kernel that last read
            // the slot, so that the copies follow each other with no wait of
            // the device's between them (which cost ~6% of the link).  They
            // alternate between two streams: one stream starts a copy ~15 us
            // after its last one.
            const uint64_t slot = u % c->n_vslots;
            hipStream_t cs = c->s_vcopy[u % 2];
            uint8_t* ring = c->d_vring + slot * vslot_bytes;
            HIPCHK(c, hipEventSynchronize(c->vfree[slot]));
            HIPCHK(c, hipMemcpyAsync(ring, src, hi - lo, hipMemcpyHostToDevice, cs));
            if (c->bounce) HIPCHK(c, hipEventRecord(c->bin_done[u % c->n_bslots], cs));
            if (timed && u + 1 == n_spans) HIPCHK(c, hipEventRecord(c->vc1, cs));
            HIPCHK(c, hipEventRecord(c->vloaded[slot], cs));
            HIPCHK(c, hipStreamWaitEvent(s, c->vloaded[slot], 0));
            src = ring;
        }
        const uint64_t t_lo = lo >> c->geo.tile_shift, t_hi = (hi + (1ull << c->geo.tile_shift) - 1) >> c->geo.tile_shift;
        hipEvent_t e0 = timed ? k0[u] : nullptr, e1 = timed ? k1[u] : nullptr;
        hipError_t e;
        if (scatter)
            e = launch_scatter(c->d_frags, c->d_tile_src, c->geo, t_lo, t_hi, src, lo, partials, grid, s, e0, e1);
        else
            e = launch_checksum(c->geo, t_lo, t_hi, src, lo, partials, grid, s, e0, e1);
        if (e != hipSuccess) return fail(c, CKPT_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
        if (scatter && c->bounce) HIPCHK(c, hipEventRecord(c->bin_done[u % c->n_bslots], s));
        if (!scatter) HIPCHK(c, hipEventRecord(c->vfree[u % c->n_vslots], s));
        e = launch_chunk_reduce(c->geo, t_lo, t_hi, partials, c->h_recomputed,
                                (const unsigned long long*)c->h_sums[b], c->h_bad, s);
        if (e != hipSuccess) return fail(c, CKPT_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
    }
    HIPCHK(c, hipEventRecord(done, s));
    if (scatter) HIPCHK(c, hipStreamWaitEvent(stream, done, 0));
    HIPCHK(c, hipEventSynchronize(done));
    if (timed) {
        ckpt_timing t{};
        for (uint64_t u = 0; u < n_spans; ++u) t.kernel_ms += elapsed(k0[u], k1[u]);
        t.kernels = (uint32_t)n_spans;
        t.copies = scatter ? 0 : (uint32_t)n_spans;
        t.copy_ms = scatter ? elapsed(k0[0], k1[n_spans - 1]) : elapsed(t0, c->vc1);
        t.total_ms = elapsed(t0, k1[n_spans - 1]);
        t.kernel_bytes = scatter ? 2 * c->payload : c->I;
        t.copy_bytes = c->I;
        t.span_ms = -1.f;
        c->op_timing[op].t = t;
        c->op_timing[op].valid = true;
    }
    uint32_t nb = 0;
    auto flag = [&](uint64_t k) {
        if (!c->h_bad[k]) return;
        if (nb < cap) bad_chunks[nb] = (uint32_t)k;
        ++nb;
    };
    if (ids) {
        for (uint64_t k : *ids) flag(k);
    } else {
        c->last_sums.assign(c->h_recomputed, c->h_recomputed + c->n_chunks);
        c->have_last_sums = true;
        for (uint64_t k = 0; k < c->n_chunks; ++k) flag(k);
    }
    *n_bad = nb;
    if (nb)
        return fail(c, CKPT_ECORRUPT, "%u of %llu chunks failed their checksum", nb,
                    (unsigned long long)(ids ? ids->size() : c->n_chunks));
    return CKPT_OK;
}

} // namespace ckpt
