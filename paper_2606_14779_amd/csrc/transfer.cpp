// Store / retrieve engine of the KV pool.
//
// Retrieval follows Sec. 4.3 of the paper: look every block up, group the
// blocks by pool device, and read all devices in parallel.  Here the groups
// are the two region classes -- pinned host regions, read by a zero-copy
// kernel over the host link (or by the copy engines through an HBM ring), and
// HBM staging regions, read by an HBM gather kernel.  "In parallel" means the
// two classes are workgroups of one launch on the caller's stream (or, where
// each class is timed or a class needs LDS, two kernels, the staging one forked
// onto the pool's internal stream and joined again), so the caller sees one
// stream-ordered operation.  The store (Alg. 1, offload) is the same path in
// the other direction.  The per-call work list (the engine-buffer pointers of
// the moved chunks, then one 16-byte item per block) travels in the kernel
// arguments when it is small enough; otherwise it is written to a pinned buffer
// and uploaded by a small kernel ahead of the call's.  Those buffers come from a
// ring guarded by events, so a call only blocks when the ring wraps onto work
// that is still running.

#include <algorithm>
#include <cmath>
#include <unordered_map>

#include "internal.hpp"

namespace kvp {

namespace {

constexpr size_t kSlotMin = 64 * 1024;   // smallest work-list buffer
// Two kernels for the two classes: staging-class bytes below which the HBM
// kernel runs on the caller's stream ahead of the host-class kernel instead of
// being forked.  Forking costs about 25 us of host time per call, more than
// such a kernel takes (32 MiB read and written at ~2.5 TB/s copied: ~13 us).
constexpr uint64_t kForkMinBytes = 32ull << 20;
// Host-class retrieve workgroups while a host-class store of this pool is in
// flight.  Under two-way traffic the reads need more in flight: a 128K-token
// LLaMA-shaped store and retrieve started together took 264.6 ms with 48
// against 320 ms with the 12 that a lone retrieve wants (which, beside HBM-bound
// work, loses with more).  Started 100 ms apart the link serves the later one
// first with any of them (store / retrieve, the store first: 328 / 220 ms with 48,
// 277 / 233 with 12).
constexpr uint32_t kDuplexReadGrid = 48;
constexpr uint64_t kMergeLdsMax = 20 * 1024;   // 160 KiB of LDS hold 8 workgroups of this size
constexpr uint64_t kHbmPerLink = 54;           // bytes that HBM moves while the link moves one

// Host-class store workgroups beside a staging-class store that takes longer.
// The link's posted writes fill the write path that the HBM kernel shares, and
// the more of them wait, the slower it gets, so the host class takes only the
// workgroups with which it ends in about two thirds of the staging class's
// time, a third of its own choice at least.  4096 Qwen3-shaped blocks on
// measured weights, 20 of them over the link (27 % of the staging class's time
// alone), took 2400 us with 12 host workgroups, 2193 with 8, 2166 with 3 to 6,
// 2177 with 2 and 2700 with 1.  Over three shapes, both pool layouts and link
// times of 2 to 95 % of HBM's (2 GB in HBM each) the rule is nowhere over 1 %
// slower than all workgroups, and gains 1 to 14 % up to 45 % (27 %: 689 against 737 us
// head-major, 704 against 751 token-major).  It is not the best choice above that:
// half of the workgroups take 655 and 692 us at 45 and 60 %, the rule 753 and
// 840.  A retrieve's reads don't have this effect (2183-2208 us with 12, 2182
// with 6).
uint32_t throttled_store_grid(uint32_t grid, uint64_t host_bytes, uint64_t staging_bytes)
{
    const double share = static_cast<double>(kHbmPerLink * host_bytes) / static_cast<double>(staging_bytes);
    const uint32_t least = (grid + 2) / 3;
    return std::max(least, static_cast<uint32_t>(std::min<double>(grid, std::floor(1.5 * share * grid) + 1)));
}

// The live allocation holding the block at map entry e, or an error.
const Allocation *resolve(const Pool &p, const kvp_loc &e, uint32_t b, const Allocation *hint)
{
    const uint32_t N = static_cast<uint32_t>(p.regions.size());
    if (e.region >= N)
        fail(KVP_ERR_INVALID, "map entry " + std::to_string(b) + ": region " + std::to_string(e.region) +
                                  " out of range");
    const Region &r = p.regions[e.region];
    if (e.offset % 16 != 0 || e.offset > r.capacity || r.capacity - e.offset < p.block_bytes)
        fail(KVP_ERR_INVALID, "map entry " + std::to_string(b) + ": offset outside region");
    const Allocation *a = hint;
    if (!(a && a->region == e.region && e.offset >= a->base && e.offset < a->base + a->blocks * p.block_bytes)) {
        auto it = r.live.upper_bound(e.offset);
        if (it == r.live.begin()) fail(KVP_ERR_STALE, "map entry " + std::to_string(b) + ": no live placement there");
        a = std::prev(it)->second;
        if (e.offset >= a->base + a->blocks * p.block_bytes)
            fail(KVP_ERR_STALE, "map entry " + std::to_string(b) + ": no live placement there");
    }
    if ((e.offset - a->base) % p.block_bytes != 0 || a->gen != e.gen)
        fail(KVP_ERR_STALE, "map entry " + std::to_string(b) + ": stale generation or block boundary");
    return a;
}

// Staging-class work items in the order in which the kernel's written side
// runs on: a retrieve's by engine slot, a store's region by region (a request's
// blocks of a region are one range, while a striped map alternates between
// regions); stable.  Pages and DRAM rows of that side are then met once,
// whatever the block table's order is, and the other side loses nothing, since
// a block is itself a contiguous megabyte or so.  HBM traffic of 8192 GPT-OSS
// shaped blocks retrieved with a permuted table: 5321 GB/s in table order, 5901
// in slot order; of 4096 Qwen3-shaped blocks stored: 6131 in map order, 6219
// by region.  A radix sort on 11-bit digits: 2 passes cover 4M slots.
void order_items(std::vector<CopyItem> &items, std::vector<CopyItem> &other, bool gather, uint32_t limit)
{
    auto key = [gather](const CopyItem &i) { return gather ? i.slot : i.region; };
    auto less = [&](const CopyItem &x, const CopyItem &y) { return key(x) < key(y); };
    if (std::is_sorted(items.begin(), items.end(), less)) return;
    if (items.size() < 64) {
        std::stable_sort(items.begin(), items.end(), less);
        return;
    }
    constexpr uint32_t kDigit = 11, kMask = (1u << kDigit) - 1;
    other.resize(items.size());
    for (uint32_t shift = 0; shift < 32 && (limit - 1) >> shift; shift += kDigit) {
        uint32_t at[kMask + 1] = {};
        for (const CopyItem &i : items) ++at[key(i) >> shift & kMask];
        uint32_t sum = 0;
        for (uint32_t &c : at) {
            const uint32_t n = c;
            c = sum;
            sum += n;
        }
        for (const CopyItem &i : items) other[at[key(i) >> shift & kMask]++] = i;
        items.swap(other);
    }
}

constexpr size_t kMaxTimedCalls = 4096;

hipEvent_t timing_event(Pool &p)
{
    if (!p.spare.empty()) {
        hipEvent_t e = p.spare.back();
        p.spare.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    check_hip(hipEventCreate(&e), "hipEventCreate");
    return e;
}

bool stream_capturing(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    const bool clean = hipPeekAtLastError() == hipSuccess;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        if (clean) clear_hip_error();   // never an error the caller has yet to read
        return false;
    }
    return st != hipStreamCaptureStatusNone;
}

Slot &acquire_slot(Pool &p, size_t bytes)
{
    Slot &s = p.ring[p.ring_next];
    p.ring_next = (p.ring_next + 1) % static_cast<uint32_t>(p.ring.size());
    wait_call(p, s.call);
    s.call = 0;
    if (s.cap < bytes) {
        free_slot(s);
        const size_t cap = round_up(std::max(bytes, kSlotMin), kSlotMin);
        void *h = nullptr, *d = nullptr;
        if (hipHostMalloc(&h, cap, kListMemory) != hipSuccess || !h) {
            clear_hip_error();
            fail(KVP_ERR_NOMEM, "work-list pinned buffer");
        }
        if (hipMalloc(&d, cap) != hipSuccess || !d) {
            clear_hip_error();
            (void)hipHostFree(h);
            fail(KVP_ERR_NOMEM, "work-list device buffer");
        }
        s.host = h;
        s.dev = d;
        check_hip(hipHostGetDevicePointer(&s.host_dev, h, 0), "hipHostGetDevicePointer");
        s.cap = cap;
    }
    return s;
}

// The file regions' blocks of a call, batch by batch through the pinned ring
// (see fileio.cpp): a retrieve reads a batch's spans by the regions' workers,
// then moves the slot to the engine cache by a kernel on stream `sf`; a store
// fills the slot by a kernel, waits for it, and has the workers write the
// spans while the next batch's kernel runs.  A slot is refilled only after
// its previous kernel and its previous reads or writes are done.  On return
// every read or write is done; on a failure the workers are drained first.
void run_file_batches(Pool &p, bool gather, const std::vector<FileBatch> &batches,
                      const std::vector<FileSpan> &spans, const CopyArgs &a, const LaunchCfg &lc, hipStream_t sf)
{
    auto submit = [&](const FileBatch &bt, bool write) {
        char *slot = p.file_ring + static_cast<uint64_t>(bt.ring) * p.file_slot_bytes;
        for (size_t i = bt.span0; i < bt.span0 + bt.spans; ++i) {
            const FileSpan &sp = spans[i];
            const Region &r = p.regions[sp.region];
            p.workers->submit(r.worker, IoJob{r.fd, write, sp.file_off, sp.len, slot + sp.slot_off, &p.file_io[bt.ring]});
        }
    };
    auto kernel = [&](const FileBatch &bt) {
        CopyArgs k = a;
        k.items = a.items + bt.first;
        k.n_items = bt.n;
        check_hip(launch_chunk_copy(k, kClassFile, gather, lc.grid, lc.flags, sf), "kernel launch");
        check_hip(hipEventRecord(p.file_free[bt.ring], sf), "hipEventRecord");
        p.file_free_rec[bt.ring] = true;
    };
    // the slot is free: its reads or writes and its kernel are done
    auto slot_free = [&](const FileBatch &bt) {
        io_wait(p.file_io[bt.ring]);
        if (p.file_free_rec[bt.ring]) check_hip(hipEventSynchronize(p.file_free[bt.ring]), "hipEventSynchronize");
    };
    try {
        if (gather) {
            // read ahead: the next batch's reads are queued behind this one's (into the
            // other slot) before this one is waited for, so each worker moves on as soon
            // as its own part of a batch is read
            if (!batches.empty()) {
                slot_free(batches[0]);
                submit(batches[0], false);
            }
            for (size_t i = 0; i < batches.size(); ++i) {
                if (i + 1 < batches.size()) {
                    slot_free(batches[i + 1]);
                    submit(batches[i + 1], false);
                }
                io_wait(p.file_io[batches[i].ring]);
                kernel(batches[i]);
            }
        } else {
            for (const FileBatch &bt : batches) {
                slot_free(bt);
                kernel(bt);
                check_hip(hipEventSynchronize(p.file_free[bt.ring]), "hipEventSynchronize");
                submit(bt, true);
            }
        }
        for (auto &g : p.file_io) io_wait(g);
    } catch (...) {
        for (auto &g : p.file_io) io_drain(g);
        p.file_next = static_cast<uint32_t>((p.file_next + batches.size()) % kFileSlots);
        throw;
    }
    p.file_next = static_cast<uint32_t>((p.file_next + batches.size()) % kFileSlots);
}

// A call whose whole list travels in kernel arguments although one launch cannot
// hold it: a series of launches on `s`, each with an equal share of both
// classes' items, so that the two still run side by side, and of the moved
// chunks too if these alone would fill the arguments (over 128 layers).
void launch_in_parts(const CopyArgs &geo, const std::vector<CopyItem> (&items)[2], const std::vector<uint64_t> &table,
                     bool gather, const LaunchCfg &lh, const LaunchCfg &ls, hipStream_t s)
{
    const uint32_t most_chunks = std::min(geo.chunks, 2 * kInlineWords / 3);
    const uint64_t most_items = (kInlineWords - most_chunks) / 2;
    const uint64_t n[2] = {items[0].size(), items[1].size()};
    // each class's share is rounded up by less than one item
    const uint64_t parts = (n[0] + n[1] + most_items - 2) / (most_items - 1);
    for (uint32_t c = 0; c < geo.chunks; c += most_chunks)
        for (uint64_t i = 0; i < parts; ++i) {
            CallArgs f = {};
            f.a = geo;
            f.a.chunk0 += c;
            f.a.chunks = std::min(most_chunks, geo.chunks - c);
            std::copy(table.begin() + c, table.begin() + c + f.a.chunks, f.words);
            auto *list = reinterpret_cast<CopyItem *>(f.words + f.a.chunks), *end = list;
            for (int cls = 0; cls < 2; ++cls) {
                end = std::copy(items[cls].begin() + n[cls] * i / parts, items[cls].begin() + n[cls] * (i + 1) / parts, end);
                if (cls == KVP_CLASS_HOST) f.n_host = static_cast<uint32_t>(end - list);
            }
            f.a.n_items = static_cast<uint32_t>(end - list);
            check_hip(launch_call(f, gather, lh.grid, ls.grid, lh.flags, ls.flags, s), "kernel launch");
        }
}

}  // namespace

// Wait for every recorded call, optionally summarise it, and recycle its events.
void drain_timed(Pool &p, kvp_timing_summary *sum)
{
    kvp_timing_summary s{};
    s.host_ms_min = s.staging_ms_min = -1.f;
    s.host_ms_max = s.staging_ms_max = -1.f;
    for (auto &tc : p.timed) {
        ++s.calls;
        for (int c = 0; c < 2; ++c) {
            if (!tc.ran[c]) continue;
            check_hip(hipEventSynchronize(tc.t1[c]), "hipEventSynchronize");
            float ms = 0.f;
            check_hip(hipEventElapsedTime(&ms, tc.t0[c], tc.t1[c]), "hipEventElapsedTime");
            float &mn = c == 0 ? s.host_ms_min : s.staging_ms_min;
            float &mx = c == 0 ? s.host_ms_max : s.staging_ms_max;
            (c == 0 ? s.host_ms_sum : s.staging_ms_sum) += ms;
            (c == 0 ? s.host_calls : s.staging_calls) += 1;
            mn = mn < 0.f ? ms : std::min(mn, ms);
            mx = std::max(mx, ms);
        }
    }
    for (auto &tc : p.timed)
        for (int c = 0; c < 2; ++c) {
            if (tc.t0[c]) p.spare.push_back(tc.t0[c]);
            if (tc.t1[c]) p.spare.push_back(tc.t1[c]);
        }
    p.timed.clear();
    if (sum) *sum = s;
}

// noalloc (retrieve only): a work list too large for the kernel arguments goes
// through the device's static scratch instead of the upload ring, and the host
// class always takes the zero-copy kernel (the copy-engine ring is memory of
// its own); no timing, so that the call makes no allocation and creates no HIP
// object.
void pool_transfer(Pool &p, const kvp_loc *map, uint32_t n_blocks, const int32_t *table, uint32_t num_slots,
                   uint32_t layer_begin, uint32_t layer_end, void *const *k_layers, void *const *v_layers,
                   void *stream_ptr, bool gather, bool noalloc)
{
    if (p.placement_only) fail(KVP_ERR_INVALID, "placement-only pool has no memory to copy");
    if (n_blocks && (!map || !table)) fail(KVP_ERR_INVALID, "null map or block table");
    const uint32_t L = p.spec.num_layers;
    if (layer_begin >= layer_end || layer_end > L)
        fail(KVP_ERR_INVALID, "layer range [" + std::to_string(layer_begin) + ", " + std::to_string(layer_end) +
                                  ") not inside [0, " + std::to_string(L) + ")");
    if (!k_layers || !v_layers) fail(KVP_ERR_INVALID, "null layer pointer array");
    for (uint32_t l = layer_begin; l < layer_end; ++l) {
        const uintptr_t k = reinterpret_cast<uintptr_t>(k_layers[l]), v = reinterpret_cast<uintptr_t>(v_layers[l]);
        if (!k || !v || (k & 15) || (v & 15))
            fail(KVP_ERR_INVALID, "layer " + std::to_string(l) + ": null or unaligned cache pointer");
    }
    // A link kernel's units (blocks x 2L chunks x at most 2 parts) and its workgroup stride (at most 2^20)
    // are summed in 32 bits: at most 2^31 units keeps that sum from wrapping.  The HBM body's units are
    // smaller; its launch makes them larger where there would be over 2^31, beside a stride of at most 2^23.
    if (static_cast<uint64_t>(n_blocks) * 4 * L > (1ull << 31)) fail(KVP_ERR_INVALID, "request too large");

    std::lock_guard<std::mutex> lock(p.mu);
    DeviceScope dev(p.device);
    const uint32_t op = gather ? KVP_OP_RETRIEVE : KVP_OP_STORE;
    if (noalloc && !gather) fail(KVP_ERR_INVALID, "the static-scratch path is a retrieve");
    const bool sdma = !noalloc && (p.launch[KVP_CLASS_HOST][op].flags & KVP_LAUNCH_SDMA) != 0;
    if (sdma && !p.bounce)   // only after a kv_pool_set_copy_ring that could not allocate
        fail(KVP_ERR_NOMEM, "copy-engine ring not allocated: set a smaller ring or clear KVP_LAUNCH_SDMA");

    // GLT-resolved locations, grouped by region class (Sec. 4.3), in buffers that
    // the pool keeps from call to call
    Plan &plan = p.plan;
    plan.reset(p.regions.size());
    std::vector<CopyItem>(&items)[2] = plan.items;
    std::vector<HostBlock> host_blocks;   // copy-engine transport: placed in ring slots below
    std::vector<HostBlock> file_blocks;   // file regions: placed in the file ring's slots below
    std::vector<RequestRec *> &touched = plan.touched;
    const uint64_t epoch = ++p.call_epoch;
    // No two present entries may write the same place: a destination slot on
    // retrieve, a pool block on store.  One pass over bitmaps -- of the
    // destination slots, or of the blocks of each allocation a store touches
    // (the block index within its allocation is exact after resolve) -- with
    // sorted slots only for a retrieve into far more slots than it moves.
    std::vector<uint64_t> &seen = plan.seen;
    const bool slot_bits = gather && num_slots <= std::max<uint64_t>(64ull * n_blocks, 1ull << 16);
    if (slot_bits) seen.assign((num_slots + 63) / 64, 0);
    std::vector<uint32_t> &wide_slots = plan.wide_slots;
    std::unordered_map<const Allocation *, uint64_t> alloc_word;   // store: first bitmap word of an allocation
    bool dup = false;
    uint64_t dup_slot = 0;
    auto mark = [&](uint64_t bit) {
        uint64_t &w = seen[bit >> 6];
        const uint64_t m = 1ull << (bit & 63);
        if ((w & m) && !dup) {
            dup = true;
            dup_slot = bit;
        }
        w |= m;
    };
    for (uint32_t b = 0; b < n_blocks; ++b) {
        const kvp_loc &e = map[b];
        if (e.region == KVP_ABSENT) continue;
        // One place per region: a request's blocks in a region share one range,
        // while consecutive blocks of a striped map alternate between regions.
        // An entry that follows the last one in its range needs no further look.
        RegionPlace *at = e.region < plan.places.size() ? &plan.places[e.region] : nullptr;
        if (at && at->alloc && e.offset == at->next && e.offset < at->end && e.gen == at->alloc->gen) {
            at->next += p.block_bytes;
            ++at->index;
        } else {
            const Allocation *a = resolve(p, e, b, at ? at->alloc : nullptr);   // throws for a bad region
            const bool other = a != at->alloc;
            at->alloc = a;
            at->index = (e.offset - a->base) / p.block_bytes;
            at->next = e.offset + p.block_bytes;
            at->end = a->base + a->blocks * p.block_bytes;
            if (other && !gather) {
                auto it = alloc_word.find(a);
                if (it == alloc_word.end()) {
                    it = alloc_word.emplace(a, seen.size()).first;
                    seen.resize(seen.size() + (a->blocks + 63) / 64, 0);
                }
                at->word = it->second;
            }
            if (other && a->owner->call_mark != epoch) {   // each request listed once
                a->owner->call_mark = epoch;
                touched.push_back(a->owner);
            }
        }
        const int32_t slot = table[b];
        if (slot < 0 || static_cast<uint32_t>(slot) >= num_slots)
            fail(KVP_ERR_INVALID, "block table entry " + std::to_string(b) + " = " + std::to_string(slot) +
                                      " outside [0, " + std::to_string(num_slots) + ")");
        if (slot_bits)
            mark(static_cast<uint64_t>(slot));
        else if (gather)
            wide_slots.push_back(static_cast<uint32_t>(slot));
        else
            mark(at->word * 64 + at->index);
        const Region &r = p.regions[e.region];
        if (r.desc.type == KVP_REGION_FILE) {
            if (noalloc)
                fail(KVP_ERR_INVALID, "map entry " + std::to_string(b) + ": the allocation-free call reads no file region");
            file_blocks.push_back(HostBlock{e.region, e.offset, static_cast<uint32_t>(slot)});
        } else {
            const uint32_t cls = r.desc.type == KVP_REGION_HOST ? KVP_CLASS_HOST : KVP_CLASS_STAGING;
            if (cls == KVP_CLASS_HOST && sdma)
                host_blocks.push_back(HostBlock{e.region, e.offset, static_cast<uint32_t>(slot)});
            else
                items[cls].push_back(
                    CopyItem{reinterpret_cast<uint64_t>(r.dev) + e.offset, static_cast<uint32_t>(slot), e.region});
        }
    }
    if (!wide_slots.empty()) {
        std::sort(wide_slots.begin(), wide_slots.end());
        auto d = std::adjacent_find(wide_slots.begin(), wide_slots.end());
        if (d != wide_slots.end()) {
            dup = true;
            dup_slot = *d;
        }
    }
    if (dup)
        fail(KVP_ERR_INVALID, gather ? "destination slot " + std::to_string(dup_slot) + " named twice"
                                     : std::string("two map entries name the same pool block"));
    order_items(items[KVP_CLASS_STAGING], plan.other, gather, gather ? num_slots : static_cast<uint32_t>(p.regions.size()));
    const uint64_t width = 2ull * (layer_end - layer_begin) * p.chunk_bytes;   // bytes moved per block
    const uint64_t skip = 2ull * layer_begin * p.chunk_bytes;
    std::vector<LinkRun> runs;
    std::vector<Batch> batches;
    if (!host_blocks.empty()) {
        const RingGeometry g{reinterpret_cast<uint64_t>(p.bounce), p.bounce_slot_bytes, kBounceSlots, p.bounce_next,
                             p.block_bytes, p.chunk_bytes};
        plan_bounce(g, host_blocks, width, 2 * layer_begin, items[KVP_CLASS_HOST], runs, batches);
    }

    std::vector<CopyItem> file_items;
    std::vector<FileSpan> spans;
    std::vector<FileBatch> file_batches;
    if (!file_blocks.empty()) {
        if (!p.file_ring || p.file_slot_bytes < p.block_bytes)   // only after a kv_pool_set_file_ring that could not allocate
            fail(KVP_ERR_NOMEM, "file-region ring not allocated: set a smaller one with kv_pool_set_file_ring");
        const FileGeometry fg{p.file_ring_dev, p.file_slot_bytes, kFileSlots, p.file_next, p.block_bytes,
                              p.chunk_bytes};
        plan_file(fg, file_blocks, skip, width, 2 * layer_begin, file_items, spans, file_batches);
    }

    const size_t n_items = items[0].size() + items[1].size() + file_items.size();
    const size_t ptr_bytes = round_up(static_cast<size_t>(2 * (layer_end - layer_begin)) * sizeof(uint64_t), 16);
    const size_t list_bytes = ptr_bytes + n_items * sizeof(CopyItem);
    if (noalloc && list_bytes > kScratchBytes)
        fail(KVP_ERR_INVALID, "work list of " + std::to_string(list_bytes) + " bytes (" + std::to_string(n_items) +
                                  " blocks) exceeds the static scratch of " + std::to_string(kScratchBytes) + " bytes");
    if (p.timing && !noalloc) {
        if (p.timed.size() >= kMaxTimedCalls) drain_timed(p, nullptr);   // bound the history
        TimedCall tc;
        for (int c = 0; c < 2; ++c) {
            tc.blocks[c] = static_cast<uint32_t>(items[c].size());
            if (!items[c].empty()) {
                tc.t0[c] = timing_event(p);
                tc.t1[c] = timing_event(p);
            }
        }
        p.timed.push_back(tc);
    }
    if (n_items == 0) return;

    hipStream_t s = static_cast<hipStream_t>(stream_ptr);
    // A call may be captured into a graph if its work list travels in kernel
    // arguments (a small call, and any allocation-free one); its replays are the
    // caller's to order, so nothing is recorded for it.
    const bool capturing = stream_capturing(s);
    if (!capturing) land_done_calls(p);
    uint64_t waited = 0;
    // The stream of an earlier call may be this one, but its handle does not tell:
    // hipStreamPerThread names another stream in every thread, and the handle of a
    // destroyed stream is given out again.  The runtime knows the streams and drops
    // a wait for work of the same one.  Under capture it refuses every wait for
    // work outside of the graph, so there a handle that names one stream counts.
    auto wait_for = [&](uint64_t call) {
        const FlightRec *f = call == waited ? nullptr : in_flight(p, call);
        waited = call;
        if (f && !(capturing && f->stream == s && s != hipStreamPerThread))
            check_hip(hipStreamWaitEvent(s, f->done, 0), "hipStreamWaitEvent");
    };
    // ordering with earlier work on the same requests from any stream:
    // retrieve after store (read after write), store after store/retrieve
    for (RequestRec *rec : touched) wait_for(gather ? rec->stored_call : rec->busy_call);
    // one host-class kernel on the link at a time, in enqueue order: two of
    // them would only share its bandwidth and both end late
    auto take_link = [&] { wait_for(p.link_call[op]); };
    Slot *slot = nullptr;        // the call's work-list buffer, once it is in use
    hipEvent_t lent = nullptr;   // the allocation-free call's event
    uint64_t link_part = 0;      // record of the host-class kernel alone, once it is recorded
    auto touch = [&](bool on_link) {   // the call is last_call()
        const uint64_t call = last_call(p);
        if (slot) slot->call = call;
        if (on_link) p.link_call[op] = link_part ? link_part : call;
        for (RequestRec *rec : touched) {
            rec->busy_call = call;
            if (!gather) rec->stored_call = call;
        }
    };
    // The call's completion.  busy must cover every call still touching the
    // request, not only this one: two retrieves of a request may run on
    // different streams at once, and release, destroy and a later store wait on
    // busy alone.  So the caller's stream first waits for the previous one (after
    // this call's kernels, so only later work on the stream is held back), and
    // the new one covers both.  Its record in flight is made before the first
    // launch, so that only the runtime can fail once something is enqueued.
    struct Opened {
        Pool &p;
        hipEvent_t done = nullptr, link_done = nullptr;
        uint32_t records = 0;   // to be taken back
        ~Opened()
        {
            for (; records; --records) cancel_call(p);
        }
    } opened{p};
    auto begin = [&](bool with_link_part = false) {
        if (capturing) return;
        if (with_link_part) opened.link_done = begin_call(p, s, nullptr, nullptr, !noalloc);
        opened.records += opened.link_done != nullptr;
        opened.done = begin_call(p, s, lent, touched.front()->event, !noalloc);
        ++opened.records;
    };
    auto link_part_done = [&] {   // the host-class kernel is enqueued, other parts of the call may outlast it
        if (!opened.link_done) return;
        check_hip(hipEventRecord(opened.link_done, s), "hipEventRecord");
        link_part = last_call(p) - 1;
    };
    auto finish = [&](bool on_link) {   // everything is enqueued: record it
        if (capturing) return;
        try {
            for (RequestRec *rec : touched) wait_for(rec->busy_call);
            check_hip(hipEventRecord(opened.done, s), "hipEventRecord");
        } catch (...) {   // nothing will tell when the call is done, so it is done before this returns
            (void)hipStreamSynchronize(s);
            throw;
        }
        opened.records = 0;
        touch(on_link);
    };
    const uint32_t chunks = 2 * (layer_end - layer_begin);
    CopyArgs geo = {};
    geo.chunks = chunks;
    geo.chunk0 = 2 * layer_begin;
    geo.parts = 1;
    geo.chunk_bytes = p.chunk_bytes;
    geo.heads = p.spec.num_kv_heads;
    geo.tokens = p.spec.block_size;
    geo.row_vec = static_cast<uint32_t>(static_cast<uint64_t>(p.spec.head_dim) * p.spec.elem_bytes / 16);
    geo.layout = p.spec.pool_layout;
    auto fill_table = [&](uint64_t *t) {   // engine buffer of moved chunk k
        for (uint32_t k = 0; k < chunks; ++k) {
            const uint32_t l = layer_begin + k / 2;
            t[k] = reinterpret_cast<uint64_t>(k % 2 ? v_layers[l] : k_layers[l]);
        }
    };

    const LaunchCfg &ls = p.launch[KVP_CLASS_STAGING][op];
    LaunchCfg lh = p.launch[KVP_CLASS_HOST][op];
    const bool host = !items[KVP_CLASS_HOST].empty();
    // One launch for both classes, unless each is timed, the host class's LDS
    // would hold the HBM kernel's workgroups back (their wavefronts fill a CU
    // with 8 workgroups), the flags ask for what the one launch does not have, or
    // the link has to be waited for or handed on while the HBM kernel runs.  In
    // two launches the internal stream takes the staging class, for enough of its
    // bytes.
    const bool lds = p.spec.pool_layout == 1 && (lh.flags & KVP_LAUNCH_LDS) != 0;
    const bool both = host && !items[KVP_CLASS_STAGING].empty();
    const uint32_t staging_hints = KVP_LAUNCH_NT_STORE | (p.spec.pool_layout == 0 ? KVP_LAUNCH_NT_LOAD : 0u);
    const bool own_forms = (lh.flags & (KVP_LAUNCH_XCD | KVP_LAUNCH_CHUNK_MAJOR | KVP_LAUNCH_TILE)) != 0 ||
                           (ls.flags & staging_hints) != staging_hints;
    const uint64_t staging_bytes = items[KVP_CLASS_STAGING].size() * width;
    const uint64_t link_bytes = kHbmPerLink * items[KVP_CLASS_HOST].size() * width;   // as HBM bytes of the same time
    const bool large = batches.empty() && staging_bytes >= kForkMinBytes;
    // The one launch ends with its longer class.  If that is the host class, the
    // end hands the link on in time.  If HBM takes more than twice as long, the
    // call does not hold the link at all: whoever shares it has it back before
    // this call ends, and sooner than by waiting for the end.  In between, the host
    // class has a kernel and a record of its own.
    const bool outlasts = both && large && staging_bytes > link_bytes;
    const bool shares_link = outlasts && staging_bytes > 2 * link_bytes;
    auto link_taken = [&] {   // by an unfinished call of another stream
        const FlightRec *f = in_flight(p, p.link_call[op]);
        return f && f->stream != s && hipPeekAtLastError() == hipSuccess && !event_done(f->done);
    };
    const bool one_launch = batches.empty() && (noalloc || !p.timing) &&
                            !(both && lds && p.chunk_bytes > kMergeLdsMax) && !(both && own_forms) &&
                            !(outlasts && !shares_link) && !(both && large && !capturing && link_taken());
    const bool fork_staging = large && host && !one_launch;
    const bool holds_link = host && batches.empty() && !(one_launch && shares_link);
    const FlightRec *storing = in_flight(p, p.link_call[KVP_OP_STORE]);
    // a store's host-class kernel not yet finished: the link carries traffic both ways
    if (gather && host && lh.default_grid && storing && lh.grid < kDuplexReadGrid && !capturing &&
        hipPeekAtLastError() == hipSuccess &&   // never clear an error the caller has yet to read
        !event_done(storing->done))
        lh.grid = kDuplexReadGrid;
    if (!gather && host && large && lh.default_grid)
        lh.grid = throttled_store_grid(lh.grid, items[KVP_CLASS_HOST].size() * width,
                                       items[KVP_CLASS_STAGING].size() * width);
    if (batches.empty() && file_batches.empty() && (noalloc || !p.timing) &&
        !((lh.flags | ls.flags) & KVP_LAUNCH_UPLOAD) &&
        chunks + 2 * n_items <= kInlineWords) {
        // Small call: table and items in the kernel arguments
        CallArgs f = {};
        f.a = geo;
        f.a.n_items = static_cast<uint32_t>(n_items);
        f.n_host = static_cast<uint32_t>(items[KVP_CLASS_HOST].size());
        fill_table(f.words);
        auto *list = reinterpret_cast<CopyItem *>(f.words + chunks);
        std::copy(items[0].begin(), items[0].end(), list);
        std::copy(items[1].begin(), items[1].end(), list + items[0].size());
        if (host) take_link();
        begin();
        check_hip(launch_call(f, gather, lh.grid, ls.grid, lh.flags, ls.flags, s), "kernel launch");
        finish(host);
        return;
    }

    if (capturing && noalloc) {
        // A replay may run after any number of other calls that used the scratch,
        // so a captured call's list goes where none of them writes: into the graph.
        std::vector<uint64_t> table(chunks);
        fill_table(table.data());
        if (host) take_link();
        launch_in_parts(geo, items, table, gather, lh, ls, s);
        return;
    }

    // work list: [chunks cache pointers][host items][staging items][file items], in a
    // ring slot of the pool, or in the device's static scratch (noalloc)
    const size_t bytes = list_bytes;
    if (capturing)   // a replay would read a buffer that later calls rewrite
        fail(KVP_ERR_HIP, "a call with an uploaded work list: operation not permitted when stream is capturing");
    ScratchDevice *sd = nullptr;
    const bool whole = bytes > kScratchBytes / 2;   // of the scratch
    uint32_t half = 0;
    std::unique_lock<std::mutex> scratch_lock;
    Slot *buffer = nullptr;
    void *host_list = nullptr, *host_list_dev = nullptr, *dev_base = nullptr;
    if (noalloc) {
        sd = &scratch_device(p.device);   // set up when the pool was created
        scratch_lock = std::unique_lock<std::mutex>(sd->mu);
        // a half is rewritten, in either memory, only after the kernels of the
        // last call that used it (from any pool, on any stream)
        half = whole ? 0 : sd->next;
        for (uint32_t h = 0; h < 2; ++h) {
            const hipEvent_t user = whole || h == half ? sd->user[h] : nullptr;
            if (!user) continue;
            check_hip(hipEventSynchronize(user), "hipEventSynchronize");
            for (hipEvent_t &u : sd->user)
                if (u == user) u = nullptr;
        }
        lent = p.scratch_done[half];   // this pool's earlier calls in this half were over before that one
        forget_event(p, lent);
        host_list = static_cast<char *>(sd->host) + half * (kScratchBytes / 2);
        host_list_dev = static_cast<char *>(sd->host_dev) + half * (kScratchBytes / 2);
        dev_base = static_cast<char *>(sd->dev) + half * (kScratchBytes / 2);
    } else {
        buffer = &acquire_slot(p, bytes);
        host_list = buffer->host;
        host_list_dev = buffer->host_dev;
        dev_base = buffer->dev;
    }
    fill_table(static_cast<uint64_t *>(host_list));
    auto *list = reinterpret_cast<CopyItem *>(static_cast<char *>(host_list) + ptr_bytes);
    std::copy(items[0].begin(), items[0].end(), list);
    std::copy(items[1].begin(), items[1].end(), list + items[0].size());
    std::copy(file_items.begin(), file_items.end(), list + items[0].size() + items[1].size());

    begin(holds_link && (fork_staging || !file_batches.empty()));
    check_hip(launch_list_copy(dev_base, host_list_dev, bytes, s), "kernel launch");
    slot = buffer;   // from here on the buffer is in use even if a launch fails
    auto took_scratch = [&] {   // after finish
        if (!noalloc) return;
        sd->user[half] = lent;
        if (whole) sd->user[1] = lent;
        sd->next = half ^ 1u;
    };
    // After a failure once the work list is on its way (a file read or write
    // that fails, a launch or copy the runtime refuses), whatever was enqueued
    // still runs and reads the work list.  So the caller's stream joins the
    // pool's stream, and the call's completion is recorded after all of it
    // before the error is returned: a later call cannot rewrite the list under
    // those kernels, and release waits for them.  Nothing here throws, so the
    // first error is the one reported.
    auto settle = [&]() noexcept {
        (void)hipEventRecord(p.stage_done, p.s_stage);
        (void)hipStreamWaitEvent(s, p.stage_done, 0);
        try {
            finish(holds_link);
            took_scratch();
        } catch (...) {   // the call is done: finish saw to it
        }
        clear_hip_error();
    };
    auto enqueue = [&] {
        if (fork_staging || !batches.empty() || !file_batches.empty())
            check_hip(hipEventRecord(p.fork, s), "hipEventRecord");

        const CopyItem *dev_list = reinterpret_cast<const CopyItem *>(static_cast<char *>(dev_base) + ptr_bytes);
        // Two launches: the staging class forked onto the internal stream first,
        // then the host class on the caller's stream itself; the caller's stream
        // then waits for the staging kernel.  One extra stream keeps the pool
        // within the few hardware queues a process gets, so caller streams (e.g.
        // compute overlapping a layerwise retrieve) are not serialised behind it.
        size_t first = 0;
        CopyArgs args[2] = {geo, geo};
        for (uint32_t c = 0; c < 2; ++c) {
            args[c].items = dev_list + first;
            args[c].cache = static_cast<const uint64_t *>(dev_base);
            args[c].n_items = static_cast<uint32_t>(items[c].size());
            first += items[c].size();
        }
        TimedCall *tc = p.timing && !noalloc ? &p.timed.back() : nullptr;
        auto launch = [&](uint32_t c, hipStream_t st) {
            const LaunchCfg &lc = c == KVP_CLASS_HOST ? lh : p.launch[c][op];
            if (tc) check_hip(hipEventRecord(tc->t0[c], st), "hipEventRecord");
            check_hip(launch_chunk_copy(args[c], c, gather, lc.grid, lc.flags, st), "kernel launch");
            if (tc) {
                check_hip(hipEventRecord(tc->t1[c], st), "hipEventRecord");
                tc->ran[c] = true;
            }
        };
        const bool staging = !items[KVP_CLASS_STAGING].empty();
        if (one_launch) {
            CallArgs f = {};
            f.a = args[KVP_CLASS_HOST];
            f.a.n_items += args[KVP_CLASS_STAGING].n_items;
            f.n_host = args[KVP_CLASS_HOST].n_items;
            if (host) take_link();
            const uint32_t c = host ? KVP_CLASS_HOST : KVP_CLASS_STAGING;
            const LaunchCfg &lc = host ? lh : ls;
            check_hip(both ? launch_call(f, gather, lh.grid, ls.grid, lh.flags, ls.flags, s)
                           : launch_chunk_copy(args[c], c, gather, lc.grid, lc.flags, s),
                      "kernel launch");
            link_part_done();
        } else if (batches.empty()) {
            if (fork_staging) {
                check_hip(hipStreamWaitEvent(p.s_stage, p.fork, 0), "hipStreamWaitEvent");
                launch(KVP_CLASS_STAGING, p.s_stage);
                check_hip(hipEventRecord(p.stage_done, p.s_stage), "hipEventRecord");
            } else if (staging) {
                launch(KVP_CLASS_STAGING, s);   // small: in order on the caller's stream
            }
            if (host) {
                take_link();
                launch(KVP_CLASS_HOST, s);
                link_part_done();
            }
            if (fork_staging) check_hip(hipStreamWaitEvent(s, p.stage_done, 0), "hipStreamWaitEvent");
        } else {
            // Copy-engine transport: the host-link copies take the internal
            // stream (no stream beyond the kernel path's two) and every kernel
            // runs on the caller's stream -- the staging class first, then one
            // ring-slot kernel per batch.  A slot is refilled only after its
            // previous contents were consumed (by any call, either op).
            if (staging) launch(KVP_CLASS_STAGING, s);
            const LaunchCfg &lc = p.launch[KVP_CLASS_STAGING][op];
            const hipMemcpyKind kind = gather ? hipMemcpyHostToDevice : hipMemcpyDeviceToHost;
            hipStream_t sc = p.s_stage;
            auto link_copies = [&](const Batch &bt) {
                char *ring = p.bounce + static_cast<uint64_t>(bt.ring) * p.bounce_slot_bytes;
                for (size_t i = bt.run0; i < bt.run0 + bt.runs; ++i) {
                    const LinkRun &run = runs[i];
                    char *hmem = static_cast<char *>(p.regions[run.region].host) + run.offset + skip;
                    char *dev = ring + run.slot_offset;
                    void *dst = gather ? static_cast<void *>(dev) : static_cast<void *>(hmem);
                    const void *src = gather ? static_cast<const void *>(hmem) : static_cast<const void *>(dev);
                    if (width == p.block_bytes)
                        check_hip(hipMemcpyAsync(dst, src, run.blocks * width, kind, sc), "hipMemcpyAsync");
                    else
                        check_hip(hipMemcpy2DAsync(dst, gather ? width : p.block_bytes, src, gather ? p.block_bytes : width,
                                                   width, run.blocks, kind, sc),
                                  "hipMemcpy2DAsync");
                }
            };
            auto ring_kernel = [&](const Batch &bt) {
                CopyArgs a = args[KVP_CLASS_HOST];
                a.items = dev_list + bt.first;
                a.n_items = bt.n;
                check_hip(launch_chunk_copy(a, kClassRing, gather, lc.grid, lc.flags, s), "kernel launch");
            };
            if (gather) {
                check_hip(hipStreamWaitEvent(sc, p.fork, 0), "hipStreamWaitEvent");
                if (tc) check_hip(hipEventRecord(tc->t0[KVP_CLASS_HOST], sc), "hipEventRecord");
                for (const Batch &bt : batches) {
                    if (p.bounce_free_rec[bt.ring])
                        check_hip(hipStreamWaitEvent(sc, p.bounce_free[bt.ring], 0), "hipStreamWaitEvent");
                    link_copies(bt);
                    check_hip(hipEventRecord(p.bounce_filled[bt.ring], sc), "hipEventRecord");
                    check_hip(hipStreamWaitEvent(s, p.bounce_filled[bt.ring], 0), "hipStreamWaitEvent");
                    ring_kernel(bt);
                    check_hip(hipEventRecord(p.bounce_free[bt.ring], s), "hipEventRecord");
                    p.bounce_free_rec[bt.ring] = true;
                }
            } else {
                if (tc) check_hip(hipEventRecord(tc->t0[KVP_CLASS_HOST], s), "hipEventRecord");
                for (const Batch &bt : batches) {
                    if (p.bounce_free_rec[bt.ring])
                        check_hip(hipStreamWaitEvent(s, p.bounce_free[bt.ring], 0), "hipStreamWaitEvent");
                    ring_kernel(bt);
                    check_hip(hipEventRecord(p.bounce_filled[bt.ring], s), "hipEventRecord");
                    check_hip(hipStreamWaitEvent(sc, p.bounce_filled[bt.ring], 0), "hipStreamWaitEvent");
                    link_copies(bt);
                    check_hip(hipEventRecord(p.bounce_free[bt.ring], sc), "hipEventRecord");
                    p.bounce_free_rec[bt.ring] = true;
                }
                check_hip(hipEventRecord(p.stage_done, sc), "hipEventRecord");
                check_hip(hipStreamWaitEvent(s, p.stage_done, 0), "hipStreamWaitEvent");
            }
            p.bounce_next = static_cast<uint32_t>((p.bounce_next + batches.size()) % kBounceSlots);
            if (tc) {
                check_hip(hipEventRecord(tc->t1[KVP_CLASS_HOST], s), "hipEventRecord");
                tc->ran[KVP_CLASS_HOST] = true;
            }
        }
        if (!file_batches.empty()) {
            // file-region kernels on the pool's stream, beside the host-class
            // kernel on the caller's, then joined back into the caller's stream
            if (!fork_staging && batches.empty()) check_hip(hipStreamWaitEvent(p.s_stage, p.fork, 0), "hipStreamWaitEvent");
            CopyArgs fa = geo;
            fa.items = dev_list + items[0].size() + items[1].size();
            fa.cache = static_cast<const uint64_t *>(dev_base);
            LaunchCfg lf = p.launch[KVP_CLASS_HOST][op];
            lf.flags &= ~(KVP_LAUNCH_SDMA | KVP_LAUNCH_UPLOAD);
            run_file_batches(p, gather, file_batches, spans, fa, lf, p.s_stage);
            check_hip(hipEventRecord(p.stage_done, p.s_stage), "hipEventRecord");
            check_hip(hipStreamWaitEvent(s, p.stage_done, 0), "hipStreamWaitEvent");
        }
    };
    try {
        enqueue();
    } catch (...) {
        settle();
        throw;
    }
    finish(holds_link);
    took_scratch();
}

}  // namespace kvp
