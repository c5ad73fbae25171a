// Data-movement kernels of the KV pool, for gfx950 (MI355X).
//
// Nothing here is a contraction, so there is no MFMA: every kernel is a bit
// copy of 16-byte vectors between pool blocks and the engine cache.  There are
// two bodies, since the host link and HBM want opposite shapes.
//
// Link body (host regions, file-ring slots): the link needs only its
// bandwidth-delay product in flight, so a dozen persistent 256-thread
// workgroups (four 64-lane wavefronts) stream whole units.  One unit is one
// (block, layer, K/V) chunk of C bytes, or half of one (KVP_LAUNCH_SPLIT2,
// plain chunks only); each lane holds up to UNROLL 16-byte loads in flight
// before it stores, so a workgroup keeps 256*UNROLL*16 bytes in flight (32 KiB
// at UNROLL = 8, one LLaMA-shaped chunk).  Workgroup g takes units g, g+G,
// g+2G, ...  With K moved chunks per block (2L for all layers, fewer for a
// layer range), unit u is part u % parts of moved chunk (u / parts) % K of
// work item u / (K*parts), so neighbouring workgroups read neighbouring pieces
// of the same pool block.  The next unit's entries are fetched while the
// current unit is copied.  Three copy forms:
//   - head-major pool chunks: the chunk is [H][bs][D] on both sides; a plain
//     contiguous copy (this moves the layer axis from inside the block to
//     the per-layer engine buffers).
//   - token-major pool chunks, direct: every 16-byte vector of a [bs][H][D]
//     chunk maps to one vector of the [H][bs][D] chunk; both sides move in
//     runs of D*elem_bytes bytes.
//   - token-major pool chunks, LDS-staged: the chunk is read contiguously
//     into LDS, then written contiguously in the other order, so both global
//     sides are fully contiguous per workgroup.
//
// HBM body (staging regions, copy-engine ring slots): see wave_copy_body.
//
// The work list and the engine pointer table are read with scalar loads.
//
// Five entry points share the bodies, so that traces and counters tell them
// apart: host_region_copy (zero-copy reads or writes of pinned host regions
// over the host link), staging_region_copy (HBM staging regions),
// ring_slot_copy (a copy-engine ring slot in HBM, whose host-link leg is a
// hipMemcpy), file_slot_copy (a file regions' ring slot in pinned host
// memory, filled or emptied by file reads and writes), and both_regions_copy
// (both region classes of a call in one launch).

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "internal.hpp"

namespace kvp {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));
// Every buffer the kernels touch is global memory (HBM or mapped host
// memory); saying so lets the compiler emit global_* instead of flat_*
// accesses, which do not occupy the LDS counter.
typedef __attribute__((address_space(1))) v4u gv4u;

constexpr uint32_t kThreads = 256;
constexpr uint32_t kWave = 64;
constexpr uint32_t kWaves = kThreads / kWave;
constexpr uint32_t kXcds = 8;     // MI355X: 8 accelerator complex dies, 32 CUs each
constexpr uint64_t kMaxLdsChunk = 64 * 1024;
constexpr uint32_t kTileItems = 8;  // KVP_LAUNCH_TILE: work items per workgroup-owned tile

template <bool NT>
__device__ __forceinline__ v4u load16(const v4u *p)
{
    const gv4u *g = (const gv4u *)p;
    if constexpr (NT)
        return __builtin_nontemporal_load(g);
    else
        return *g;
}

template <bool NT>
__device__ __forceinline__ void store16(v4u *p, v4u v)
{
    gv4u *g = (gv4u *)p;
    if constexpr (NT)
        __builtin_nontemporal_store(v, g);
    else
        *g = v;
}

// Loads of a batch must not sit under per-lane branches: the compiler then
// waits for each load before issuing the next, leaving one 16-byte load in
// flight per lane.  Out-of-range lanes therefore load a clamped (valid)
// index and only their stores are predicated.
__device__ __forceinline__ uint32_t clamp_index(uint32_t v, uint32_t nvec) { return v < nvec ? v : nvec - 1; }

// Workgroup-cooperative contiguous copy of nvec 16-byte vectors.
template <int UNROLL, bool NTL, bool NTS>
__device__ __forceinline__ void wg_copy(const v4u *__restrict__ src, v4u *__restrict__ dst, uint32_t nvec)
{
    const uint32_t tid = threadIdx.x;
    uint32_t base = 0;
    for (; base + kThreads * UNROLL <= nvec; base += kThreads * UNROLL) {
        v4u r[UNROLL];
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) r[i] = load16<NTL>(src + base + i * kThreads + tid);
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) store16<NTS>(dst + base + i * kThreads + tid, r[i]);
    }
    if (base < nvec) {  // ragged tail: one batch, clamped loads, predicated stores
        v4u r[UNROLL];
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) r[i] = load16<NTL>(src + clamp_index(base + i * kThreads + tid, nvec));
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
            const uint32_t v = base + i * kThreads + tid;
            if (v < nvec) store16<NTS>(dst + v, r[i]);
        }
    }
}

// Index maps between the two chunk orders, in 16-byte vectors; rv vectors
// make one head_dim row.  Head-major [H][bs][rv] index v <-> token-major
// [bs][H][rv] index.
__device__ __forceinline__ uint32_t hm_to_tm(uint32_t v, uint32_t heads, uint32_t tokens, uint32_t rv)
{
    const uint32_t row = v / rv, w = v - row * rv;
    const uint32_t h = row / tokens, t = row - h * tokens;
    return (t * heads + h) * rv + w;
}

__device__ __forceinline__ uint32_t tm_to_hm(uint32_t v, uint32_t heads, uint32_t tokens, uint32_t rv)
{
    const uint32_t row = v / rv, w = v - row * rv;
    const uint32_t t = row / heads, h = row - t * heads;
    return (h * tokens + t) * rv + w;
}

// Source index of destination vector v.  GATHER: destination head-major
// (cache), source token-major (pool); store: the reverse.
template <bool GATHER>
__device__ __forceinline__ uint32_t src_of(uint32_t v, uint32_t heads, uint32_t tokens, uint32_t rv)
{
    if constexpr (GATHER)
        return hm_to_tm(v, heads, tokens, rv);
    else
        return tm_to_hm(v, heads, tokens, rv);
}

// Direct token-major <-> head-major chunk conversion.  The lane index runs
// over the destination, so stores are contiguous; loads come in runs of rv
// vectors (one head_dim row).
template <bool GATHER, int UNROLL, bool NTL, bool NTS>
__device__ __forceinline__ void wg_convert(const v4u *__restrict__ src, v4u *__restrict__ dst, uint32_t nvec,
                                           uint32_t heads, uint32_t tokens, uint32_t rv)
{
    const uint32_t tid = threadIdx.x;
    for (uint32_t base = 0; base < nvec; base += kThreads * UNROLL) {
        v4u r[UNROLL];
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
            const uint32_t v = clamp_index(base + i * kThreads + tid, nvec);
            r[i] = load16<NTL>(src + src_of<GATHER>(v, heads, tokens, rv));
        }
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
            const uint32_t v = base + i * kThreads + tid;
            if (v < nvec) store16<NTS>(dst + v, r[i]);
        }
    }
}

// LDS-staged conversion: the chunk is read contiguously into LDS (UNROLL
// 16-byte loads in flight per lane, as in the plain copy), then written
// contiguously in the other order out of LDS.
template <bool GATHER, int UNROLL, bool NTL, bool NTS>
__device__ __forceinline__ void wg_convert_lds(const v4u *__restrict__ src, v4u *__restrict__ dst, uint32_t nvec,
                                               uint32_t heads, uint32_t tokens, uint32_t rv, v4u *lds)
{
    const uint32_t tid = threadIdx.x;
    for (uint32_t base = 0; base < nvec; base += kThreads * UNROLL) {
        v4u r[UNROLL];
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) r[i] = load16<NTL>(src + clamp_index(base + i * kThreads + tid, nvec));
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
            const uint32_t v = base + i * kThreads + tid;
            if (v < nvec) lds[v] = r[i];
        }
    }
    __syncthreads();
    for (uint32_t base = 0; base < nvec; base += kThreads * UNROLL) {
        v4u r[UNROLL];
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
            const uint32_t v = clamp_index(base + i * kThreads + tid, nvec);
            r[i] = lds[src_of<GATHER>(v, heads, tokens, rv)];
        }
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
            const uint32_t v = base + i * kThreads + tid;
            if (v < nvec) store16<NTS>(dst + v, r[i]);
        }
    }
    __syncthreads();  // LDS is reused by the next chunk
}

enum Form { kPlain = 0, kConvert = 1, kConvertLds = 2 };

// The work list and the engine pointer table are written by the host before
// the launch and only read here; reading them through the constant address
// space lets the compiler use scalar loads (uniform per workgroup) instead
// of vector loads, and the next unit's entries are fetched while the current
// chunk is copied.
typedef __attribute__((address_space(4))) const CopyItem citem_t;
typedef __attribute__((address_space(4))) const uint64_t cptr_t;

struct Unit {
    uint64_t pool;   // device address of the chunk in its region
    uint64_t cache;  // device address of the chunk in the engine cache
};

// Unit u of a launch: item u / (chunks * parts), then chunk, then part of
// the chunk (parts > 1 only for plain chunks); or, chunk-major, chunk
// u / (items * parts), then item, then part, so that the units in flight
// write neighbouring slots of one per-layer buffer.  table[k] is the engine
// buffer of moved chunk k; the pool block holds chunk chunk0 + k.
__device__ __forceinline__ Unit unit_at(const CopyArgs &a, citem_t *items, cptr_t *table, uint32_t u)
{
    uint32_t item, k, p;
    if (a.chunk_major) {
        const uint32_t per_chunk = a.n_items * a.parts;
        k = u / per_chunk;
        const uint32_t r = u - k * per_chunk;
        item = r / a.parts;
        p = r - item * a.parts;
    } else {
        const uint32_t per_item = a.chunks * a.parts;
        item = u / per_item;
        const uint32_t r = u - item * per_item;
        k = r / a.parts;
        p = r - k * a.parts;
    }
    const uint32_t c = a.chunk0 + k;
    const uint64_t part = static_cast<uint64_t>(p) * (a.chunk_bytes / a.parts);
    const uint64_t pool = items[item].pool;
    const uint64_t slot = items[item].slot;
    return Unit{pool + static_cast<uint64_t>(c) * a.chunk_bytes + part, table[k] + slot * a.chunk_bytes + part};
}

// Workgroup g of the G that share the launch's a.n_items items takes units
// g, g + G, g + 2G, ...
template <bool GATHER, int FORM, int UNROLL, bool NTL, bool NTS>
__device__ __forceinline__ void chunk_copy_body(const CopyArgs &a, citem_t *items, cptr_t *table, uint32_t g,
                                                uint32_t G)
{
    extern __shared__ v4u lds[];
    const uint32_t units = a.n_items * a.chunks * a.parts;
    const uint32_t nvec = static_cast<uint32_t>((a.chunk_bytes / a.parts) >> 4);
    uint32_t u = g;
    if (u >= units) return;
    Unit cur = unit_at(a, items, table, u);
    for (;;) {
        const uint32_t nu = u + G;
        const bool more = nu < units;
        const Unit next = more ? unit_at(a, items, table, nu) : cur;   // fetched while this chunk is copied
        const v4u *src = reinterpret_cast<const v4u *>(GATHER ? cur.pool : cur.cache);
        v4u *dst = reinterpret_cast<v4u *>(GATHER ? cur.cache : cur.pool);
        if constexpr (FORM == kPlain)
            wg_copy<UNROLL, NTL, NTS>(src, dst, nvec);
        else if constexpr (FORM == kConvert)
            wg_convert<GATHER, UNROLL, NTL, NTS>(src, dst, nvec, a.heads, a.tokens, a.row_vec);
        else
            wg_convert_lds<GATHER, UNROLL, NTL, NTS>(src, dst, nvec, a.heads, a.tokens, a.row_vec, lds);
        if (!more) break;
        u = nu;
        cur = next;
    }
}

// Workgroup-owned tiles (KVP_LAUNCH_TILE): tile t is moved chunk t % K of
// the a.tile_items consecutive work items from (t / K) * a.tile_items on;
// workgroup g takes tiles g, g+G, ... and copies each itself, item by item
// (the parts of a chunk in turn).  Its writes then run over neighbouring
// slots of one per-layer engine buffer, and its reads over the same chunk
// of neighbouring pool blocks.
template <bool GATHER, int FORM, int UNROLL, bool NTL, bool NTS>
__device__ __forceinline__ void chunk_copy_tiles(const CopyArgs &a, citem_t *items, cptr_t *table, uint32_t g,
                                                 uint32_t G)
{
    extern __shared__ v4u lds[];
    const uint32_t K = a.chunks, TB = kTileItems;   // a.tile_items is kTileItems when set
    const uint32_t tiles = (a.n_items + TB - 1) / TB * K;
    const uint64_t part_bytes = a.chunk_bytes / a.parts;
    const uint32_t nvec = static_cast<uint32_t>(part_bytes >> 4);
    for (uint32_t t = g; t < tiles; t += G) {
        const uint32_t grp = t / K, k = t - grp * K;
        const uint32_t i0 = grp * TB;
        const uint32_t ni = a.n_items - i0 < TB ? a.n_items - i0 : TB;
        const uint64_t cache = table[k];
        const uint64_t coff = static_cast<uint64_t>(a.chunk0 + k) * a.chunk_bytes;
        // the tile's work items, all fetched (scalar loads) before its first copy;
        // indices past the last item are clamped to it and never copied
        uint64_t pool_of[kTileItems], slot_of[kTileItems];
#pragma unroll
        for (uint32_t j = 0; j < kTileItems; ++j) {
            const uint32_t i = i0 + (j < ni ? j : ni - 1);
            pool_of[j] = items[i].pool + coff;
            slot_of[j] = cache + static_cast<uint64_t>(items[i].slot) * a.chunk_bytes;
        }
#pragma unroll
        for (uint32_t j = 0; j < kTileItems; ++j) {
            if (j >= ni) break;
            const uint64_t pool = pool_of[j], slot = slot_of[j];
            for (uint32_t p = 0; p < a.parts; ++p) {
                const uint64_t off = p * part_bytes;
                const v4u *src = reinterpret_cast<const v4u *>(GATHER ? pool + off : slot + off);
                v4u *dst = reinterpret_cast<v4u *>(GATHER ? slot + off : pool + off);
                if constexpr (FORM == kPlain)
                    wg_copy<UNROLL, NTL, NTS>(src, dst, nvec);
                else if constexpr (FORM == kConvert)
                    wg_convert<GATHER, UNROLL, NTL, NTS>(src, dst, nvec, a.heads, a.tokens, a.row_vec);
                else
                    wg_convert_lds<GATHER, UNROLL, NTL, NTS>(src, dst, nvec, a.heads, a.tokens, a.row_vec, lds);
            }
        }
    }
}

// A launch of one class: the work list and table in device memory, every
// workgroup on its items.
template <bool GATHER, int FORM, int UNROLL, bool NTL, bool NTS>
__device__ __forceinline__ void class_body(const CopyArgs &a)
{
    uint32_t g = blockIdx.x;
    if (a.xcd_remap) {
        // workgroups are dealt to the 8 XCDs round-robin; renumber them so that
        // each XCD takes one contiguous run of units per pass over the grid
        const uint32_t per = gridDim.x / kXcds;          // grid is a multiple of 8 here
        g = (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
    }
    if (a.tile_items)
        chunk_copy_tiles<GATHER, FORM, UNROLL, NTL, NTS>(a, (citem_t *)a.items, (cptr_t *)a.cache, g, gridDim.x);
    else
        chunk_copy_body<GATHER, FORM, UNROLL, NTL, NTS>(a, (citem_t *)a.items, (cptr_t *)a.cache, g, gridDim.x);
}

// HBM body: one 16-byte vector per lane, one load and one store, for HBM on
// both sides.  Bound by HBM bandwidth, and there by how the traffic is spread
// in time, not by bytes in flight: a contiguous 8 GiB copy on this chip moves
// 5.5 TB/s (read + written) with four vectors per lane and 16 KiB per
// workgroup, 5.8 with two and 6.4 with one, whose short-lived wavefronts keep
// the addresses in flight in a window of 8 MiB instead of 32.
//
// A unit is one wavefront's 64 vectors (1 KiB) of a chunk, the last of a chunk
// shorter; a workgroup is four units.  Units are ordered so that the *written*
// side runs on: the retrieve by groups of 4 chunks (chunk group, work item,
// chunk, unit: with work items in slot order it writes up to 64-slot runs of
// four engine buffers while it reads 4-chunk pieces of each block), the store
// item by item (it writes whole pool blocks).  Within that order each XCD
// takes runs of 256 workgroups (1 MiB) instead of every eighth workgroup.  Whole
// calls, dealt out one by one / in runs: 8192 LLaMA-shaped blocks over four
// regions 5843 / 5482 us, 2048 of them token-major 1537 / 1427, the same layer
// by layer 1691 / 1667, 3271 Qwen3-shaped ones 1721 / 1690, 4096 of those stored
// and 8192 GPT-OSS-shaped ones level.  What a run gains depends on where the
// memory lies: blocks of a single region of 4 to 17 GB took -1 to +7 % more time
// with runs in a retrieve and -5 to +2 % in a store.  It is not translation
// (level UTCL1 misses in the retrieve, 3 to 50 times as many in the store).
// Measured on 8.6 GB in 32 KiB chunks with ascending slots, traffic of the kernel
// alone: retrieve 6465 GB/s against 5694 for half-chunk units of four vectors
// per lane in chunk order; store 6151 against 5407.  Chunks that are no whole
// number of units (6400 bytes) retrieve at 6122 chunk by chunk and at 5770 in
// groups of four.
//
// Token-major chunks take the same body: a lane's source vector is looked up
// by its destination index, so stores stay contiguous and loads come in rows
// of head_dim, which the caches merge into whole lines (rows of 256 bytes:
// 6267 GB/s retrieved against 5560 staged through LDS, whose barrier puts a
// chunk's loads and stores in turn; 160 bytes: 5692; 64 bytes: 5682).
constexpr uint32_t kRunShift = 8;     // workgroups of an XCD's run: 2^8
constexpr uint32_t kChunkGroup = 4;   // chunks of a retrieve's chunk group

// Workgroup b of n in run order: of every 8 * 2^kRunShift workgroups, those of
// one XCD (dealt round-robin, b % 8) take a contiguous 2^kRunShift, and of a
// shorter rest an equal share.  A permutation of [0, n).
__device__ __host__ inline uint32_t run_order(uint32_t b, uint32_t n)
{
    constexpr uint32_t kGroup = kXcds << kRunShift;
    const uint32_t full = n & ~(kGroup - 1), x = b % kXcds;
    if (b < full) return (b & ~(kGroup - 1)) + (x << kRunShift) + (b & (kGroup - 1)) / kXcds;
    const uint32_t share = (n - full) / kXcds, longer = (n - full) % kXcds;
    return full + x * share + (x < longer ? x : longer) + (b - full) / kXcds;
}

template <bool GATHER, bool TOKEN_MAJOR, bool NTL, bool NTS>
__device__ __forceinline__ void wave_copy_body(const CopyArgs &a, citem_t *items, cptr_t *table, uint32_t g, uint32_t G)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const uint32_t nvec = static_cast<uint32_t>(a.chunk_bytes >> 4);
    const uint32_t wgs = (a.units + kWaves - 1) / kWaves;
    for (uint32_t b = g; b < wgs; b += G) {
        const uint32_t u = run_order(b, wgs) * kWaves + wave;
        if (u >= a.units) continue;
        const uint32_t per_group = a.n_items * a.chunk_units * a.group;
        const uint32_t k0 = u / per_group * a.group;
        uint32_t r = u - k0 * a.n_items * a.chunk_units;
        const uint32_t per_item = (a.chunks - k0 < a.group ? a.chunks - k0 : a.group) * a.chunk_units;
        const uint32_t item = r / per_item;
        r -= item * per_item;
        const uint32_t kk = r / a.chunk_units;
        const uint32_t k = k0 + kk;
        const uint64_t pool = items[item].pool + static_cast<uint64_t>(a.chunk0 + k) * a.chunk_bytes;
        const uint64_t cache = table[k] + static_cast<uint64_t>(items[item].slot) * a.chunk_bytes;
        const v4u *src = reinterpret_cast<const v4u *>(GATHER ? pool : cache);
        v4u *dst = reinterpret_cast<v4u *>(GATHER ? cache : pool);
        uint32_t v = (r - kk * a.chunk_units) * a.unit_vecs + lane;
        for (uint32_t i = 0; i < a.unit_vecs; i += kWave, v += kWave) {   // once, but for chunks of gigabytes
            const uint32_t d = clamp_index(v, nvec);   // loads are never predicated
            uint32_t w = d;
            if constexpr (TOKEN_MAJOR) w = src_of<GATHER>(d, a.heads, a.tokens, a.row_vec);
            const v4u x = load16<NTL>(src + w);
            if (v < nvec) store16<NTS>(dst + v, x);
        }
    }
}

// One entry point per kind of source, so that traces and counters tell the
// zero-copy (host link) kernel, the HBM staging kernel and the kernel that
// empties / fills a copy-engine ring slot apart.  The body is the same.
template <bool GATHER, int FORM, int UNROLL, bool NTL, bool NTS>
__global__ __launch_bounds__(kThreads) void host_region_copy(CopyArgs a)
{
    class_body<GATHER, FORM, UNROLL, NTL, NTS>(a);
}

template <bool GATHER, bool TOKEN_MAJOR, bool NTL, bool NTS>
__global__ __launch_bounds__(kThreads) void staging_region_copy(CopyArgs a)
{
    wave_copy_body<GATHER, TOKEN_MAJOR, NTL, NTS>(a, (citem_t *)a.items, (cptr_t *)a.cache, blockIdx.x, gridDim.x);
}

template <bool GATHER, bool TOKEN_MAJOR, bool NTL, bool NTS>
__global__ __launch_bounds__(kThreads) void ring_slot_copy(CopyArgs a)
{
    wave_copy_body<GATHER, TOKEN_MAJOR, NTL, NTS>(a, (citem_t *)a.items, (cptr_t *)a.cache, blockIdx.x, gridDim.x);
}

template <bool GATHER, int FORM, int UNROLL, bool NTL, bool NTS>
__global__ __launch_bounds__(kThreads) void file_slot_copy(CopyArgs a)
{
    class_body<GATHER, FORM, UNROLL, NTL, NTS>(a);
}

// Both classes of a call in one launch: workgroups [0, grid_host) take the
// host-class items, the others the staging-class items, so the two run side by
// side with no second stream and no events between.  FORM to NTS are the host
// class's copy form; the staging class takes its own body with non-temporal
// stores, and loads too unless cached_loads.  The table and the
// items are read with scalar loads, from the kernel arguments (a small call) or
// from the uploaded work list.  The class split is uniform per workgroup.
template <bool GATHER, int FORM, int UNROLL, bool NTL, bool NTS>
__global__ __launch_bounds__(kThreads) void both_regions_copy(CallArgs f)
{
    // f is the kernel's only explicit argument, so it sits at offset 0 of the
    // kernel-argument segment; the table and the items are addressed there
    // (constant address space, scalar loads), never through a copy of f.
    typedef __attribute__((address_space(4))) const char cchar_t;
    cchar_t *words = (cchar_t *)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(CallArgs, words);
    const bool inlined = f.a.items == nullptr;
    cptr_t *table = inlined ? (cptr_t *)words : (cptr_t *)f.a.cache;
    citem_t *items = inlined ? (citem_t *)(words + static_cast<uint64_t>(f.a.chunks) * sizeof(uint64_t))
                             : (citem_t *)f.a.items;
    CopyArgs a = f.a;
    // the staging-class workgroups start at a multiple of 8, so that their
    // numbers tell their XCD; up to 7 workgroups between the classes end at once
    const uint32_t first = (f.grid_host + kXcds - 1) / kXcds * kXcds;
    if (blockIdx.x < f.grid_host) {
        a.n_items = f.n_host;
        chunk_copy_body<GATHER, FORM, UNROLL, NTL, NTS>(a, items, table, blockIdx.x, f.grid_host);
    } else if (blockIdx.x >= first) {
        a.n_items = f.a.n_items - f.n_host;
        const uint32_t g = blockIdx.x - first, G = gridDim.x - first;
        if (FORM != kPlain && f.cached_loads)
            wave_copy_body<GATHER, FORM != kPlain, false, true>(a, items + f.n_host, table, g, G);
        else
            wave_copy_body<GATHER, FORM != kPlain, true, true>(a, items + f.n_host, table, g, G);
    }
}

// A call's work list from its pinned buffer to device memory, one 16-byte
// vector per lane.  A kernel and not a copy: in line on the caller's stream it
// takes about 4 us and needs neither the copy's own barriers nor an event from
// another stream (a stream copy of the same list left the stream idle for 23 us
// before and 11 us after its 4 us).
__global__ __launch_bounds__(kThreads) void list_copy(const v4u *__restrict__ src, v4u *__restrict__ dst, uint32_t nvec)
{
    const uint32_t v = blockIdx.x * kThreads + threadIdx.x;
    if (v < nvec) store16<false>(dst + v, load16<false>(src + v));
}

// Contiguous streaming copy over tiles of 256*UNROLL vectors (bandwidth probe; one
// vector per lane and one tile per workgroup is what HBM copies fastest).
template <int UNROLL, bool NTL, bool NTS>
__global__ __launch_bounds__(kThreads) void probe_copy_kernel(const v4u *__restrict__ src, v4u *__restrict__ dst,
                                                              uint64_t nvec)
{
    const uint64_t tile = static_cast<uint64_t>(kThreads) * UNROLL;
    const uint64_t tiles = (nvec + tile - 1) / tile;
    for (uint64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const uint64_t base = t * tile;
        const uint64_t left = nvec - base;
        wg_copy<UNROLL, NTL, NTS>(src + base, dst + base, static_cast<uint32_t>(left < tile ? left : tile));
    }
}

// ---------------------------------------------------------------- static work-list scratch

// The work list of kv_pool_retrieve_noalloc lives here instead of in memory
// the library allocates.  Host code never passes this name to a kernel or a
// copy: on the host it is only a stand-in for the symbol, and its device
// address (one per GPU) comes from hipGetSymbolAddress in scratch_setup.
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
ScratchDevice g_scratch[kMaxScratchDevices];
std::mutex g_scratch_setup;
}  // namespace

ScratchDevice &scratch_setup(int device)
{
    if (device < 0 || device >= kMaxScratchDevices)
        fail(KVP_ERR_INVALID, "device " + std::to_string(device) + " outside the scratch table");
    ScratchDevice &sd = g_scratch[device];
    std::lock_guard<std::mutex> lock(g_scratch_setup);
    if (sd.ready) return sd;
    void *dev = nullptr;
    check_hip(hipGetSymbolAddress(&dev, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    if (!dev || (reinterpret_cast<uintptr_t>(dev) & 255))
        fail(KVP_ERR_HIP, "scratch symbol has no 256-byte aligned device address");
    void *host = nullptr, *host_dev = nullptr;
    if (hipHostMalloc(&host, kScratchBytes, kListMemory) != hipSuccess || !host) {
        clear_hip_error();
        fail(KVP_ERR_NOMEM, "pinned staging buffer of the static scratch");
    }
    if (const hipError_t r = hipHostGetDevicePointer(&host_dev, host, 0); r != hipSuccess) {
        (void)hipHostFree(host);
        check_hip(r, "hipHostGetDevicePointer");
    }
    sd.dev = dev;
    sd.host = host;
    sd.host_dev = host_dev;
    sd.ready = true;
    return sd;
}

ScratchDevice &scratch_device(int device)
{
    if (device < 0 || device >= kMaxScratchDevices || !g_scratch[device].ready)
        fail(KVP_ERR_INVALID, "static scratch of device " + std::to_string(device) + " is not set up");
    return g_scratch[device];
}

// ---------------------------------------------------------------- host-side dispatch

constexpr uint32_t kClassBoth = 3;   // dispatch only: both_regions_copy

__device__ __host__ inline const CopyArgs &geometry(const CopyArgs &a) { return a; }
__device__ __host__ inline const CopyArgs &geometry(const CallArgs &f) { return f.a; }

template <uint32_t CLS, bool GATHER, int FORM, int UNROLL, bool NTL, bool NTS, class A>
static void launch_one(const A &a, dim3 g, size_t lds, hipStream_t s)
{
    if constexpr (CLS == kClassBoth)
        hipLaunchKernelGGL((both_regions_copy<GATHER, FORM, UNROLL, NTL, NTS>), g, dim3(kThreads), lds, s, a);
    else if constexpr (CLS == KVP_CLASS_HOST)
        hipLaunchKernelGGL((host_region_copy<GATHER, FORM, UNROLL, NTL, NTS>), g, dim3(kThreads), lds, s, a);
    else
        hipLaunchKernelGGL((file_slot_copy<GATHER, FORM, UNROLL, NTL, NTS>), g, dim3(kThreads), lds, s, a);
}

template <uint32_t CLS, bool GATHER, int FORM, int UNROLL, class A>
static hipError_t launch_form(const A &a, uint32_t grid, uint32_t flags, size_t lds, hipStream_t s)
{
    const bool ntl = flags & KVP_LAUNCH_NT_LOAD, nts = flags & KVP_LAUNCH_NT_STORE;
    const dim3 g(grid);
    if (ntl && nts)
        launch_one<CLS, GATHER, FORM, UNROLL, true, true>(a, g, lds, s);
    else if (ntl)
        launch_one<CLS, GATHER, FORM, UNROLL, true, false>(a, g, lds, s);
    else if (nts)
        launch_one<CLS, GATHER, FORM, UNROLL, false, true>(a, g, lds, s);
    else
        launch_one<CLS, GATHER, FORM, UNROLL, false, false>(a, g, lds, s);
    return hipGetLastError();
}

template <uint32_t CLS, bool GATHER, int FORM, class A>
static hipError_t launch_unroll(const A &a, uint32_t grid, uint32_t flags, size_t lds, hipStream_t s)
{
    // enough 16-byte loads in flight per lane to cover the whole unit, up to 8
    const CopyArgs &geo = geometry(a);
    const uint64_t per_lane = (geo.chunk_bytes / geo.parts / 16 + kThreads - 1) / kThreads;
    if (per_lane >= 8) return launch_form<CLS, GATHER, FORM, 8>(a, grid, flags, lds, s);
    if (per_lane >= 4) return launch_form<CLS, GATHER, FORM, 4>(a, grid, flags, lds, s);
    if (per_lane >= 2) return launch_form<CLS, GATHER, FORM, 2>(a, grid, flags, lds, s);
    return launch_form<CLS, GATHER, FORM, 1>(a, grid, flags, lds, s);
}

template <uint32_t CLS, bool GATHER, class A>
static hipError_t launch_dir(const A &a, uint32_t grid, uint32_t flags, hipStream_t s)
{
    const CopyArgs &geo = geometry(a);
    if (geo.layout == 0) return launch_unroll<CLS, GATHER, kPlain>(a, grid, flags, 0, s);
    if ((flags & KVP_LAUNCH_LDS) && geo.chunk_bytes <= kMaxLdsChunk)
        return launch_unroll<CLS, GATHER, kConvertLds>(a, grid, flags, geo.chunk_bytes, s);
    return launch_unroll<CLS, GATHER, kConvert>(a, grid, flags, 0, s);
}

// Units of the HBM body and their order for a launch of n items.  Launches of
// over 2^31 units (terabytes) take more vectors per unit, so that a unit index
// plus the workgroup stride stays within 32 bits.
static void wave_units(CopyArgs &a, uint32_t n, bool gather)
{
    const uint64_t nvec = a.chunk_bytes >> 4, per_vec = static_cast<uint64_t>(n) * a.chunks;
    uint64_t vecs = kWave;
    while (per_vec * ((nvec + vecs - 1) / vecs) > (1ull << 31)) vecs *= 2;
    a.unit_vecs = static_cast<uint32_t>(vecs);
    a.chunk_units = static_cast<uint32_t>((nvec + vecs - 1) / vecs);
    a.units = static_cast<uint32_t>(per_vec * a.chunk_units);
    a.group = !gather ? a.chunks : a.chunk_bytes % (kWave * 16) ? 1u : a.chunks < kChunkGroup ? a.chunks : kChunkGroup;
}

// Workgroups of the HBM body: one per four units, at most `grid` of them.
static uint32_t wave_grid(const CopyArgs &a, uint32_t grid)
{
    const uint32_t wgs = a.units / kWaves + (a.units % kWaves != 0);
    return grid == 0 ? 1u : grid < wgs ? grid : wgs;
}

template <uint32_t CLS, bool GATHER, bool TOKEN_MAJOR, bool NTL, bool NTS>
static hipError_t launch_wave_one(const CopyArgs &a, dim3 g, hipStream_t s)
{
    if constexpr (CLS == KVP_CLASS_STAGING)
        hipLaunchKernelGGL((staging_region_copy<GATHER, TOKEN_MAJOR, NTL, NTS>), g, dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((ring_slot_copy<GATHER, TOKEN_MAJOR, NTL, NTS>), g, dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

template <uint32_t CLS, bool GATHER, bool TOKEN_MAJOR>
static hipError_t launch_wave_nt(const CopyArgs &a, dim3 g, uint32_t flags, hipStream_t s)
{
    const bool ntl = flags & KVP_LAUNCH_NT_LOAD, nts = flags & KVP_LAUNCH_NT_STORE;
    if (ntl && nts) return launch_wave_one<CLS, GATHER, TOKEN_MAJOR, true, true>(a, g, s);
    if (ntl) return launch_wave_one<CLS, GATHER, TOKEN_MAJOR, true, false>(a, g, s);
    if (nts) return launch_wave_one<CLS, GATHER, TOKEN_MAJOR, false, true>(a, g, s);
    return launch_wave_one<CLS, GATHER, TOKEN_MAJOR, false, false>(a, g, s);
}

template <uint32_t CLS>
static hipError_t launch_wave(CopyArgs a, bool gather, uint32_t grid, uint32_t flags, hipStream_t s)
{
    wave_units(a, a.n_items, gather);
    const dim3 g(wave_grid(a, grid));
    if (a.layout == 0)
        return gather ? launch_wave_nt<CLS, true, false>(a, g, flags, s) : launch_wave_nt<CLS, false, false>(a, g, flags, s);
    return gather ? launch_wave_nt<CLS, true, true>(a, g, flags, s) : launch_wave_nt<CLS, false, true>(a, g, flags, s);
}

hipError_t launch_chunk_copy(const CopyArgs &args, uint32_t cls, bool gather, uint32_t grid, uint32_t flags,
                             hipStream_t s)
{
    if (args.n_items == 0) return hipSuccess;
    if (cls == KVP_CLASS_STAGING) return launch_wave<KVP_CLASS_STAGING>(args, gather, grid, flags, s);
    if (cls == kClassRing) return launch_wave<kClassRing>(args, gather, grid, flags, s);
    CopyArgs a = args;
    // halves of a plain chunk are independent contiguous copies
    a.parts = (a.layout == 0 && (flags & KVP_LAUNCH_SPLIT2) && a.chunk_bytes % 32 == 0) ? 2u : 1u;
    const uint64_t units = static_cast<uint64_t>(a.n_items) * a.chunks * a.parts;
    if (grid > units) grid = static_cast<uint32_t>(units);
    if (grid == 0) grid = 1;
    // the XCD renumbering is a permutation of [0, grid) only for multiples of 8
    a.xcd_remap = (flags & KVP_LAUNCH_XCD) && grid % kXcds == 0 ? 1u : 0u;
    a.chunk_major = (flags & KVP_LAUNCH_CHUNK_MAJOR) ? 1u : 0u;
    a.tile_items = (flags & KVP_LAUNCH_TILE) ? kTileItems : 0u;
    if (a.tile_items) {   // a grid of at most one workgroup per tile
        const uint64_t tiles = (static_cast<uint64_t>(a.n_items) + kTileItems - 1) / kTileItems * a.chunks;
        if (grid > tiles) grid = static_cast<uint32_t>(tiles);
        a.xcd_remap = (flags & KVP_LAUNCH_XCD) && grid % kXcds == 0 ? 1u : 0u;
    }
    if (cls == KVP_CLASS_HOST)
        return gather ? launch_dir<KVP_CLASS_HOST, true>(a, grid, flags, s)
                      : launch_dir<KVP_CLASS_HOST, false>(a, grid, flags, s);
    return gather ? launch_dir<kClassFile, true>(a, grid, flags, s) : launch_dir<kClassFile, false>(a, grid, flags, s);
}

hipError_t launch_call(CallArgs &f, bool gather, uint32_t grid_host, uint32_t grid_staging, uint32_t flags,
                       uint32_t staging_flags, hipStream_t s)
{
    CopyArgs &a = f.a;
    if (a.n_items == 0) return hipSuccess;
    a.parts = (a.layout == 0 && (flags & KVP_LAUNCH_SPLIT2) && a.chunk_bytes % 32 == 0) ? 2u : 1u;
    a.xcd_remap = 0;
    a.chunk_major = 0;
    a.tile_items = 0;
    const uint64_t host_units = static_cast<uint64_t>(f.n_host) * a.chunks * a.parts;
    f.grid_host = static_cast<uint32_t>(grid_host < host_units ? grid_host : host_units);
    uint32_t grid = f.grid_host;
    const uint32_t n_staging = a.n_items - f.n_host;
    if (n_staging) {
        wave_units(a, n_staging, gather);
        grid = (grid + kXcds - 1) / kXcds * kXcds + wave_grid(a, grid_staging);
    }
    f.cached_loads = (staging_flags & KVP_LAUNCH_NT_LOAD) ? 0u : 1u;
    if (f.n_host == 0) flags &= ~KVP_LAUNCH_LDS;   // the staging class stages nothing through LDS
    return gather ? launch_dir<kClassBoth, true>(f, grid, flags, s) : launch_dir<kClassBoth, false>(f, grid, flags, s);
}

hipError_t launch_list_copy(void *dst, const void *src, uint64_t bytes, hipStream_t s)
{
    const uint32_t nvec = static_cast<uint32_t>(bytes / 16);
    if (nvec == 0) return hipSuccess;
    hipLaunchKernelGGL(list_copy, dim3((nvec + kThreads - 1) / kThreads), dim3(kThreads), 0, s,
                       static_cast<const v4u *>(src), static_cast<v4u *>(dst), nvec);
    return hipGetLastError();
}

template <int UNROLL>
static hipError_t launch_probe(const v4u *sp, v4u *dp, uint64_t nvec, uint32_t grid, uint32_t flags, hipStream_t s)
{
    const uint64_t tile = kThreads * UNROLL, tiles = (nvec + tile - 1) / tile;
    if (grid == 0) grid = UNROLL == 1 ? 1u << 23 : 2048u;
    const dim3 g(static_cast<uint32_t>(grid < tiles ? grid : tiles)), b(kThreads);
    const bool ntl = flags & KVP_LAUNCH_NT_LOAD, nts = flags & KVP_LAUNCH_NT_STORE;
    if (ntl && nts)
        hipLaunchKernelGGL((probe_copy_kernel<UNROLL, true, true>), g, b, 0, s, sp, dp, nvec);
    else if (ntl)
        hipLaunchKernelGGL((probe_copy_kernel<UNROLL, true, false>), g, b, 0, s, sp, dp, nvec);
    else if (nts)
        hipLaunchKernelGGL((probe_copy_kernel<UNROLL, false, true>), g, b, 0, s, sp, dp, nvec);
    else
        hipLaunchKernelGGL((probe_copy_kernel<UNROLL, false, false>), g, b, 0, s, sp, dp, nvec);
    return hipGetLastError();
}

hipError_t launch_probe_copy(void *dst, const void *src, uint64_t bytes, uint32_t grid, uint32_t flags,
                             hipStream_t s)
{
    const uint64_t nvec = bytes / 16;
    if (nvec == 0) return hipSuccess;
    const v4u *sp = static_cast<const v4u *>(src);
    v4u *dp = static_cast<v4u *>(dst);
    if (flags & KVP_LAUNCH_TILE) return launch_probe<1>(sp, dp, nvec, grid, flags, s);
    if (flags & KVP_LAUNCH_SPLIT2) return launch_probe<4>(sp, dp, nvec, grid, flags, s);
    return launch_probe<8>(sp, dp, nvec, grid, flags, s);
}

}  // namespace kvp
