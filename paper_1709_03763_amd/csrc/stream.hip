// Memory-capped streaming of voxel blocks between the GPU and the host
// (Sec. 3, "SDF volume": only the blocks near the camera are kept in GPU
// memory, the others are streamed to the host; Sec. 4.3: before a
// re-integration the blocks around the poses it works at are streamed in).
//
// The device pool holds at most max_blocks blocks.  sc_stream_out moves
// every block whose centre lies outside a sphere to a host store and
// compacts the pool; in streaming mode every operation (plain or batched)
// first streams in, from the host store, exactly those of its candidate
// blocks that the store holds, so each operation sees every block it can
// touch and the field equals the one a fully resident volume would hold,
// bit for bit, whatever sphere the caller streams to.  The sphere decides
// only how much stays on the device between calls.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <unordered_map>
#include <vector>

#include "common.hpp"
#include "internal.hpp"
#include "kernels.hpp"

// A block on its way: its host record, and its pool slot (out) with the slot
// of the block that takes its place (out: -1 for none).  The kernels read the
// list in pinned memory.
struct StreamItem {
    uint64_t key;
    unsigned char* host;
    int32_t slot, mover;
};

// What an operation's stage tells the host: requested and candidate blocks,
// allocated blocks, sticky error.
struct StreamReport {
    uint32_t n_req, n_cand, n_blocks;
    int32_t err;
};

// A host record.
struct StreamRec {
    unsigned char* p;
    bool pinned;
};
struct StreamChunk {
    unsigned char* p;
    size_t blocks;
    bool pinned;
};
constexpr size_t kStageBlocks = 256;  // records of pageable memory moved at once

// Host side of the streaming mode.  The records lie in chunks of pinned
// memory, which the kernels write and read themselves: no staging copy on
// either side, and the host waits once an operation, for the report.  Where no
// more memory can be pinned the chunks are pageable, and their records pass
// through a pinned staging buffer, with a wait for every kStageBlocks of them.
struct StreamStore {
    bool enabled = false;
    size_t block_bytes = 0;                              // one block's record in the pool
    std::unordered_map<uint64_t, StreamRec> where;       // block key -> host record
    std::vector<StreamChunk> chunks;
    size_t pinned = 0, pinned_limit = SIZE_MAX;          // bytes of the pinned chunks, and at most
    size_t cur = 0, pos = 0;                             // first record never used: in chunk cur at pos
    std::vector<StreamRec> free_recs;
    unsigned char* stage = nullptr;                      // pinned, kStageBlocks records
    bool surplus = false;  // a reset left chunks beyond kKeepBytes: freed at the next wait
    StreamItem* in = nullptr;   // pinned lists
    StreamItem* out = nullptr;
    size_t in_cap = 0, out_cap = 0;
    StreamReport* report = nullptr;  // pinned
    uint64_t* h_keys = nullptr;      // pinned: requested keys, or those of the device blocks
    uint64_t* d_all = nullptr;       // device: every candidate key of the operation or chunk
    size_t keys_cap = 0;
    uint32_t* d_req = nullptr;       // device counter, zero between operations
    hipEvent_t done = nullptr;       // after the last kernel that uses the lists or records
    int64_t blocks_out = 0, blocks_in = 0;
};

namespace sc {

// ---------------------------------------------------------------------------
// device kernels
// ---------------------------------------------------------------------------

// Inserts (key, slot) into the block hash (the key is absent).
__device__ inline void hash_put(const VolDev& v, uint64_t key, int slot)
{
    int bx, by, bz;
    unpack_key(key, bx, by, bz);
    uint32_t h = hash_block(bx, by, bz) & v.bucket_mask;
    for (uint32_t probe = 0; probe <= v.bucket_mask; ++probe) {
        const uint64_t old =
            atomicCAS((unsigned long long*)(v.keys + h), (unsigned long long)kKeyEmpty, (unsigned long long)key);
        if (old == kKeyEmpty) {
            v.vals[h] = slot;
            return;
        }
        h = (h + 1) & v.bucket_mask;
    }
    set_error(v.err, SC_EHASHFULL);
}

// Appends the requested keys of a wavefront to the list in pinned memory: one
// counter update, and the keys leave in one piece.
__device__ inline void request(bool mine, uint64_t key, uint64_t* req, uint32_t* count, uint32_t cap)
{
    const uint64_t m = __ballot(mine);
    if (m == 0ull) return;
    const int lane = threadIdx.x & 63;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(count, (uint32_t)__popcll(m));
    base = __shfl(base, 0);
    const uint32_t p = base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    if (mine && p < cap) req[p] = key;
}

// Keys of the batched candidate blocks (all of them into `all`, count in
// cd.counters[4]) and of those without a device slot (new blocks, or blocks
// held by the host store) into `req`.
__global__ void stream_req_batch_kernel(CandDev cd, uint64_t* all, uint64_t* req, uint32_t* count, uint32_t cap)
{
    const uint32_t n = min(cd.counters[4], cap);
    // whole wavefronts stay in the loop
    for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < n; i0 += gridDim.x * blockDim.x) {
        const uint32_t i = i0 + threadIdx.x;
        const uint64_t key = i < n ? cd.skey[i] : 0ull;
        if (i < n) all[i] = key;
        request(i < n && cd.sslot[min(i, n - 1)] < 0, key, req, count, cap);
    }
}

// The same for the plain path's candidate list (its length in
// counters[parity]).
__global__ void stream_req_plain_kernel(CandDev cd, VolDev v, int parity, uint64_t* all, uint64_t* req,
                                        uint32_t* count, uint32_t cap)
{
    const uint32_t n = min(min(cd.counters[parity], cd.cap), cap);
    for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < n; i0 += gridDim.x * blockDim.x) {
        const uint32_t i = i0 + threadIdx.x;
        bool mine = false;
        uint64_t key = 0;
        if (i < n) {
            key = cd.keys[cd.list[i]];
            all[i] = key;
            int bx, by, bz;
            unpack_key(key, bx, by, bz);
            mine = vol_find(v, key, bx, by, bz) < 0;
        }
        request(mine, key, req, count, cap);
    }
}

// The report of the requests, which it also empties.
__global__ void stream_report_kernel(const uint32_t* n_cand, uint32_t* n_req, VolDev v, StreamReport* r)
{
    r->n_cand = *n_cand;
    r->n_req = *n_req;
    r->n_blocks = *v.n_blocks;
    r->err = *v.err;
    *n_req = 0u;
}

// Keys of the device blocks in slot order, with their number and the error.
__global__ void stream_keys_kernel(VolDev v, uint64_t* keys, uint32_t cap, StreamReport* r)
{
    const uint32_t nb = *v.n_blocks, n = min(nb, cap);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        keys[i] = v.slot_keys[i];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        r->n_blocks = nb;
        r->err = *v.err;
    }
}

// Streamed-in blocks i < n take pool slots base + i: data from the host
// record, key, hash entry.  A workgroup a block, 16 bytes a lane: bound by the
// bus, 450 blocks of 8 KB in 75 us (49 GB/s).  Copied to staging by the host,
// to the device, and from there into the pool, with five waits, an integration
// that streamed in so many took 335 us, now 160.
__global__ __launch_bounds__(256) void stream_in_kernel(VolDev v, const StreamItem* __restrict__ items, int64_t n,
                                                        int64_t base)
{
    const int64_t i = blockIdx.x;
    if (i >= n) return;
    const int slot = (int)(base + i);
    const StreamItem it = items[i];
    float4* dst = reinterpret_cast<float4*>(v.pool + (size_t)slot * v.stride);
    const float4* __restrict__ src = reinterpret_cast<const float4*>(it.host);
#pragma unroll 2
    for (int k = threadIdx.x; k < v.stride / 4; k += blockDim.x) dst[k] = src[k];
    if (threadIdx.x == 0) {
        v.slot_keys[slot] = it.key;
        hash_put(v, it.key, slot);
        if (i == 0) *v.n_blocks = (uint32_t)(base + n);
    }
}

// Looks up the pool slot of every batched candidate again (blocks were
// streamed in, or moved by a compaction).
__global__ void sslot_refresh_kernel(CandDev cd, VolDev v)
{
    const uint32_t n = cd.counters[4];
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        int bx, by, bz;
        unpack_key(cd.skey[i], bx, by, bz);
        cd.sslot[i] = vol_find(v, cd.skey[i], bx, by, bz);
    }
}

// Evicted block i goes to its host record; the live block of slot `mover`
// takes its slot, if there is one, and the slot left free is cleared to the
// empty state.  A lane does all of that for its own elements, so nothing waits
// on another.  The workgroups also empty the hash table.  Bound by the bus, 500
// blocks of 8 KB in 77 us (53 GB/s).  Gathered to staging, copied to the host
// and again into the store, then the moves and fills in launches of their own,
// a call that sent 420 blocks out took 380 us, now 145.
__global__ __launch_bounds__(256) void stream_out_kernel(VolDev v, const StreamItem* __restrict__ items, int64_t n)
{
    const int64_t i = blockIdx.x;
    if (i < n) {
        const StreamItem it = items[i];
        float4* at = reinterpret_cast<float4*>(v.pool + (size_t)it.slot * v.stride);
        float4* from = it.mover >= 0 ? reinterpret_cast<float4*>(v.pool + (size_t)it.mover * v.stride) : at;
        float4* host = reinterpret_cast<float4*>(it.host);
        const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 2
        for (int k = threadIdx.x; k < v.stride / 4; k += blockDim.x) {
            const float4 gone = at[k], live = from[k];
            host[k] = gone;
            if (it.mover >= 0) at[k] = live;
            from[k] = zero;
        }
        if (threadIdx.x == 0 && it.mover >= 0) v.slot_keys[it.slot] = v.slot_keys[it.mover];
    }
    for (uint64_t b = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; b <= v.bucket_mask;
         b += (uint64_t)gridDim.x * blockDim.x) {
        v.keys[b] = kKeyEmpty;
        v.vals[b] = -1;
    }
}

// Re-inserts the blocks of slots [0, n) into the (cleared) hash table.
__global__ void hash_rebuild_kernel(VolDev v, int64_t n)
{
    for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < n; s += (int64_t)gridDim.x * blockDim.x)
        hash_put(v, v.slot_keys[s], (int)s);
    if (blockIdx.x == 0 && threadIdx.x == 0) *v.n_blocks = (uint32_t)n;
}

__global__ void set_error_kernel(int32_t* err, int32_t code) { set_error(err, code); }

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

static bool grow_items(StreamItem*& list, size_t& cap, size_t n)
{
    if (n <= cap) return true;
    const size_t c = std::max({n, 2 * cap, (size_t)1024});
    if (list) (void)hipHostFree(list);
    list = nullptr;
    cap = 0;
    if (hipHostMalloc((void**)&list, c * sizeof(StreamItem), hipHostMallocCoherent) != hipSuccess) {
        (void)hipGetLastError();
        list = nullptr;
        return false;
    }
    cap = c;
    return true;
}

static bool grow_keys(StreamStore* st, size_t n)
{
    if (n <= st->keys_cap) return true;
    const size_t cap = std::max(n, 2 * st->keys_cap);
    if (hipDeviceSynchronize() != hipSuccess) return false;
    if (st->h_keys) (void)hipHostFree(st->h_keys);
    (void)hipFree(st->d_all);
    st->h_keys = nullptr;
    st->d_all = nullptr;
    st->keys_cap = 0;
    if (hipHostMalloc((void**)&st->h_keys, cap * sizeof(uint64_t), hipHostMallocCoherent) != hipSuccess ||
        !device_alloc(&st->d_all, cap * sizeof(uint64_t))) {
        (void)hipGetLastError();
        return false;
    }
    st->keys_cap = cap;
    return true;
}

// Room for n more host records: chunks of 1,024 blocks and more, doubling up
// to 8,192 (64 MiB of RGBA8 blocks).
static bool reserve_recs(StreamStore* st, size_t n)
{
    size_t have = st->free_recs.size();
    for (size_t c = st->cur; c < st->chunks.size(); ++c) have += st->chunks[c].blocks - (c == st->cur ? st->pos : 0);
    while (have < n) {
        const size_t blocks = st->chunks.empty() ? 1024 : std::min<size_t>(2 * st->chunks.back().blocks, 8192);
        const size_t bytes = blocks * st->block_bytes;
        StreamChunk c{nullptr, blocks, false};
        if (bytes <= st->pinned_limit && st->pinned <= st->pinned_limit - bytes) {
            c.pinned = hipHostMalloc((void**)&c.p, bytes, hipHostMallocCoherent) == hipSuccess;
            if (!c.pinned) (void)hipGetLastError();
        }
        if (!c.pinned) c.p = static_cast<unsigned char*>(malloc(bytes));
        if (!c.p) return false;
        if (c.pinned) st->pinned += bytes;
        st->chunks.push_back(c);
        have += blocks;
    }
    return true;
}

// Frees the chunks from the n-th on.
static void drop_chunks(StreamStore* st, size_t n)
{
    for (size_t c = n; c < st->chunks.size(); ++c) {
        if (st->chunks[c].pinned) {
            (void)hipHostFree(st->chunks[c].p);
            st->pinned -= st->chunks[c].blocks * st->block_bytes;
        } else {
            free(st->chunks[c].p);
        }
    }
    st->chunks.resize(std::min(n, st->chunks.size()));
}

// A free record; there is one (reserve_recs).
static StreamRec take_rec(StreamStore* st)
{
    if (!st->free_recs.empty()) {
        const StreamRec r = st->free_recs.back();
        st->free_recs.pop_back();
        return r;
    }
    while (st->pos == st->chunks[st->cur].blocks) {
        ++st->cur;
        st->pos = 0;
    }
    const StreamChunk& c = st->chunks[st->cur];
    return StreamRec{c.p + st->block_bytes * st->pos++, c.pinned};
}

// The list of an operation's items, their records, and which of them go
// through the staging buffer: the i-th such one at its place i modulo
// kStageBlocks.
struct StreamMoves {
    std::vector<StreamRec> recs;
    std::vector<size_t> staged;  // items

    unsigned char* add(const StreamStore* st, StreamRec r)
    {
        recs.push_back(r);
        if (r.pinned) return r.p;
        staged.push_back(recs.size() - 1);
        return st->stage + st->block_bytes * ((staged.size() - 1) % kStageBlocks);
    }

    // Runs move(a, b) over ranges [a, b) of the items that the staging buffer
    // holds, and before or after it their copies between staging and records.
    template <class Move>
    sc_status run(const StreamStore* st, bool out, hipStream_t s, Move move) const
    {
        size_t a = 0, p = 0;
        while (a < recs.size()) {
            const size_t q = std::min(staged.size(), p + kStageBlocks);
            const size_t b = q < staged.size() ? staged[q] : recs.size();
            auto copy = [&] {
                for (size_t i = p; i < q; ++i) {
                    unsigned char* const rec = recs[staged[i]].p;
                    unsigned char* const stage = st->stage + st->block_bytes * (i - p);
                    memcpy(out ? rec : stage, out ? stage : rec, st->block_bytes);
                }
            };
            if (!out) copy();
            move(a, b);
            if (q > p && (out || b < recs.size()) && hipStreamSynchronize(s) != hipSuccess) return SC_EDEVICE;
            if (out) copy();
            a = b;
            p = q;
        }
        return SC_OK;
    }
};

static bool streaming(const sc_volume* vol) { return vol->stream && vol->stream->enabled; }

int64_t stream_host_blocks(const sc_volume* vol) { return vol->stream ? (int64_t)vol->stream->where.size() : 0; }

// The emptied store keeps chunks up to this size; the others are given back.
constexpr size_t kKeepBytes = (size_t)256 << 20;

// Waits for the report enqueued on `s`, and for the last use of the lists and
// records if that was on another stream; then nothing on the device uses the
// chunks that a reset left over.
static sc_status wait_report(sc_volume* vol, hipStream_t s)
{
    StreamStore* st = vol->stream;
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess ||
        hipEventSynchronize(st->done) != hipSuccess)
        return SC_EDEVICE;
    if (st->surplus) {
        st->surplus = false;
        size_t n = 0, bytes = 0;
        while (n < st->chunks.size() && bytes + st->chunks[n].blocks * st->block_bytes <= kKeepBytes)
            bytes += st->chunks[n++].blocks * st->block_bytes;
        drop_chunks(st, n);
    }
    return SC_OK;
}

static int64_t reported_blocks(const sc_volume* vol)
{
    return std::min<int64_t>((int64_t)vol->stream->report->n_blocks, vol->p.max_blocks);
}

static sc_status d2h(void* dst, const void* src, size_t bytes, hipStream_t s)
{
    if (bytes == 0) return SC_OK;
    if (hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return SC_EDEVICE;
    return SC_OK;
}

// Keys of the device blocks, in slot order, in h_keys (and the number).
// Waits once.
static sc_status device_keys(sc_volume* vol, hipStream_t s, int64_t& nb)
{
    StreamStore* st = vol->stream;
    if (!grow_keys(st, (size_t)vol->p.max_blocks)) return SC_ENOMEM;
    stream_keys_kernel<<<vol->n_cu, 256, 0, s>>>(vol->dev, st->h_keys, (uint32_t)vol->p.max_blocks, st->report);
    const sc_status e = wait_report(vol, s);
    if (e != SC_OK) return e;
    nb = reported_blocks(vol);
    return (sc_status)st->report->err;
}

// Streams in the host-held blocks among the n of `want` (host keys),
// appending them to the pool's nb blocks.  Enqueues on `s`.
static sc_status stream_in_keys(sc_volume* vol, const uint64_t* want, size_t n, int64_t nb, hipStream_t s,
                                size_t& moved)
{
    StreamStore* st = vol->stream;
    moved = 0;
    if (st->where.empty()) return SC_OK;
    if (!grow_items(st->in, st->in_cap, std::min(n, st->where.size()))) return SC_ENOMEM;
    StreamMoves moves;
    for (size_t i = 0; i < n; ++i) {
        auto it = st->where.find(want[i]);
        if (it == st->where.end()) continue;
        const size_t j = moves.recs.size();
        st->in[j] = StreamItem{it->first, moves.add(st, it->second), -1, -1};
    }
    const size_t m = moves.recs.size();
    if (m == 0) return SC_OK;
    if (nb + (int64_t)m > vol->p.max_blocks) {
        // the work cannot run with every block it may touch: the field is
        // left unspecified, as for any full pool
        set_error_kernel<<<1, 1, 0, s>>>(vol->dev.err, SC_EPOOLFULL);
        return SC_EPOOLFULL;
    }
    const sc_status e = moves.run(st, false, s, [&](size_t a, size_t b) {
        stream_in_kernel<<<(unsigned)(b - a), 256, 0, s>>>(vol->dev, st->in + a, (int64_t)(b - a), nb + (int64_t)a);
    });
    if (e != SC_OK) return e;
    if (hipGetLastError() != hipSuccess || hipEventRecord(st->done, s) != hipSuccess) return SC_EDEVICE;
    // later uses of the records are enqueued behind the kernel
    for (size_t i = 0; i < m; ++i) {
        st->free_recs.push_back(moves.recs[i]);
        st->where.erase(st->in[i].key);
    }
    st->blocks_in += (int64_t)m;
    moved = m;
    return SC_OK;
}

// Moves the device blocks (keys in slot order) whose index `out` marks to the
// host store and compacts the pool: the live blocks above the new count fill
// the holes below it (disjoint ranges), the freed slots are cleared to the
// empty state, and the hash table is rebuilt.  Enqueues on `s`.
static sc_status evict(sc_volume* vol, const uint64_t* keys, const std::vector<char>& out, hipStream_t s)
{
    StreamStore* st = vol->stream;
    const int64_t nb = (int64_t)out.size();
    const size_t e = (size_t)std::count(out.begin(), out.end(), (char)1);
    if (e == 0) return SC_OK;
    const int64_t live = nb - (int64_t)e;
    if (!grow_items(st->out, st->out_cap, e) || !reserve_recs(st, e)) return SC_ENOMEM;
    StreamMoves moves;
    moves.recs.reserve(e);
    int64_t mover = live;
    for (int64_t i = 0; i < nb; ++i) {
        if (!out[i]) continue;
        int64_t from = -1;
        if (i < live) {  // as many holes below the new count as live blocks above it
            while (out[mover]) ++mover;
            from = mover++;
        }
        const size_t k = moves.recs.size();
        st->out[k] = StreamItem{keys[i], moves.add(st, take_rec(st)), (int32_t)i, (int32_t)from};
    }
    // (the hash table is emptied by every range)
    const sc_status r = moves.run(st, true, s, [&](size_t a, size_t b) {
        stream_out_kernel<<<(unsigned)std::max<size_t>(b - a, (size_t)vol->n_cu * 2), 256, 0, s>>>(
            vol->dev, st->out + a, (int64_t)(b - a));
    });
    if (r != SC_OK) return r;
    hash_rebuild_kernel<<<vol->n_cu * 4, 256, 0, s>>>(vol->dev, live);
    if (hipGetLastError() != hipSuccess || hipEventRecord(st->done, s) != hipSuccess) return SC_EDEVICE;
    for (size_t i = 0; i < e; ++i) st->where[st->out[i].key] = moves.recs[i];
    st->blocks_out += (int64_t)e;
    return SC_OK;
}

// Before a voxel pass in streaming mode: the candidate keys of the work are
// in d_all (ncand of them), those without a device slot in h_keys, and the
// report is in.  When the pool cannot take all of the latter, resident
// blocks that are not candidates are streamed out, farthest from the
// candidates' mean first, until it can (with an eighth of the pool to
// spare when possible).  Then the host-held ones are streamed in.  `moved`
// tells whether any pool slot changed.
static sc_status prepare_work(sc_volume* vol, hipStream_t s, uint32_t ncand, bool& moved)
{
    StreamStore* st = vol->stream;
    moved = false;
    const uint32_t n = st->report->n_req;
    if (n > st->keys_cap) return SC_ENOMEM;
    if (n == 0) return SC_OK;
    sc_status e = (sc_status)st->report->err;
    if (e != SC_OK) return e;
    int64_t nb = reported_blocks(vol);
    std::vector<uint64_t> kept;  // the requests, where h_keys is used again
    const uint64_t* want = st->h_keys;
    const int64_t cap = vol->p.max_blocks;
    if (nb + (int64_t)n > cap) {
        kept.assign(want, want + n);
        want = kept.data();
        std::vector<uint64_t> cand(ncand);
        e = d2h(cand.data(), st->d_all, sizeof(uint64_t) * ncand, s);
        if (e != SC_OK) return e;
        std::unordered_map<uint64_t, char> is_cand;
        is_cand.reserve(ncand * 2);
        double mx = 0.0, my = 0.0, mz = 0.0;
        for (uint64_t k : cand) {
            is_cand[k] = 1;
            int bx, by, bz;
            unpack_key(k, bx, by, bz);
            mx += bx;
            my += by;
            mz += bz;
        }
        if (ncand) {
            mx /= ncand;
            my /= ncand;
            mz /= ncand;
        }
        e = device_keys(vol, s, nb);
        if (e != SC_OK) return e;
        const uint64_t* keys = st->h_keys;
        std::vector<std::pair<double, size_t>> far;
        for (size_t i = 0; i < (size_t)nb; ++i) {
            if (is_cand.count(keys[i])) continue;
            int bx, by, bz;
            unpack_key(keys[i], bx, by, bz);
            const double dx = bx - mx, dy = by - my, dz = bz - mz;
            far.emplace_back(-(dx * dx + dy * dy + dz * dz), i);
        }
        std::sort(far.begin(), far.end());
        // blocks that may stay: room for the requests, and an eighth of the
        // pool to spare when there is room for that too
        const int64_t room = cap - (int64_t)n;
        const int64_t keep = (room - cap / 8 >= 0) ? room - cap / 8 : room;
        const int64_t need = std::max<int64_t>(0, std::min<int64_t>(nb - keep, (int64_t)far.size()));
        std::vector<char> out((size_t)nb, 0);
        for (int64_t i = 0; i < need; ++i) out[far[(size_t)i].second] = 1;
        e = evict(vol, keys, out, s);
        if (e != SC_OK) return e;
        moved = need > 0;
        nb -= need;
        if (nb + (int64_t)n > cap) {
            set_error_kernel<<<1, 1, 0, s>>>(vol->dev.err, SC_EPOOLFULL);
            return SC_EPOOLFULL;
        }
    }
    size_t in = 0;
    e = stream_in_keys(vol, want, n, nb, s, in);
    if (e != SC_OK) return e;
    moved = moved || in > 0;
    return SC_OK;
}

// A streaming step that failed after the candidates were generated leaves
// the operation undone and its candidate entries in place: the failure is
// made sticky, so the volume is reset before further use.
static sc_status fail_sticky(sc_volume* vol, sc_status e, hipStream_t s)
{
    if (e != SC_OK && e != SC_EPOOLFULL) set_error_kernel<<<1, 1, 0, s>>>(vol->dev.err, e);
    return e;
}

static sc_status stream_in_batch_impl(sc_volume* vol, hipStream_t s);
static sc_status stream_in_plain_impl(sc_volume* vol, int parity, hipStream_t s);

sc_status stream_in_batch(sc_volume* vol, hipStream_t s)
{
    return streaming(vol) ? fail_sticky(vol, stream_in_batch_impl(vol, s), s) : SC_OK;
}

sc_status stream_in_plain(sc_volume* vol, int parity, hipStream_t s)
{
    return streaming(vol) ? fail_sticky(vol, stream_in_plain_impl(vol, parity, s), s) : SC_OK;
}

// Batched path, after the candidate stage: room for every candidate block,
// the host-held ones streamed in, and the candidates' pool slots refreshed.
static sc_status stream_in_batch_impl(sc_volume* vol, hipStream_t s)
{
    StreamStore* st = vol->stream;
    if (!grow_keys(st, vol->cand_buckets)) return SC_ENOMEM;
    stream_req_batch_kernel<<<vol->n_cu * 4, 256, 0, s>>>(vol->cand, st->d_all, st->h_keys, st->d_req,
                                                          (uint32_t)st->keys_cap);
    stream_report_kernel<<<1, 1, 0, s>>>(vol->cand.counters + 4, st->d_req, vol->dev, st->report);
    sc_status e = wait_report(vol, s);
    if (e != SC_OK) return e;
    bool moved = false;
    e = prepare_work(vol, s, std::min<uint32_t>(st->report->n_cand, (uint32_t)st->keys_cap), moved);
    if (e != SC_OK) return e;
    if (moved) sslot_refresh_kernel<<<vol->n_cu * 4, 256, 0, s>>>(vol->cand, vol->dev);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

// Plain path, after the candidate list of one operation is built (the
// update kernel looks its blocks up itself).
static sc_status stream_in_plain_impl(sc_volume* vol, int parity, hipStream_t s)
{
    StreamStore* st = vol->stream;
    if (!grow_keys(st, vol->cand.cap)) return SC_ENOMEM;
    stream_req_plain_kernel<<<vol->n_cu * 4, 256, 0, s>>>(vol->cand, vol->dev, parity, st->d_all, st->h_keys,
                                                          st->d_req, (uint32_t)st->keys_cap);
    stream_report_kernel<<<1, 1, 0, s>>>(vol->cand.counters + parity, st->d_req, vol->dev, st->report);
    const sc_status e = wait_report(vol, s);
    if (e != SC_OK) return e;
    bool moved = false;
    return prepare_work(
        vol, s, std::min<uint32_t>(std::min<uint32_t>(st->report->n_cand, vol->cand.cap), (uint32_t)st->keys_cap),
        moved);
}

// Host side of a reset, which only enqueues: it waits for nothing and frees
// nothing (a kernel may still read the records).  No record is in use until
// the next wait.
void stream_clear(sc_volume* vol)
{
    StreamStore* st = vol->stream;
    if (!st) return;
    st->where.clear();
    st->free_recs.clear();
    st->cur = st->pos = 0;
    st->surplus = true;
}

void stream_destroy(sc_volume* vol)
{
    StreamStore* st = vol->stream;
    if (!st) return;
    drop_chunks(st, 0);
    if (st->stage) (void)hipHostFree(st->stage);
    if (st->in) (void)hipHostFree(st->in);
    if (st->out) (void)hipHostFree(st->out);
    if (st->report) (void)hipHostFree(st->report);
    if (st->h_keys) (void)hipHostFree(st->h_keys);
    (void)hipFree(st->d_all);
    (void)hipFree(st->d_req);
    if (st->done) (void)hipEventDestroy(st->done);
    delete st;
    vol->stream = nullptr;
}

}  // namespace sc

using namespace sc;

extern "C" {

sc_status sc_stream_enable(sc_volume* vol, int32_t enable)
{
    if (!vol) return SC_EINVAL;
    if (!vol->stream) {
        vol->stream = new (std::nothrow) StreamStore();
        if (!vol->stream) return SC_ENOMEM;
        StreamStore* st = vol->stream;
        st->block_bytes = sizeof(float) * (size_t)vol->dev.stride;
        if (!device_alloc(&st->d_req, sizeof(uint32_t)) ||
            hipHostMalloc((void**)&st->report, sizeof(StreamReport), hipHostMallocCoherent) != hipSuccess ||
            hipHostMalloc((void**)&st->stage, kStageBlocks * st->block_bytes, hipHostMallocCoherent) != hipSuccess ||
            hipEventCreateWithFlags(&st->done, hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            stream_destroy(vol);
            return SC_ENOMEM;
        }
        // operations may come on any stream
        fill_u32(st->d_req, 0u, 1, 0);
        if (hipStreamSynchronize(0) != hipSuccess) {
            stream_destroy(vol);
            return SC_EDEVICE;
        }
    }
    if (!enable && !vol->stream->where.empty()) return SC_EINVAL;  // blocks still on the host
    vol->stream->enabled = enable != 0;
    return SC_OK;
}

sc_status sc_stream_pinned_limit(sc_volume* vol, int64_t bytes)
{
    if (!vol || !vol->stream || bytes < 0) return SC_EINVAL;
    vol->stream->pinned_limit = (size_t)bytes;
    return SC_OK;
}

sc_status sc_stream_out(sc_volume* vol, const double* center, double radius, void* stream)
{
    if (!vol || !center || !(radius >= 0.0)) return SC_EINVAL;
    if (!streaming(vol)) return SC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    int64_t nb = 0;
    sc_status e = device_keys(vol, s, nb);
    if (e != SC_OK) return e;
    const uint64_t* keys = vol->stream->h_keys;
    // block centre: voxel centres s * n for n in [8 b, 8 b + 7], so 8 b + 3.5
    const double vs = (double)vol->p.voxel_size, r2 = radius * radius;
    std::vector<char> out((size_t)nb, 0);
    for (size_t i = 0; i < out.size(); ++i) {
        int bx, by, bz;
        unpack_key(keys[i], bx, by, bz);
        const double dx = vs * (8.0 * bx + 3.5) - center[0];
        const double dy = vs * (8.0 * by + 3.5) - center[1];
        const double dz = vs * (8.0 * bz + 3.5) - center[2];
        out[i] = (dx * dx + dy * dy + dz * dz > r2) ? 1 : 0;
    }
    e = evict(vol, keys, out, s);
    if (e != SC_OK) return e;
    return hipStreamSynchronize(s) == hipSuccess ? SC_OK : SC_EDEVICE;
}

sc_status sc_stream_in_all(sc_volume* vol, void* stream)
{
    if (!vol) return SC_EINVAL;
    if (!vol->stream || vol->stream->where.empty()) return SC_OK;
    StreamStore* st = vol->stream;
    hipStream_t s = (hipStream_t)stream;
    std::vector<uint64_t> want;
    want.reserve(st->where.size());
    for (const auto& kv : st->where) want.push_back(kv.first);
    stream_keys_kernel<<<1, 1, 0, s>>>(vol->dev, nullptr, 0u, st->report);
    sc_status e = wait_report(vol, s);
    if (e == SC_OK) e = (sc_status)st->report->err;
    if (e != SC_OK) return e;
    size_t in = 0;
    e = stream_in_keys(vol, want.data(), want.size(), reported_blocks(vol), s, in);
    if (e != SC_OK) return e;
    return hipStreamSynchronize(s) == hipSuccess ? SC_OK : SC_EDEVICE;
}

sc_status sc_stream_export(sc_volume* vol, int32_t* block_xyz, float* D, float* W, void* C, int64_t cap,
                           int64_t* n_out)
{
    if (!vol || cap < 0) return SC_EINVAL;
    const StreamStore* st = vol->stream;
    const int64_t n = st ? (int64_t)st->where.size() : 0;
    if (n_out) *n_out = n;
    if (!st) return SC_OK;
    if (hipEventSynchronize(st->done) != hipSuccess) return SC_EDEVICE;
    const bool rgba = vol->p.color_mode == SC_COLOR_RGBA8;
    int64_t b = 0;
    for (const auto& kv : st->where) {
        if (b >= cap) break;
        const float* rec = reinterpret_cast<const float*>(kv.second.p);
        int x, y, z;
        unpack_key(kv.first, x, y, z);
        if (block_xyz) {
            block_xyz[3 * b] = x;
            block_xyz[3 * b + 1] = y;
            block_xyz[3 * b + 2] = z;
        }
        const double* Dd = reinterpret_cast<const double*>(rec);
        for (int i = 0; i < kBlockVox; ++i) {
            if (D) D[b * kBlockVox + i] = (float)Dd[i];
            if (W) W[b * kBlockVox + i] = rec[kPoolW + i];
        }
        if (C) {
            if (rgba) {
                memcpy(reinterpret_cast<uint32_t*>(C) + b * kBlockVox, rec + kPoolC, sizeof(uint32_t) * kBlockVox);
            } else {
                const double* Cd = reinterpret_cast<const double*>(rec + kPoolC);
                float* Cf = reinterpret_cast<float*>(C) + b * 3 * kBlockVox;
                for (int i = 0; i < 3 * kBlockVox; ++i) Cf[i] = (float)Cd[i];
            }
        }
        ++b;
    }
    return SC_OK;
}

sc_status sc_stream_stats(sc_volume* vol, void* stream, int64_t* stats)
{
    if (!vol || !stats) return SC_EINVAL;
    int64_t nb = 0;
    const sc_status e = sc_volume_query(vol, stream, &nb, nullptr);
    if (e != SC_OK) return e;
    const StreamStore* st = vol->stream;
    const int64_t bb = (int64_t)sizeof(float) * vol->dev.stride;
    stats[0] = nb;
    stats[1] = st ? (int64_t)st->where.size() : 0;
    stats[2] = st ? st->blocks_out : 0;
    stats[3] = st ? st->blocks_in : 0;
    stats[4] = st ? st->blocks_out * bb : 0;
    stats[5] = st ? st->blocks_in * bb : 0;
    return SC_OK;
}

}  // extern "C"
