// Voxel-hashed TSDF volume (Sec. 3, "SDF volume"): lifecycle, block
// allocation, and the plain per-keyframe integration (running weighted
// average) and de-integration (Sec. 4.3, Eq. 2).
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <unordered_map>
#include <vector>

#include "common.hpp"
#include "kernels.hpp"
#include "internal.hpp"

namespace sc {

// ---------------------------------------------------------------------------
// small kernels
// ---------------------------------------------------------------------------

__global__ void fill_u64_kernel(uint64_t* p, uint64_t v, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

__global__ void fill_u32_kernel(uint32_t* p, uint32_t v, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

void fill_u64(uint64_t* p, uint64_t v, size_t n, hipStream_t s)
{
    if (n == 0) return;
    const int grid = (int)std::min<size_t>((n + 255) / 256, 8192);
    fill_u64_kernel<<<grid, 256, 0, s>>>(p, v, n);
}

void fill_u32(uint32_t* p, uint32_t v, size_t n, hipStream_t s)
{
    if (n == 0) return;
    const int grid = (int)std::min<size_t>((n + 255) / 256, 8192);
    fill_u32_kernel<<<grid, 256, 0, s>>>(p, v, n);
}

// Stores `v` over the 32-bit words of [p, p + bytes) (bytes a multiple of 4,
// p 16-byte aligned), 16 bytes a store.
__device__ inline void fill_words(void* p, size_t bytes, uint32_t v)
{
    const size_t i0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
    const size_t n16 = bytes / 16;
    uint4* q = static_cast<uint4*>(p);
    for (size_t i = i0; i < n16; i += step) q[i] = make_uint4(v, v, v, v);
    uint32_t* w = static_cast<uint32_t*>(p);
    for (size_t i = 4 * n16 + i0; i < bytes / 4; i += step) w[i] = v;
}

// Empties a volume in one launch: the block hash, the pool and the
// per-batch counters.  Slots beyond the allocated blocks have never been
// written (eviction clears what it frees), so only the allocated ones are
// cleared unless `full`, and the candidate table, which every pass leaves
// empty, only when a device error or the host (`cand_dirty`) says that one
// did not.  The bound is the bytes stored: 28,700 of 524,288 RGBA8 blocks and
// a 2^21-bucket hash, 261 MB instead of 4.5 GB: reset and batched integration
// of 40 keyframes 1.91 -> 1.12 ms, against fourteen fills of everything.
// The counters that this kernel reads are cleared by
// reset_counts_kernel after it.
__global__ __launch_bounds__(256) void reset_kernel(VolDev v, CandDev c, double* adj_acc, bool full, bool cand_dirty)
{
    const uint32_t nb = full ? (uint32_t)v.max_blocks : min(*v.n_blocks, (uint32_t)v.max_blocks);
    const size_t buckets = (size_t)v.bucket_mask + 1, cand = (size_t)c.mask_bits + 1;
    fill_words(v.pool, sizeof(float) * (size_t)v.stride * nb, 0u);
    fill_words(v.keys, sizeof(uint64_t) * buckets, ~0u);
    fill_words(v.vals, sizeof(int32_t) * buckets, ~0u);
    if (full || cand_dirty || *v.err != 0) {
        fill_words(c.keys, sizeof(uint64_t) * cand, ~0u);
        fill_words(c.mask, sizeof(uint64_t) * cand * c.words, 0u);
    }
    fill_words(c.counters, sizeof(uint32_t) * 64, 0u);
    fill_words(c.bins, sizeof(uint32_t) * 2 * (kMaxBatchOps + 2), 0u);
    fill_words(c.cursors, sizeof(uint32_t) * 2 * kCursorSet, 0u);
    fill_words(c.big, sizeof(uint32_t), 0u);
    fill_words(c.stats, sizeof(unsigned long long) * 4 * kStatSlots * kStatStride, 0u);
    fill_words(adj_acc, sizeof(double) * 3 * kAdjChunk, 0u);
}
static_assert(kKeyEmpty == ~0ull, "reset_kernel stores the empty key as two words of ones");

__global__ void reset_counts_kernel(VolDev v)
{
    if (threadIdx.x < 16) {
        v.n_blocks[threadIdx.x] = 0u;
        v.err[threadIdx.x] = 0;
    }
}

// ---------------------------------------------------------------------------
// hash_alloc: wavefront ballot deduplication (one round per distinct key),
// CAS insert, LDS-staged queue of new blocks and one pool reservation per
// workgroup
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void hash_alloc_kernel(VolDev v, const int32_t* xyz, int64_t n)
{
    __shared__ uint32_t q_bucket[256];
    __shared__ uint32_t q_n;
    __shared__ uint32_t q_base;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    if (tid == 0) q_n = 0;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + tid;
    const bool have = i < n;
    int bx = 0, by = 0, bz = 0;
    uint64_t key = kKeyEmpty;
    if (have) {
        bx = xyz[3 * i];
        by = xyz[3 * i + 1];
        bz = xyz[3 * i + 2];
        key = pack_key(bx, by, bz);
    }
    __syncthreads();
    // one leader per distinct key within each wavefront, by ballot: the
    // lowest lane still undecided takes its key, every lane holding that key
    // is decided; one round per distinct key of the wavefront
    bool leader = false;
    uint64_t todo = __ballot(have);
    while (todo) {
        const int l = __ffsll((unsigned long long)todo) - 1;
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)key, l);
        const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(key >> 32), l);
        const uint64_t k = ((uint64_t)hi << 32) | lo;
        leader = leader || lane == l;
        todo &= ~__ballot(key == k);
    }
    if (leader) {
        uint32_t h = hash_block(bx, by, bz) & v.bucket_mask;
        bool done = false;
        for (uint32_t probe = 0; probe <= v.bucket_mask; ++probe) {
            const uint64_t old = atomicCAS((unsigned long long*)(v.keys + h), (unsigned long long)kKeyEmpty,
                                           (unsigned long long)key);
            if (old == kKeyEmpty) {
                const uint32_t q = atomicAdd(&q_n, 1u);
                q_bucket[q] = h;
                done = true;
                break;
            }
            if (old == key) {
                done = true;
                break;
            }
            h = (h + 1) & v.bucket_mask;
        }
        if (!done) set_error(v.err, SC_EHASHFULL);
    }
    __syncthreads();
    if (tid == 0) q_base = q_n ? atomicAdd(v.n_blocks, q_n) : 0u;
    __syncthreads();
    for (uint32_t j = tid; j < q_n; j += blockDim.x) {
        const uint32_t slot = q_base + j;
        const uint32_t h = q_bucket[j];
        if (slot >= (uint32_t)v.max_blocks) {
            v.vals[h] = -1;
            set_error(v.err, SC_EPOOLFULL);
        } else {
            v.slot_keys[slot] = v.keys[h];
            v.vals[h] = (int)slot;
        }
    }
}

__global__ void hash_lookup_kernel(VolDev v, const int32_t* xyz, int64_t n, int32_t* slots)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int bx = xyz[3 * i], by = xyz[3 * i + 1], bz = xyz[3 * i + 2];
    slots[i] = vol_find(v, pack_key(bx, by, bz), bx, by, bz);
}

// ---------------------------------------------------------------------------
// plain path: one keyframe operation
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void cand_plain_kernel(OpDesc op, VolDev v, CandDev cd, int parity)
{
    __shared__ uint64_t lds[CandCfg<kTilePlain, kCellPlain>::lds_set];
    __shared__ uint16_t idx[CandCfg<kTilePlain, kCellPlain>::lds_set];
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        cd.counters[1 - parity] = 0u;
    }
    // the integration's record starts empty
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kRecShards && op.rec_mode == 1)
        record_clear(op, (int)threadIdx.x);
    cand_tile<kTilePlain, kCellPlain>(op, v, cd, cd.counters + parity, blockIdx.x, blockIdx.y, -1, lds, idx);
}

// Applies one operation to its candidate blocks, one wavefront a block, eight
// voxels a lane (lane = x + 8 y, z in registers), and clears the blocks'
// candidate entries.  Workgroup wavefronts take the list's entries in a fixed
// stride: a keyframe proposes a few thousand blocks, about one a wavefront,
// and a queue counter that every wavefront reads once more to find the list
// empty is served one wavefront at a time.  For the same reason the blocks of
// a touched-block record are kept per wavefront and appended with one atomic
// per workgroup.
// Bound: the latency of a block's chain of loads (list, key, then slot and
// keyframe samples together, then the voxels four slices at a time: all eight
// at once take 169 registers, or spill).  640x480 keyframe: 1 cm voxels, in an
// online session, 79 -> 27 us; 5 mm voxels 86 -> 24 us.
constexpr int kPlainRec = 16;  // recorded blocks a wavefront holds; appended by itself when there are more

template <int CM, bool kPacked>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void update_plain_kernel(OpDesc op, VolDev v, CandDev cd, int parity)
{
    __shared__ uint64_t rec[4][kPlainRec];
    __shared__ uint32_t rec_n[4];
    __shared__ uint32_t rec_base;
    const int lane = threadIdx.x & 63;
    const int wave = (int)bcast(threadIdx.x >> 6);
    const uint32_t n = min(cd.counters[parity], cd.cap);
    const uint32_t n_workers = gridDim.x * 4u;
    const uint32_t shard = blockIdx.x % kRecShards;
    uint32_t held = 0u;  // recorded blocks not yet appended
    bool bad = false;
    for (uint32_t i = blockIdx.x * 4u + (uint32_t)wave; i < n; i += n_workers) {
        const uint32_t h = bcast(cd.list[i]);
        const uint64_t key = bcast64(cd.keys[h]);
        int bx, by, bz;
        unpack_key(key, bx, by, bz);
        RingGeom g;
        ring_geom(op, v, bx, by, bz, lane, g);
        RingFetch<CM> f[2];
        ring_fetch<CM, kPacked>(op, g, 0, f[0]);
        ring_fetch<CM, kPacked>(op, g, 4, f[1]);
        int slot = (int)bcast((uint32_t)vol_find(v, key, bx, by, bz));
        float w[8];
        bool t[8];
        ring_decide<CM, kPacked>(f[0], v.mu, w, t);
        ring_decide<CM, kPacked>(f[1], v.mu, w + 4, t + 4);
        bool any = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) any = any || t[j];
        cd.keys[h] = kKeyEmpty;
        if (__ballot(any) == 0ull) continue;
        if (op.rec_mode == 1) {
            if (held == (uint32_t)kPlainRec) {
                wave_lds_sync();
                uint32_t at = 0u;
                if (lane == 0) at = atomicAdd(op.rec_count + shard * kRecCountStride, held);
                at = bcast(at);
                if ((uint32_t)lane < held) record_put(op, shard, at + (uint32_t)lane, rec[wave][lane]);
                held = 0u;
            }
            rec[wave][held++] = key;  // every lane, the same value
        }
        if (slot < 0 && op.sign > 0) slot = vol_insert_wave(v, key, bx, by, bz, lane);
        if (slot < 0) {
            if (op.sign < 0) set_error(v.err, SC_ENOTALLOC);
            continue;
        }
        float* blk = v.pool + (size_t)slot * v.stride;
        double* Dp = reinterpret_cast<double*>(blk);
        float* Wp = blk + kPoolW;
        const double bz64 = (g.qz + (double)(lane & 7) * op.az[0]) + (double)(lane >> 3) * op.az[1];
        if (CM == SC_COLOR_RGBA8) {
            uint32_t* Cp = reinterpret_cast<uint32_t*>(blk + kPoolC);
#pragma unroll
            for (int p = 0; p < 8; p += 4) {
                double D[4];
                float W[4];
                uint32_t C[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // a lane without a touched voxel reads the block's first: no branch between the loads
                    const int x = t[p + q] ? lane + 64 * (p + q) : 0;
                    D[q] = Dp[x];
                    W[q] = Wp[x];
                    C[q] = Cp[x];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (!t[p + q]) continue;
                    const int x = lane + 64 * (p + q);
                    bad |= !update_rgba8_fast(D[q], W[q], C[q],
                                              distance(f[p / 4].z[q], bz64 + (double)(p + q) * op.az[2]), w[p + q],
                                              f[p / 4].c[q], op.sign);
                    Dp[x] = D[q];
                    Wp[x] = W[q];
                    Cp[x] = C[q];
                }
            }
        } else {
            double* Cd = reinterpret_cast<double*>(blk + kPoolC);
            const float* col = reinterpret_cast<const float*>(op.color);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (!t[j]) continue;
                const int x = lane + 64 * j;
                const RingFetch<CM>& fj = f[j >> 2];
                const float* cp = col + 3 * (size_t)fj.pix[j & 3];
                double C[3] = {Cd[x], Cd[512 + x], Cd[1024 + x]};
                const float c[3] = {cp[0], cp[1], cp[2]};
                double D = Dp[x];
                float W = Wp[x];
                bad |= !update_f32(D, W, C, distance(fj.z[j & 3], bz64 + (double)j * op.az[2]), w[j], c, op.sign);
                Dp[x] = D;
                Wp[x] = W;
                Cd[x] = C[0];
                Cd[512 + x] = C[1];
                Cd[1024 + x] = C[2];
            }
        }
    }
    if (__ballot(bad) != 0) set_error(v.err, SC_EWEIGHT);
    if (op.rec_mode != 1) return;
    if (lane == 0) rec_n[wave] = held;
    __syncthreads();
    uint32_t sum = 0u, before = 0u;
    for (int q = 0; q < 4; ++q) {
        before += q < wave ? rec_n[q] : 0u;
        sum += rec_n[q];
    }
    if (sum == 0u) return;
    if (threadIdx.x == 0) rec_base = atomicAdd(op.rec_count + shard * kRecCountStride, sum);
    __syncthreads();
    if ((uint32_t)lane < held) record_put(op, shard, rec_base + before + (uint32_t)lane, rec[wave][lane]);
}

// Writes imported block records into their pool slots (D widened to FP64;
// FP32 colour widened to the FP64 planes).
__global__ void import_kernel(VolDev v, const int32_t* __restrict__ slots, int64_t n, const float* __restrict__ D,
                              const float* __restrict__ W, const void* __restrict__ C)
{
    const int64_t b = blockIdx.x;
    if (b >= n) return;
    const int slot = slots[b];
    if (slot < 0) return;
    float* blk = v.pool + (size_t)slot * v.stride;
    for (int i = threadIdx.x; i < kBlockVox; i += blockDim.x) {
        const size_t g = (size_t)b * kBlockVox + i;
        reinterpret_cast<double*>(blk)[i] = D ? (double)D[g] : 0.0;
        blk[kPoolW + i] = W ? W[g] : 0.0f;
        if (v.color_mode == SC_COLOR_RGBA8) {
            reinterpret_cast<uint32_t*>(blk + kPoolC)[i] = C ? reinterpret_cast<const uint32_t*>(C)[g] : 0u;
        } else {
            const float* Cf = reinterpret_cast<const float*>(C) + (size_t)b * 3 * kBlockVox;
            double* Cd = reinterpret_cast<double*>(blk + kPoolC);
            Cd[i] = C ? (double)Cf[i] : 0.0;
            Cd[512 + i] = C ? (double)Cf[512 + i] : 0.0;
            Cd[1024 + i] = C ? (double)Cf[1024 + i] : 0.0;
        }
    }
}

// The first min(allocated, cap) blocks.  The number is read here, so that the
// host waits once, for the blocks and their number together: an update of 4
// operations with its export (4,500 blocks) took 178 us with the number asked
// for first, now 154.  Bound by memory: the benchmark's volume in 486 us (480
// with a workgroup a block).
__global__ __launch_bounds__(256) void export_kernel(VolDev v, int64_t cap, int32_t* xyz, float* D, float* W, void* C)
{
    const int64_t n = min(min((int64_t)*v.n_blocks, (int64_t)v.max_blocks), cap);
    for (int64_t b = blockIdx.x; b < n; b += gridDim.x) {
        const float* blk = v.pool + (size_t)b * v.stride;
        for (int i = threadIdx.x; i < kBlockVox; i += blockDim.x) {
            if (D) D[b * kBlockVox + i] = (float)reinterpret_cast<const double*>(blk)[i];
            if (W) W[b * kBlockVox + i] = blk[kPoolW + i];
            if (C) {
                if (v.color_mode == SC_COLOR_RGBA8) {
                    reinterpret_cast<uint32_t*>(C)[b * kBlockVox + i] =
                        reinterpret_cast<const uint32_t*>(blk + kPoolC)[i];
                } else {
                    const double* Cd = reinterpret_cast<const double*>(blk + kPoolC);
                    float* Cf = reinterpret_cast<float*>(C) + b * 3 * kBlockVox;
                    Cf[i] = (float)Cd[i];
                    Cf[512 + i] = (float)Cd[512 + i];
                    Cf[1024 + i] = (float)Cd[1024 + i];
                }
            }
        }
        if (xyz && threadIdx.x == 0) {
            int x, y, z;
            unpack_key(v.slot_keys[b], x, y, z);
            xyz[3 * b] = x;
            xyz[3 * b + 1] = y;
            xyz[3 * b + 2] = z;
        }
    }
}

// Packed record of a pixel: the quantised weight, and the depth only where
// that weight is positive (-inf elsewhere, which fails every band test); and
// the depth range {zmin, zmax} of the valid pixels (positive quantised weight,
// 0 < depth < 1e30) of each 4 x 4 cell, {+inf, -inf} without one: the
// candidate stage's per-cell test without reading the pixels.
// A wavefront takes 64 columns of one row of cells, a lane a column of four
// pixels (its loads issue together), and four lanes share a cell.  Bound: the
// launch and one round of loads; records and cells in two kernels, the cells
// reading every pixel again, took 5.1 + 5.5 us at 640x480, now 6.0 (traced).
__global__ __launch_bounds__(256) void pack_kernel(const float* __restrict__ depth, const float* __restrict__ weight,
                                                   const uint32_t* __restrict__ color, uint4* out, float2* cells,
                                                   int width, int height, int cells_w, int64_t n_items)
{
    const int lane = threadIdx.x & 63;
    const int strips = (width + 63) / 64;
    const int64_t item = blockIdx.x * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6);
    if (item >= n_items) return;
    const int cy = (int)(item / strips), u = (int)(item - (int64_t)cy * strips) * 64 + lane;
    float z[4], w[4];
    uint32_t c[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int y = 4 * cy + r;
        const bool in = u < width && y < height;
        const int64_t i = in ? (int64_t)y * width + u : 0;
        z[r] = depth[i];
        w[r] = in ? weight[i] : 0.0f;
        c[r] = color[i];
    }
    float zmin = __builtin_inff(), zmax = -__builtin_inff();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int y = 4 * cy + r;
        const float q = qweight(w[r]);
        if (u < width && y < height)
            out[(int64_t)y * width + u] =
                make_uint4(__float_as_uint(q > 0.0f ? z[r] : -__builtin_inff()), __float_as_uint(q), c[r], 0u);
        if (q > 0.0f && z[r] > 0.0f && z[r] < 1.0e30f) {
            zmin = fminf(zmin, z[r]);
            zmax = fmaxf(zmax, z[r]);
        }
    }
#pragma unroll
    for (int o = 1; o < 4; o <<= 1) {
        zmin = fminf(zmin, __shfl_xor(zmin, o));
        zmax = fmaxf(zmax, __shfl_xor(zmax, o));
    }
    if ((lane & 3) == 0 && u < width) cells[(int64_t)cy * cells_w + (u >> 2)] = make_float2(zmin, zmax);
}

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------

void make_op(const sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* in, const sc_pose* T, int sign,
             int kf_index, OpDesc* op)
{
    memset(op, 0, sizeof(*op));
    op->depth = kf->depth;
    op->weight = kf->weight;
    op->color = kf->color;
    op->packed = (vol->p.color_mode == SC_COLOR_RGBA8) ? reinterpret_cast<const uint4*>(kf->packed) : nullptr;
    // the cell depth ranges follow the width x height records
    op->cells = op->packed ? reinterpret_cast<const float2*>(op->packed + (size_t)in->width * in->height) : nullptr;
    op->width = in->width;
    op->height = in->height;
    op->fx = in->fx;
    op->fy = in->fy;
    op->cx = in->cx;
    op->cy = in->cy;
    memcpy(op->R, T->R, sizeof(op->R));
    memcpy(op->t, T->t, sizeof(op->t));
    const double s = (double)vol->p.voxel_size;
    for (int c = 0; c < 3; ++c) {
        for (int r = 0; r < 3; ++r) op->a[c][r] = (float)(s * T->R[3 * c + r]);
        op->az[c] = s * T->R[3 * c + 2];
    }
    for (int k = 0; k < 8; ++k)
        for (int r = 0; r < 3; ++r) op->za[k][r] = (float)k * op->a[2][r];  // one FP32 rounding, as on the device
    op->wl = (float)(in->width - 1);
    op->hl = (float)(in->height - 1);
    op->wf = (float)in->width;
    // one extra 2^-21 covers the rounding of the bound itself to FP32
    op->kin_u = (float)(0.5 - (2.0 + fabs((double)in->cx)) * 0x1p-21);
    op->kin_v = (float)(0.5 - (2.0 + fabs((double)in->cy)) * 0x1p-21);
    op->sign = sign;
    op->kf = kf_index;
}

// Host staging of operation descriptors, double-buffered: a buffer is
// refilled only after the copy that last read it has run, so the host can
// prepare the next chunk while the device still works on the previous one.
OpDesc* stage_begin(sc_volume* vol)
{
    if (hipEventSynchronize(vol->staged[vol->stage]) != hipSuccess) return nullptr;
    return vol->h_ops + (size_t)vol->stage * vol->p.max_batch_ops;
}

BatchHdr* stage_hdr(sc_volume* vol) { return vol->h_hdr + vol->stage; }

// Records the current buffer's copies on `s` and switches buffers.
sc_status stage_end(sc_volume* vol, hipStream_t s)
{
    if (hipEventRecord(vol->staged[vol->stage], s) != hipSuccess) return SC_EDEVICE;
    vol->stage ^= 1;
    return SC_OK;
}

static bool intr_ok(const sc_intrinsics* in)
{
    return in && in->width > 0 && in->height > 0 && in->fx > 0.0f && in->fy > 0.0f && in->width <= 16384 &&
           in->height <= 16384;
}

bool keyframe_ok(const sc_keyframe* kf)
{
    return kf && kf->depth && kf->weight && kf->color && ((uintptr_t)kf->packed & 15u) == 0u;
}

// ---------------------------------------------------------------------------
// touched-block records
//
// A keyframe integrated at a pose touches a set of blocks that depends only
// on the keyframe and the pose; de-integrating it at that pose (Eq. 2)
// touches exactly the same set.  Integrations therefore append the blocks
// they touch to a record keyed by (keyframe buffers, intrinsics, pose), and
// a later de-integration of the same key takes the record as its candidate
// blocks instead of generating frustum candidates.  A record is dropped when
// as many de-integrations as integrations of its key have been applied, on
// reset and on import; a record that overflowed its capacity is ignored on
// the device (frustum candidates are generated instead).
// ---------------------------------------------------------------------------

}  // namespace sc

struct RecordRegistry {
    struct Entry {
        int slot;
        int refs;
    };
    std::unordered_map<std::string, Entry> map;
    std::vector<int> free_slots;
    std::vector<int> pending;  // slots released by de-integrations of the call in flight
    uint64_t* d_keys = nullptr;
    uint32_t* d_count = nullptr;
    int slots = 0, cap = 0;
    bool failed = false;
};

namespace sc {

constexpr int kRecSlots = 1024;   // records held at once
constexpr int kRecCap = 1024;     // blocks per part of a record, of kRecShards

static std::string rec_fingerprint(const sc_keyframe* kf, const sc_intrinsics* in, const sc_pose* T)
{
    std::string f;
    f.reserve(4 * sizeof(void*) + sizeof(sc_intrinsics) + sizeof(sc_pose));
    const void* ptrs[4] = {kf->depth, kf->weight, kf->color, kf->packed};
    f.append(reinterpret_cast<const char*>(ptrs), sizeof(ptrs));
    f.append(reinterpret_cast<const char*>(in), sizeof(*in));
    f.append(reinterpret_cast<const char*>(T), sizeof(*T));
    return f;
}

static bool rec_ready(sc_volume* vol)
{
    if (!vol->rec) vol->rec = new (std::nothrow) RecordRegistry();
    RecordRegistry* r = vol->rec;
    if (!r || r->failed) return false;
    if (r->d_keys) return true;
    const int cap = (int)std::min<int64_t>(kRecCap, vol->p.max_blocks);
    if (!device_alloc(&r->d_keys, sizeof(uint64_t) * (size_t)kRecSlots * kRecShards * cap) ||
        !device_alloc(&r->d_count, sizeof(uint32_t) * (size_t)kRecSlots * kRecShards * kRecCountStride)) {
        (void)hipGetLastError();
        hipFree(r->d_keys);
        r->d_keys = nullptr;
        r->failed = true;
        return false;
    }
    r->slots = kRecSlots;
    r->cap = cap;
    r->free_slots.clear();
    for (int i = kRecSlots - 1; i >= 0; --i) r->free_slots.push_back(i);
    return true;
}

void rec_clear(sc_volume* vol)
{
    RecordRegistry* r = vol->rec;
    if (!r || !r->d_keys) return;
    r->map.clear();
    r->pending.clear();
    r->free_slots.clear();
    for (int i = r->slots - 1; i >= 0; --i) r->free_slots.push_back(i);
}

void rec_destroy(sc_volume* vol)
{
    RecordRegistry* r = vol->rec;
    if (!r) return;
    hipFree(r->d_keys);
    hipFree(r->d_count);
    delete r;
    vol->rec = nullptr;
}

// An integration of kf at T: an existing record of the key only gains a
// reference (the same keyframe at the same pose touches the same blocks, so
// the record still holds them); otherwise, with `records` (the kernel that
// will run appends the touched blocks), the op fills a fresh record (rec_mode
// 1; its count is cleared on the device before the pass).
void rec_for_integration(sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* in, const sc_pose* T,
                         bool records, OpDesc* op)
{
    if (!rec_ready(vol)) return;
    RecordRegistry* r = vol->rec;
    const std::string f = rec_fingerprint(kf, in, T);
    auto it = r->map.find(f);
    if (!records) {
        if (it != r->map.end()) it->second.refs += 1;
        return;
    }
    if (it != r->map.end()) {
        // the same keyframe at the same pose touches the same blocks: the
        // record stands as it is (so a slot being recorded is always a fresh
        // one, never one a de-integration of the same batch reads)
        it->second.refs += 1;
        return;
    }
    if (r->free_slots.empty()) return;
    const int slot = r->free_slots.back();
    r->free_slots.pop_back();
    r->map.emplace(f, RecordRegistry::Entry{slot, 1});
    op->rec_keys = r->d_keys + (size_t)slot * kRecShards * r->cap;
    op->rec_count = r->d_count + (size_t)slot * kRecShards * kRecCountStride;
    op->rec_cap = r->cap;
    op->rec_mode = 1;
}

// A de-integration of kf at T: takes the key's record when there is one
// (rec_mode 2) and releases one reference to it; the slot becomes free once
// the call's work is enqueued (rec_commit).
void rec_for_deintegration(sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* in, const sc_pose* T,
                           OpDesc* op)
{
    RecordRegistry* r = vol->rec;
    if (!r || !r->d_keys) return;
    auto it = r->map.find(rec_fingerprint(kf, in, T));
    if (it == r->map.end()) return;
    const int slot = it->second.slot;
    op->rec_keys = r->d_keys + (size_t)slot * kRecShards * r->cap;
    op->rec_count = r->d_count + (size_t)slot * kRecShards * kRecCountStride;
    op->rec_cap = r->cap;
    op->rec_mode = 2;
    if (--it->second.refs == 0) {
        r->pending.push_back(slot);
        r->map.erase(it);
    }
}

// Frees the slots released during a call, once all its work is enqueued:
// later work on the stream runs after it.
void rec_commit(sc_volume* vol)
{
    RecordRegistry* r = vol->rec;
    if (!r) return;
    for (int slot : r->pending) r->free_slots.push_back(slot);
    r->pending.clear();
}

sc_status plain_op(sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* in, const sc_pose* T, int sign,
                   hipStream_t s)
{
    if (!vol || !keyframe_ok(kf) || !intr_ok(in) || !T) return SC_EINVAL;
    OpDesc op;
    make_op(vol, kf, in, T, sign, 0, &op);
    if (sign > 0) {
        rec_for_integration(vol, kf, in, T, true, &op);
    } else {
        // the plain de-integration generates its own candidates: only the
        // reference is released
        OpDesc tmp = op;
        rec_for_deintegration(vol, kf, in, T, &tmp);
    }
    const int p = vol->parity;
    vol->parity ^= 1;
    dim3 tiles((in->width + kTilePlain - 1) / kTilePlain, (in->height + kTilePlain - 1) / kTilePlain);
    const bool dirty = vol->cand_dirty;
    vol->cand_dirty = true;
    cand_plain_kernel<<<tiles, CandCfg<kTilePlain, kCellPlain>::threads, 0, s>>>(op, vol->dev, vol->cand, p);
    const sc_status sst = stream_in_plain(vol, p, s);
    if (sst != SC_OK) {
        rec_commit(vol);
        return sst;
    }
    const int grid = vol->n_cu * vol->plain_wgs;  // resident at once
    if (vol->p.color_mode == SC_COLOR_F32)
        update_plain_kernel<SC_COLOR_F32, false><<<grid, 256, 0, s>>>(op, vol->dev, vol->cand, p);
    else if (op.packed)
        update_plain_kernel<SC_COLOR_RGBA8, true><<<grid, 256, 0, s>>>(op, vol->dev, vol->cand, p);
    else
        update_plain_kernel<SC_COLOR_RGBA8, false><<<grid, 256, 0, s>>>(op, vol->dev, vol->cand, p);
    rec_commit(vol);
    if (hipGetLastError() != hipSuccess) return SC_EDEVICE;
    vol->cand_dirty = dirty;  // the pass leaves the candidate table as it found it
    return SC_OK;
}

}  // namespace sc

namespace sc {

// full: nothing is known about the buffers (a new volume).
static sc_status reset_volume(sc_volume* vol, bool full, hipStream_t s)
{
    reset_kernel<<<vol->n_cu * 8, 256, 0, s>>>(vol->dev, vol->cand, vol->adj_acc, full, vol->cand_dirty);
    reset_counts_kernel<<<1, 64, 0, s>>>(vol->dev);
    vol->parity = 0;
    vol->cand_dirty = false;
    rec_clear(vol);
    stream_clear(vol);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

}  // namespace sc

using namespace sc;

#define HIP_TRY(x)                                \
    do {                                          \
        if ((x) != hipSuccess) return SC_EDEVICE; \
    } while (0)

extern "C" {

const char* sc_version(void) { return "scsurf 0.1 (gfx950)"; }

sc_status sc_volume_create(const sc_volume_params* p, sc_volume** out)
{
    if (!out) return SC_EINVAL;
    *out = nullptr;
    if (!p || !(p->voxel_size > 0.0f) || !(p->trunc > 0.0f) || !is_pow2(p->n_buckets) || p->n_buckets > (1ll << 30) ||
        p->max_blocks <= 0 || p->max_blocks > (1ll << 30) ||
        (p->color_mode != SC_COLOR_RGBA8 && p->color_mode != SC_COLOR_F32) || p->max_batch_ops <= 0 ||
        p->max_batch_ops > kMaxBatchOps)
        return SC_EINVAL;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, dev));
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) return SC_ENOLIB;
    sc_volume* vol = new (std::nothrow) sc_volume();
    if (!vol) return SC_ENOMEM;
    memset(vol, 0, sizeof(*vol));
    scratch_volumes(+1);
    vol->p = *p;
    vol->device = dev;
    vol->n_cu = prop.multiProcessorCount;
    for (int k = 0; k < 3; ++k) vol->cand_wgs[k] = cand_batch_resident_wgs(k);
    {
        int n = 0;
        const void* k = p->color_mode == SC_COLOR_F32 ? (const void*)update_plain_kernel<SC_COLOR_F32, false>
                                                      : (const void*)update_plain_kernel<SC_COLOR_RGBA8, false>;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, 256, 0);
        vol->plain_wgs = (e == hipSuccess) ? std::max(1, std::min(n, 4)) : 1;
    }
    // default voxel-pass schedule: RGBA8 volumes take the ring pass (two
    // wavefronts per workgroup, eight workgroups per CU), the fastest measured
    // on a 400-operation update of 200 keyframes at 640x480, which also keeps
    // touched-block records for later de-integrations; FP32-colour volumes
    // the per-lane pass
    vol->sched.vpl = 8;
    if (p->color_mode == SC_COLOR_RGBA8) {
        vol->sched.waves_per_wg = 2;
        vol->sched.wgs_per_cu = 8;
        vol->sched.compact = 4;
    } else {
        vol->sched.waves_per_wg = 4;
        vol->sched.wgs_per_cu = 4;
    }
    VolDev& d = vol->dev;
    d.bucket_mask = (uint32_t)(p->n_buckets - 1);
    d.max_blocks = (int32_t)p->max_blocks;
    d.stride = (p->color_mode == SC_COLOR_RGBA8) ? 4 * kBlockVox : 9 * kBlockVox;
    d.color_mode = p->color_mode;
    d.s = p->voxel_size;
    d.mu = p->trunc;
    // candidate table: as many buckets as the volume, capped; one mask word per 64 batch operations
    uint64_t cb = (uint64_t)std::min<int64_t>(std::max<int64_t>(p->n_buckets, 1 << 16), 1 << 23);
    vol->cand_buckets = (uint32_t)cb;
    CandDev& c = vol->cand;
    c.mask_bits = (uint32_t)(cb - 1);
    c.cap = (uint32_t)(cb / 2);
    c.words = (p->max_batch_ops + 63) / 64;
    c.seg_cap = (uint32_t)(cb / 16);  // twice an even share; what does not fit goes to the last list
    bool ok = true;
    ok &= device_alloc(&d.keys, sizeof(uint64_t) * p->n_buckets);
    ok &= device_alloc(&d.vals, sizeof(int32_t) * p->n_buckets);
    ok &= device_alloc(&d.slot_keys, sizeof(uint64_t) * p->max_blocks);
    ok &= device_alloc(&d.pool, sizeof(float) * (size_t)d.stride * p->max_blocks);
    ok &= device_alloc(&d.n_blocks, 64);
    ok &= device_alloc(&d.err, 64);
    ok &= device_alloc(&c.keys, sizeof(uint64_t) * cb);
    ok &= device_alloc(&c.mask, sizeof(uint64_t) * cb * c.words);
    ok &= device_alloc(&c.list, sizeof(uint32_t) * c.cap);
    ok &= device_alloc(&c.sorted, sizeof(uint32_t) * cb);  // every bucket may be a candidate
    ok &= device_alloc(&c.skey, sizeof(uint64_t) * cb);
    ok &= device_alloc(&c.sslot, sizeof(int32_t) * cb);
    ok &= device_alloc(&c.counters, 64 * sizeof(uint32_t));
    ok &= device_alloc(&c.bins, sizeof(uint32_t) * 2 * (kMaxBatchOps + 2));
    ok &= device_alloc(&c.seg, sizeof(uint32_t) * ((size_t)kSegs * c.seg_cap + cb));
    ok &= device_alloc(&c.seg_n, sizeof(uint32_t) * (kSegs + 1) * kRecCountStride);
    ok &= device_alloc(&c.cursors, sizeof(uint32_t) * 2 * kCursorSet);
    ok &= device_alloc(&c.big, sizeof(uint32_t) * (kBigCap + 1));
    ok &= device_alloc(&c.stats, sizeof(unsigned long long) * 4 * kStatSlots * kStatStride);
    ok &= device_alloc(&vol->d_ops, sizeof(OpDesc) * p->max_batch_ops);
    ok &= device_alloc(&vol->adj_acc, sizeof(double) * 3 * kAdjChunk);
    ok &= hipHostMalloc((void**)&vol->h_ops, 2 * sizeof(OpDesc) * p->max_batch_ops, hipHostMallocDefault) ==
          hipSuccess;
    ok &= device_alloc(&vol->d_hdr, sizeof(BatchHdr));
    ok &= hipHostMalloc((void**)&vol->h_hdr, 2 * sizeof(BatchHdr), hipHostMallocDefault) == hipSuccess;
    ok &= hipStreamCreateWithFlags(&vol->cap_stream, hipStreamNonBlocking) == hipSuccess;
    ok &= hipEventCreateWithFlags(&vol->staged[0], hipEventDisableTiming) == hipSuccess;
    ok &= hipEventCreateWithFlags(&vol->staged[1], hipEventDisableTiming) == hipSuccess;
    if (!ok) {
        sc_volume_destroy(vol);
        return SC_ENOMEM;
    }
    hipStream_t s = 0;
    sc_status st = reset_volume(vol, true, s);
    for (int b = 0; b < 2; ++b)
        if (st == SC_OK && hipEventRecord(vol->staged[b], s) != hipSuccess) st = SC_EDEVICE;
    if (st != SC_OK || hipStreamSynchronize(s) != hipSuccess) {
        sc_volume_destroy(vol);
        return SC_EDEVICE;
    }
    *out = vol;
    return SC_OK;
}

void sc_volume_destroy(sc_volume* vol)
{
    if (!vol) return;
    hipDeviceSynchronize();
    for (hipGraphExec_t g : vol->graph_pre)
        if (g) hipGraphExecDestroy(g);
    for (auto& g : vol->graph_main)
        if (g) hipGraphExecDestroy(g);
    for (int i = 0; i < 2 * vol->timing_cap; ++i) hipEventDestroy(vol->timing_ev[i]);
    delete[] vol->timing_ev;
    hipFree(vol->cand.stats);
    hipFree(vol->cand.skey);
    hipFree(vol->cand.sslot);
    hipFree(vol->dev.keys);
    hipFree(vol->dev.vals);
    hipFree(vol->dev.slot_keys);
    hipFree(vol->dev.pool);
    hipFree(vol->dev.n_blocks);
    hipFree(vol->dev.err);
    hipFree(vol->cand.keys);
    hipFree(vol->cand.mask);
    hipFree(vol->cand.list);
    hipFree(vol->cand.sorted);
    hipFree(vol->cand.counters);
    hipFree(vol->cand.bins);
    hipFree(vol->cand.seg);
    hipFree(vol->cand.seg_n);
    hipFree(vol->cand.cursors);
    hipFree(vol->cand.big);
    hipFree(vol->d_ops);
    hipFree(vol->adj_acc);
    hipFree(vol->d_hdr);
    if (vol->h_ops) hipHostFree(vol->h_ops);
    if (vol->h_hdr) hipHostFree(vol->h_hdr);
    if (vol->cap_stream) hipStreamDestroy(vol->cap_stream);
    for (hipEvent_t e : vol->staged)
        if (e) hipEventDestroy(e);
    rec_destroy(vol);
    stream_destroy(vol);
    scratch_volumes(-1);
    delete vol;
}

sc_status sc_volume_reset(sc_volume* vol, void* stream)
{
    if (!vol) return SC_EINVAL;
    return reset_volume(vol, false, (hipStream_t)stream);
}

sc_status sc_volume_query(sc_volume* vol, void* stream, int64_t* n_blocks, int32_t* sticky_error)
{
    if (!vol) return SC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    uint32_t nb = 0;
    int32_t e = 0;
    HIP_TRY(hipMemcpyAsync(&nb, vol->dev.n_blocks, sizeof(nb), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(&e, vol->dev.err, sizeof(e), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (n_blocks) *n_blocks = std::min<int64_t>((int64_t)nb, vol->p.max_blocks);
    if (sticky_error) *sticky_error = e;
    return SC_OK;
}

sc_status sc_volume_export(sc_volume* vol, void* stream, int32_t* block_xyz, float* D, float* W, void* C, int64_t cap,
                           int64_t* n_out)
{
    if (!vol || cap < 0) return SC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    if (cap > 0)
        export_kernel<<<(unsigned)std::min<int64_t>(std::min(cap, vol->p.max_blocks), vol->n_cu * 64), 256, 0, s>>>(
            vol->dev, cap, block_xyz, D, W, C);
    HIP_TRY(hipGetLastError());
    uint32_t nb = 0;
    HIP_TRY(hipMemcpyAsync(&nb, vol->dev.n_blocks, sizeof(nb), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (n_out) *n_out = std::min<int64_t>((int64_t)nb, vol->p.max_blocks);
    return SC_OK;
}

sc_status sc_volume_import(sc_volume* vol, void* stream, const int32_t* block_xyz, const float* D, const float* W,
                           const void* C, int64_t n)
{
    if (!vol || n < 0 || (n > 0 && !block_xyz) || n > vol->p.max_blocks || stream_host_blocks(vol) > 0)
        return SC_EINVAL;
    if (n == 0) return SC_OK;
    hipStream_t s = (hipStream_t)stream;
    Scratch buf = scratch_take(sizeof(int32_t) * (size_t)n);
    if (!buf.p) return SC_EDEVICE;
    int32_t* slots = reinterpret_cast<int32_t*>(buf.p);
    sc_status st = hash_alloc(vol, block_xyz, n, slots, stream);
    if (st == SC_OK) {
        import_kernel<<<(unsigned)n, 256, 0, s>>>(vol->dev, slots, n, D, W, C);
        st = hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
    }
    int64_t nb = 0;
    int32_t sticky = 0;
    if (st == SC_OK) st = sc_volume_query(vol, stream, &nb, &sticky);
    scratch_give(buf, st == SC_OK);
    if (st != SC_OK) return st;
    return sticky;
}

int64_t sc_keyframe_pack_bytes(int32_t width, int32_t height)
{
    if (width <= 0 || height <= 0 || width > 16384 || height > 16384) return 0;
    const int64_t cells = (int64_t)((width + 3) / 4) * ((height + 3) / 4);
    return (int64_t)width * height * 16 + cells * 8;
}

sc_status sc_keyframe_pack(const sc_keyframe* kf, int32_t width, int32_t height, void* packed, int64_t packed_bytes,
                           void* stream)
{
    const int64_t need = sc_keyframe_pack_bytes(width, height);
    if (!kf || !kf->depth || !kf->weight || !kf->color || !packed || ((uintptr_t)packed & 15u) || need == 0 ||
        packed_bytes < need)
        return SC_EINVAL;
    const int64_t n = (int64_t)width * height;
    const int cells_w = (width + 3) / 4, cells_h = (height + 3) / 4;
    const int64_t items = (int64_t)((width + 63) / 64) * cells_h;  // wavefronts
    pack_kernel<<<(unsigned)((items + 3) / 4), 256, 0, (hipStream_t)stream>>>(
        kf->depth, kf->weight, reinterpret_cast<const uint32_t*>(kf->color), reinterpret_cast<uint4*>(packed),
        reinterpret_cast<float2*>(reinterpret_cast<uint4*>(packed) + n), width, height, cells_w, items);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

sc_status hash_alloc(sc_volume* vol, const int32_t* block_xyz, int64_t n, int32_t* slots_out, void* stream)
{
    if (!vol || n < 0 || (n > 0 && !block_xyz) || stream_host_blocks(vol) > 0) return SC_EINVAL;
    if (n == 0) return SC_OK;
    hipStream_t s = (hipStream_t)stream;
    const unsigned grid = (unsigned)((n + 255) / 256);
    hash_alloc_kernel<<<grid, 256, 0, s>>>(vol->dev, block_xyz, n);
    if (slots_out) hash_lookup_kernel<<<grid, 256, 0, s>>>(vol->dev, block_xyz, n, slots_out);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

sc_status tsdf_integrate(sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* intr, const sc_pose* T,
                         void* stream)
{
    return plain_op(vol, kf, intr, T, +1, (hipStream_t)stream);
}

sc_status tsdf_deintegrate(sc_volume* vol, const sc_keyframe* kf, const sc_intrinsics* intr, const sc_pose* T,
                           void* stream)
{
    return plain_op(vol, kf, intr, T, -1, (hipStream_t)stream);
}

sc_status reintegrate_plain(sc_volume* vol, const sc_keyframe* kfs, int32_t n_kf, const sc_intrinsics* intr,
                            sc_pose* T_integrated, const sc_pose* T_new, int32_t m, int32_t mode,
                            int32_t* selected_out, int32_t* n_selected, void* stream)
{
    if (!vol || !kfs || n_kf <= 0 || !T_integrated || !T_new || !intr_ok(intr)) return SC_EINVAL;
    for (int i = 0; i < n_kf; ++i)
        if (!keyframe_ok(&kfs[i])) return SC_EINVAL;
    int32_t* order = new (std::nothrow) int32_t[n_kf];
    if (!order) return SC_ENOMEM;
    const int32_t ns = sc_select(T_integrated, T_new, n_kf, m, mode, order, nullptr);
    if (ns < 0) {
        delete[] order;
        return ns;
    }
    hipStream_t s = (hipStream_t)stream;
    sc_status st = SC_OK;
    for (int j = 0; j < ns && st == SC_OK; ++j) st = plain_op(vol, &kfs[order[j]], intr, &T_integrated[order[j]], -1, s);
    for (int j = 0; j < ns && st == SC_OK; ++j) st = plain_op(vol, &kfs[order[j]], intr, &T_new[order[j]], +1, s);
    if (st == SC_OK) {
        for (int j = 0; j < ns; ++j) T_integrated[order[j]] = T_new[order[j]];
        if (selected_out) memcpy(selected_out, order, sizeof(int32_t) * ns);
        if (n_selected) *n_selected = ns;
    }
    delete[] order;
    return st;
}

}  // extern "C"
