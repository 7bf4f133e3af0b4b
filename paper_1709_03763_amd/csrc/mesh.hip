// Iso-surface extraction (Sec. 3 "SDF volume": Marching Cubes over the SDF)
// and the surface metrics of Sec. 5 (mean absolute deviation of
// nearest-neighbour distances between point sets: CORR and COMPL).
#include <string.h>

#include <algorithm>
#include <mutex>

#include "common.hpp"
#include "internal.hpp"
#include "kernels.hpp"

#define MESH_TRY(x)                               \
    do {                                          \
        if ((x) != hipSuccess) return SC_EDEVICE; \
    } while (0)

namespace sc {

// ---------------------------------------------------------------------------
// case table
// ---------------------------------------------------------------------------

// Corner k of the cube of voxel n sits at n + (k & 1, (k >> 1) & 1, k >> 2).
// Edge e = 4 a + o1 + 2 o2 runs along axis a from the corner whose offsets on
// the two other axes (in increasing axis order) are (o1, o2).  A corner is
// inside when D < 0.  The table is built on the host from a rule: on each
// face, with its corners counter-clockwise about the outward normal, every
// run of inside corners is cut off by a segment from the edge that enters
// the run to the edge that leaves it (diagonal inside corners of a face stay
// apart, identically on both cubes sharing the face).  Segments chain across
// faces into loops; loops are ordered by their smallest edge and start
// there.  A loop holding two segments of one face is fanned around an added
// centre vertex (the mean of its vertices, summed in loop order), any other
// loop from its first vertex, so no triangle side lies inside a face.
//
// Per case, 16 bytes: loops in order, each a header byte (length, | 0x80
// when fanned around a centre) followed by its edges; a zero header (or the
// end of the 16 bytes) ends the case.
// `tri` states the same triangles one by one, their corners as edges or, from
// kMcCentre, loop centres: what the fill pass reads (at most one triangle an
// edge: twelve).
constexpr int kMcMaxTri = 12, kMcCentre = 12;  // at most four loops: corners fit four bits

struct McTable {
    uint8_t loops[256][16];
    uint8_t ntri[256];
    alignas(4) uint8_t tri[256][kMcMaxTri][4];
};

static __device__ McTable g_mc;

static int mc_corner(const int off[3]) { return off[0] + 2 * off[1] + 4 * off[2]; }

static int mc_edge_between(int k0, int k1)
{
    const int o0[3] = {k0 & 1, (k0 >> 1) & 1, (k0 >> 2) & 1};
    const int o1[3] = {k1 & 1, (k1 >> 1) & 1, (k1 >> 2) & 1};
    int a = 0;
    while (o0[a] == o1[a]) ++a;
    const int* lo = (o0[a] < o1[a]) ? o0 : o1;
    int other[2], m = 0;
    for (int b = 0; b < 3; ++b)
        if (b != a) other[m++] = b;
    return 4 * a + lo[other[0]] + 2 * lo[other[1]];
}

static bool mc_build(McTable& T)
{
    memset(&T, 0, sizeof(T));
    int ring[6][4];
    for (int a = 0; a < 3; ++a) {
        const int u = (a + 1) % 3, v = (a + 2) % 3;
        static const int uv[4][2] = {{0, 0}, {1, 0}, {1, 1}, {0, 1}};  // counter-clockwise about +e_a
        for (int side = 0; side < 2; ++side) {
            for (int i = 0; i < 4; ++i) {
                int off[3];
                off[a] = side;
                off[u] = uv[i][0];
                off[v] = uv[i][1];
                // about -e_a on the low face: the same corners in reverse
                ring[2 * a + side][side ? i : 3 - i] = mc_corner(off);
            }
        }
    }
    for (int c = 0; c < 256; ++c) {
        int next[12], face[12];
        for (int e = 0; e < 12; ++e) next[e] = face[e] = -1;
        for (int f = 0; f < 6; ++f) {
            int ce[4], enters[4], n = 0;
            for (int i = 0; i < 4; ++i) {
                const int k0 = ring[f][i], k1 = ring[f][(i + 1) & 3];
                const int in0 = (c >> k0) & 1, in1 = (c >> k1) & 1;
                if (in0 != in1) {
                    ce[n] = mc_edge_between(k0, k1);
                    enters[n] = in1;
                    ++n;
                }
            }
            for (int j = 0; j < n; ++j)
                if (enters[j]) {
                    next[ce[j]] = ce[(j + 1) % n];
                    face[ce[j]] = f;
                }
        }
        bool seen[12] = {};
        int p = 0, ntri = 0, li = 0;
        for (int e0 = 0; e0 < 12; ++e0) {
            if (next[e0] < 0 || seen[e0]) continue;
            uint8_t loop[12];
            int len = 0, e = e0;
            unsigned fmask = 0;
            bool centre = false;
            while (!seen[e]) {
                seen[e] = true;
                loop[len++] = (uint8_t)e;
                centre |= ((fmask >> face[e]) & 1u) != 0;
                fmask |= 1u << face[e];
                e = next[e];
            }
            if (p + 1 + len > 16) return false;  // at most four loops over twelve edges: never
            T.loops[c][p++] = (uint8_t)(len | (centre ? 0x80 : 0));
            for (int i = 0; i < len; ++i) T.loops[c][p++] = loop[i];
            const int n_t = centre ? len : len - 2;
            if (ntri + n_t > kMcMaxTri) return false;  // never: a loop has no more triangles than edges
            for (int i = 0; i < n_t; ++i) {
                uint8_t* t = T.tri[c][ntri++];
                t[0] = centre ? (uint8_t)(kMcCentre + li) : loop[0];
                t[1] = centre ? loop[i] : loop[i + 1];
                t[2] = centre ? loop[(i + 1) % len] : loop[i + 2];
            }
            ++li;
        }
        T.ntri[c] = (uint8_t)ntri;
    }
    return true;
}

static sc_status mc_table_ready()
{
    static std::mutex mu;
    static bool done[64] = {};
    int dev = 0;
    MESH_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return SC_EDEVICE;
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev]) {
        McTable T;
        if (!mc_build(T)) return SC_EDEVICE;
        MESH_TRY(hipMemcpyToSymbol(HIP_SYMBOL(g_mc), &T, sizeof(T), 0, hipMemcpyHostToDevice));
        done[dev] = true;
    }
    return SC_OK;
}

// ---------------------------------------------------------------------------
// Marching Cubes: one wavefront per allocated block and its +x, +y, +z
// neighbours' first layers (9 x 9 x 9 voxels).  A count pass stores each
// block's triangle count, a scan turns the counts into offsets, and the fill
// pass writes every block's triangles from its offset: no shared counter, and
// the output order is fixed (pool order, then by lane and z-slice).
//
// Bound: the loads of the halo (64-byte lines holding one or eight wanted
// voxels) and, filling, the bytes written.  Every load of a wavefront issues
// before the first is used; what a cube's case needs of a voxel is two bits
// (observed, inside), so the nine voxels of a column are two 9-bit masks in a
// lane's register, the columns of the +x and +y layers are cut out of
// wavefront ballots and a cube's three other columns come by shuffles; only
// the fill pass puts D into LDS, for blocks that hold a triangle.  It lists
// the block's triangles in LDS and then makes one vertex instance a thread,
// so its stores are consecutive.  28,700 blocks, 3.6 M triangles: 227 us a
// pass (a serial loop over a lane's eight cubes, 4-byte stores 36 and 48
// bytes apart) -> 68 us counting, 181 us filling.
// ---------------------------------------------------------------------------

struct MeshOut {
    float* xyz;               // cap x 3 x 3, or null
    int32_t* keys;            // cap x 3 x 4, or null
    uint32_t* counts;         // triangles per block: written by the count pass, read by the fill pass
    const uint64_t* offsets;  // fill pass: first triangle of each block, counted from its scan group's,
    const uint64_t* sums;     //   and the groups' (kScanGroup blocks each)
    int64_t cap;
};
constexpr uint32_t kScanGroup = 1024;

// Position (FP64, metres) and key (x, y, z, axis) of the vertex on edge e of
// the cube whose corner 0 is LDS cell r0 and voxel g.
__device__ inline void mc_edge_vertex(int e, const double* sD, int r0, const int g[3], double s, double p[3],
                                      int key[4])
{
    const int a = e >> 2, r = e & 3;
    const int o1 = (a == 0) ? 1 : 0, o2 = (a == 2) ? 1 : 2;
    const int b1 = r & 1, b2 = r >> 1;
    const int off[3] = {o1 == 0 ? b1 : 0, o1 == 1 ? b1 : o2 == 1 ? b2 : 0, o2 == 2 ? b2 : 0};
    const int lo = r0 + off[0] + 9 * off[1] + 81 * off[2];
    const int hi = lo + ((a == 0) ? 1 : (a == 1) ? 9 : 81);
    const double d0 = sD[lo], d1 = sD[hi];
    const double t = d0 / (d0 - d1);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        key[b] = g[b] + off[b];
        p[b] = s * (a == b ? (double)key[b] + t : (double)key[b]);
    }
    key[3] = a;
}

// Centre of loop li of a case: the mean of its vertices, summed in loop order.
__device__ inline void mc_centre_vertex(uint32_t cs, int li, const double* sD, int r0, const int g[3], double s,
                                        double p[3], int key[4])
{
    const uint8_t* tab = g_mc.loops[cs];
    for (int k = 0; k < li; ++k) tab += 1 + (tab[0] & 0x7f);
    const int len = tab[0] & 0x7f;
    p[0] = p[1] = p[2] = 0.0;
    for (int i = 0; i < len; ++i) {
        double q[3];
        mc_edge_vertex(tab[1 + i], sD, r0, g, s, q, key);
#pragma unroll
        for (int b = 0; b < 3; ++b) p[b] = p[b] + q[b];
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        p[b] = p[b] / (double)len;
        key[b] = g[b];
    }
    key[3] = 3 + li;
}

// Bits y, y + 8, ..., y + 56 of a mask, as eight consecutive ones.
__device__ inline uint32_t every_eighth(uint64_t m, int y)
{
    return (uint32_t)((((m >> y) & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56);
}

constexpr int kMeshList = 1024;  // triangles listed at once (a block seldom holds more than 300)

template <bool kFill>
__global__ __launch_bounds__(64) void mesh_kernel(VolDev v, MeshOut out)
{
    __shared__ double sD[kFill ? 729 : 1];
    __shared__ uint16_t list[kFill ? kMeshList : 1];  // cube | triangle of its case << 9
    __shared__ uint8_t scase[kFill ? 512 : 1];
    const int lane = threadIdx.x;
    const int b = blockIdx.x;
    if (kFill && out.counts[b] == 0u) return;
    const float* const blk = v.pool + (size_t)b * v.stride;
    double d[8];
    float w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        d[j] = reinterpret_cast<const double*>(blk)[lane + 64 * j];
        w[j] = blk[kPoolW + lane + 64 * j];
    }
    int bx, by, bz;
    unpack_key(v.slot_keys[b], bx, by, bz);
    // the neighbour at offset (n & 1, n >> 1 & 1, n >> 2) is lane n's
    int found = -1;
    if (lane >= 1 && lane < 8) {
        const int x = bx + (lane & 1), y = by + ((lane >> 1) & 1), z = bz + (lane >> 2);
        found = vol_find(v, pack_key(x, y, z), x, y, z);
    }
    int slot[8];
#pragma unroll
    for (int n = 1; n < 8; ++n) slot[n] = (int)__builtin_amdgcn_readlane((uint32_t)found, n);
    // the layers x = 8 (lane = y + 8 z), y = 8 (x + 8 z), z = 8 (x + 8 y), and the lines where two or three of
    // them meet: lanes 0-7 (8, 8, z), 8-15 (8, y, 8), 16-23 (x, 8, 8), lane 24 the corner
    const int lo3 = lane & 7, hi3 = lane >> 3;
    double hd[4] = {0.0, 0.0, 0.0, 0.0};
    float hw[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto halo = [&](int k, int sl, int i) {
        if (sl >= 0) {
            const float* nb = v.pool + (size_t)sl * v.stride;
            hd[k] = reinterpret_cast<const double*>(nb)[i];
            hw[k] = nb[kPoolW + i];
        }
    };
    halo(0, slot[1], 8 * lo3 + 64 * hi3);
    halo(1, slot[2], lo3 + 64 * hi3);
    halo(2, slot[4], lane);
    {
        const int line = hi3;  // 0, 1, 2, and 3 for the corner
        const int sl = line == 0 ? slot[3] : line == 1 ? slot[5] : line == 2 ? slot[6] : lane == 24 ? slot[7] : -1;
        halo(3, sl, line == 0 ? 64 * lo3 : line == 1 ? 8 * lo3 : line == 2 ? lo3 : 0);
    }
    // columns: bit z of the low half, observed; of the high half, inside
    uint32_t own = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) own |= (w[j] > 0.0f ? 1u << j : 0u) | (d[j] < 0.0 ? 0x10000u << j : 0u);
    own |= (hw[2] > 0.0f ? 1u << 8 : 0u) | (hd[2] < 0.0 ? 0x10000u << 8 : 0u);
    uint64_t ok[4], in[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        ok[k] = __ballot(hw[k] > 0.0f);
        in[k] = __ballot(hd[k] < 0.0);
    }
    auto column = [&](int k, int i, int top) {  // column i of layer k; its z = 8 voxel is bit `top` of the lines
        return every_eighth(ok[k], i) | (every_eighth(in[k], i) << 16) | ((uint32_t)((ok[3] >> top) & 1u) << 8) |
               ((uint32_t)((in[3] >> top) & 1u) << 24);
    };
    const uint32_t corner = (uint32_t)(ok[3] & 255u) | ((uint32_t)(in[3] & 255u) << 16) |
                            ((uint32_t)((ok[3] >> 24) & 1u) << 8) | ((uint32_t)((in[3] >> 24) & 1u) << 24);
    const uint32_t right = (uint32_t)__shfl((int)own, lane + 1), up = (uint32_t)__shfl((int)own, lane + 8),
                   diag = (uint32_t)__shfl((int)own, lane + 9);
    const bool ex = lo3 == 7, ey = hi3 == 7;
    const int yn = min(hi3 + 1, 7), xn = min(lo3 + 1, 7);
    const uint32_t c10 = ex ? column(0, hi3, 8 + hi3) : right;
    const uint32_t c01 = ey ? column(1, lo3, 16 + lo3) : up;
    const uint32_t c11 = ex ? (ey ? corner : column(0, yn, 8 + yn)) : (ey ? column(1, xn, 16 + xn) : diag);
    const uint32_t seen = own & c10 & c01 & c11;
    const uint32_t all = seen & (seen >> 1);  // bit j: the cube of slice j is observed
    uint32_t cases[8];
    uint32_t mine = 0u, per = 0u;  // per: four bits a cube
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t lo = ((own >> (16 + j)) & 1u) | (((c10 >> (16 + j)) & 1u) << 1) |
                            (((c01 >> (16 + j)) & 1u) << 2) | (((c11 >> (16 + j)) & 1u) << 3);
        const uint32_t hi = ((own >> (17 + j)) & 1u) | (((c10 >> (17 + j)) & 1u) << 1) |
                            (((c01 >> (17 + j)) & 1u) << 2) | (((c11 >> (17 + j)) & 1u) << 3);
        cases[j] = ((all >> j) & 1u) ? lo | (hi << 4) : 0u;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t nt = g_mc.ntri[cases[j]];
        per |= nt << (4 * j);
        mine += nt;
    }
    // wavefront-exclusive prefix of the triangle counts: the count pass
    // stores the block's total, the fill pass lists from the lane's place
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    const uint32_t total = (uint32_t)__shfl((int)incl, 63);
    if (!kFill) {
        if (lane == 0) out.counts[b] = total;
        return;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        sD[lo3 + 9 * hi3 + 81 * j] = d[j];
        scase[lane + 64 * j] = (uint8_t)cases[j];
    }
    sD[8 + 9 * lo3 + 81 * hi3] = hd[0];
    sD[lo3 + 72 + 81 * hi3] = hd[1];
    sD[lo3 + 9 * hi3 + 648] = hd[2];
    if (lane < 25) sD[hi3 == 0 ? 80 + 81 * lo3 : hi3 == 1 ? 656 + 9 * lo3 : hi3 == 2 ? 720 + lo3 : 728] = hd[3];
    const unsigned long long first = out.offsets[b] + out.sums[(uint32_t)b / kScanGroup];
    const double s = (double)v.s;
    for (uint32_t w0 = 0u; w0 < total; w0 += kMeshList) {
        // the triangles [w0, w0 + n) of the block
        const uint32_t n = min(total - w0, (uint32_t)kMeshList);
        uint32_t t = incl - mine - w0;  // below w0: wraps to a large number
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t nt = (per >> (4 * j)) & 15u;
            for (uint32_t i = 0; i < nt; ++i, ++t)
                if (t < n) list[t] = (uint16_t)((uint32_t)(lane + 64 * j) | (i << 9));
        }
        __syncthreads();
        // two instances a round, so that their table reads overlap
        for (uint32_t i0 = (uint32_t)lane; i0 < 3u * n; i0 += 128u) {
            uint32_t cube[2], cs[2], corner[2];
            int e[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint32_t i = min(i0 + 64u * k, 3u * n - 1u);
                const uint32_t tri = i / 3u;
                corner[k] = i - 3u * tri;
                const uint32_t it = list[tri];
                cube[k] = it & 511u;
                cs[k] = scase[cube[k]];
                e[k] = g_mc.tri[cs[k]][it >> 9][corner[k]];
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint32_t i = i0 + 64u * k;
                const unsigned long long to = first + w0 + i / 3u;
                if (i >= 3u * n || to >= (unsigned long long)out.cap) break;
                const int x = (int)(cube[k] & 7u), y = (int)((cube[k] >> 3) & 7u), z = (int)(cube[k] >> 6);
                const int r0 = x + 9 * y + 81 * z;
                const int g[3] = {8 * bx + x, 8 * by + y, 8 * bz + z};
                double p[3];
                int key[4];
                if (e[k] < kMcCentre)
                    mc_edge_vertex(e[k], sD, r0, g, s, p, key);
                else
                    mc_centre_vertex(cs[k], e[k] - kMcCentre, sD, r0, g, s, p, key);
                if (out.xyz) {
                    float* o = out.xyz + (to * 3 + corner[k]) * 3;
                    o[0] = (float)p[0];
                    o[1] = (float)p[1];
                    o[2] = (float)p[2];
                }
                if (out.keys) {
                    // the caller's keys are int32: 4-byte aligned
                    int32_t* o = out.keys + (to * 3 + corner[k]) * 4;
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[q] = key[q];
                }
            }
        }
        __syncthreads();
    }
}

// Exclusive scan of per-block triangle counts into 64-bit offsets: 1024
// counts per workgroup, then one workgroup scans the workgroup sums in
// chunks with a running carry, which the fill pass adds.
__global__ __launch_bounds__(256) void scan_local_kernel(const uint32_t* __restrict__ in, uint64_t* out, uint64_t* sums,
                                                         uint32_t n)
{
    __shared__ uint64_t part[256];
    const uint32_t i0 = (blockIdx.x * 256u + threadIdx.x) * 4u;
    uint64_t v[4], mine = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = (i0 + k < n) ? (uint64_t)in[i0 + k] : 0ull;
        mine += v[k];
    }
    part[threadIdx.x] = mine;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const uint64_t y = (threadIdx.x >= (unsigned)o) ? part[threadIdx.x - o] : 0ull;
        __syncthreads();
        part[threadIdx.x] += y;
        __syncthreads();
    }
    uint64_t run = part[threadIdx.x] - mine;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (i0 + k < n) out[i0 + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 255) sums[blockIdx.x] = part[255];
}

__global__ __launch_bounds__(256) void scan_sums_kernel(uint64_t* sums, uint32_t n, uint64_t* total)
{
    __shared__ uint64_t part[256];
    __shared__ uint64_t carry;
    if (threadIdx.x == 0) carry = 0ull;
    __syncthreads();
    for (uint32_t c0 = 0; c0 < n; c0 += 256u) {
        const uint32_t i = c0 + threadIdx.x;
        const uint64_t mine = (i < n) ? sums[i] : 0ull;
        part[threadIdx.x] = mine;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {
            const uint64_t y = (threadIdx.x >= (unsigned)o) ? part[threadIdx.x - o] : 0ull;
            __syncthreads();
            part[threadIdx.x] += y;
            __syncthreads();
        }
        if (i < n) sums[i] = carry + part[threadIdx.x] - mine;
        __syncthreads();
        if (threadIdx.x == 255) carry += part[255];
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

// ---------------------------------------------------------------------------
// unique vertices: a hash set over vertex keys
// ---------------------------------------------------------------------------

constexpr int kKeyRange = 1 << 19;  // |voxel coordinate| bound of the vertex key packing

__device__ inline uint64_t vertex_key(const int32_t* k, bool& bad)
{
    bad |= k[0] < -kKeyRange || k[0] >= kKeyRange || k[1] < -kKeyRange || k[1] >= kKeyRange || k[2] < -kKeyRange ||
           k[2] >= kKeyRange || k[3] < 0 || k[3] > 7;
    return ((uint64_t)(k[0] & 0xFFFFF) << 43) | ((uint64_t)(k[1] & 0xFFFFF) << 23) | ((uint64_t)(k[2] & 0xFFFFF) << 3) |
           (uint64_t)(k[3] & 7);
}

constexpr int kVertPerThread = 4;  // vertex instances per thread: one reservation per 1024
constexpr int kVertPerWg = 256 * kVertPerThread;
constexpr uint32_t kVertSet = 2048;  // LDS set entries of a workgroup (at most half full)

// Bucket of a key: neighbours along z, and the axes at one voxel, lie in one
// 32-entry stretch, so that the instances of a surface patch share lines.
__device__ inline uint32_t vertex_bucket(uint64_t key)
{
    return ((uint32_t)(((key >> 5) * 0x9E3779B97F4A7C15ull) >> 32) << 5) | ((uint32_t)key & 31u);
}

// Distinct keys of the instances.  A workgroup first reduces its 1024
// consecutive instances, a few hundred vertices of a mesh, in an LDS set; the
// first instance of each key inserts it in the hash set in memory (a plain
// read before the CAS: entries only go from free to a key), and those that
// insert first append their positions, a range reserved with one atomic per
// workgroup.  Bound: the latency of the random accesses to the table, five
// times fewer than with every instance inserting (10.8 M instances, 2.0 M
// vertices: 548 -> 206 us, and 45 -> 25 us to clear a table half as large).
// Eight instances a thread, 40 KB of LDS and so half the wavefronts: 262 us.
__global__ __launch_bounds__(256) void unique_vertex_kernel(const float* __restrict__ xyz, const int32_t* __restrict__ keys,
                                                            int64_t n, uint64_t* table, uint32_t mask, float* out,
                                                            int64_t cap, unsigned long long* count, int* err)
{
    __shared__ unsigned long long set[kVertSet];
    __shared__ uint16_t first[kVertPerWg], won[kVertPerWg];  // instances of the workgroup
    __shared__ uint32_t n_first, n_won;
    __shared__ unsigned long long base;
    for (uint32_t i = threadIdx.x; i < kVertSet; i += 256u) set[i] = kKeyEmpty;
    if (threadIdx.x == 0) n_first = n_won = 0u;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * kVertPerWg;
    bool bad = false;
    uint64_t mine[kVertPerThread];
#pragma unroll
    for (int k = 0; k < kVertPerThread; ++k) {
        const int64_t i = i0 + threadIdx.x + 256 * k;
        mine[k] = i < n ? vertex_key(keys + 4 * i, bad) : kKeyEmpty;
    }
#pragma unroll
    for (int k = 0; k < kVertPerThread; ++k) {
        const int e = (int)threadIdx.x + 256 * k;
        const uint64_t key = mine[k];
        if (key != kKeyEmpty) {
            uint32_t h = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 32) & (kVertSet - 1u);
            // fewer instances than entries: the probe ends
            for (;;) {
                const unsigned long long old = atomicCAS(&set[h], (unsigned long long)kKeyEmpty, (unsigned long long)key);
                if (old == kKeyEmpty) first[atomicAdd(&n_first, 1u)] = (uint16_t)e;
                if (old == kKeyEmpty || old == key) break;
                h = (h + 1u) & (kVertSet - 1u);
            }
        }
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < n_first; j += 256u) {
        const uint16_t e = first[j];
        bool seen = false;
        const uint64_t key = vertex_key(keys + 4 * (i0 + e), seen);
        uint32_t h = vertex_bucket(key) & mask;
        for (uint32_t probe = 0; probe <= mask; ++probe) {
            uint64_t old = table[h];
            if (old == kKeyEmpty)
                old = atomicCAS((unsigned long long*)(table + h), (unsigned long long)kKeyEmpty, (unsigned long long)key);
            if (old == kKeyEmpty) won[atomicAdd(&n_won, 1u)] = e;
            if (old == kKeyEmpty || old == key) break;
            h = (h + 1) & mask;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) base = atomicAdd(count, (unsigned long long)n_won);
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < 3u * n_won; j += 256u) {
        const uint64_t pos = base + j / 3u;
        if ((int64_t)pos < cap) out[3 * pos + j % 3u] = xyz[3 * (i0 + won[j / 3u]) + j % 3u];
    }
    if (bad) atomicOr(err, 1);
}

// ---------------------------------------------------------------------------
// capped nearest-neighbour distances over a uniform grid of cells of edge
// radius (1 + 2^-6): a point within the radius of a query lies in one of the
// 27 cells around the query's cell (the margin absorbs the rounding of the
// FP32 cell coordinate while |x| / radius stays below about 10^5)
//
// The cells are found by hashing, a cell's key, first point and count in one
// 16-byte entry (one load a probe), the points sorted by cell as 16 bytes
// each.  Build: every point finds or inserts its cell and takes its rank in
// it (lanes of a wavefront in one cell share one atomic; coherent clouds put
// tens of points in a row into a cell), the inserted cells, listed, get their
// ranges, and the points are stored at range + rank.
// ---------------------------------------------------------------------------

struct NnCell {
    unsigned long long key;  // kKeyEmpty = free
    uint32_t off, cnt;       // points [off, off + cnt) of `pts`
};

struct NnGrid {
    NnCell* cells;
    float4* pts;       // reference points sorted by cell (x, y, z, -)
    uint32_t* list;    // slots of the occupied cells
    uint32_t* counts;  // [0] listed cells, [32] points given a range (its own line)
    uint32_t mask;
    float inv;         // 1 / cell edge
    float edge;
};

__device__ inline int nn_cell(float x, float inv)
{
    const float c = floorf(x * inv);
    return (int)fminf(fmaxf(c, -1.0e6f), 1.0e6f);
}

__global__ __launch_bounds__(256) void nn_clear_kernel(NnGrid g)
{
    const uint64_t n = (uint64_t)g.mask + 1;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        reinterpret_cast<uint4*>(g.cells)[i] = make_uint4(~0u, ~0u, 0u, 0u);
    if (blockIdx.x == 0 && threadIdx.x < 2) g.counts[32 * threadIdx.x] = 0u;
}

constexpr int kNnPer = 8;  // points per thread: one reservation in the cell list per 2048

// Slot and rank of every point.  Bound: the latency of the probes and of one
// atomic a round.
__global__ __launch_bounds__(256) void nn_count_kernel(const float* __restrict__ ref, int64_t n, NnGrid g,
                                                       uint2* slot_rank)
{
    __shared__ uint32_t fresh[256 * kNnPer];
    __shared__ uint32_t n_fresh, base;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) n_fresh = 0u;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * (256 * kNnPer) + threadIdx.x;
    for (int k = 0; k < kNnPer; ++k) {
        const int64_t i = i0 + 256 * k;
        const bool have = i < n;
        uint32_t h = ~0u;
        if (have) {
            const int cx = nn_cell(ref[3 * i], g.inv), cy = nn_cell(ref[3 * i + 1], g.inv),
                      cz = nn_cell(ref[3 * i + 2], g.inv);
            const uint64_t key = pack_key(cx, cy, cz);
            h = hash_block(cx, cy, cz) & g.mask;
            // at least as many slots as points: the probe ends
            for (uint32_t probe = 0; probe <= g.mask; ++probe) {
                // entries only go from free to a key, so a plain read that finds the key is reliable
                const uint64_t seen = g.cells[h].key;
                if (seen == key) break;
                if (seen == kKeyEmpty) {
                    const uint64_t old = atomicCAS(&g.cells[h].key, (unsigned long long)kKeyEmpty,
                                                   (unsigned long long)key);
                    if (old == kKeyEmpty) {
                        fresh[atomicAdd(&n_fresh, 1u)] = h;
                        break;
                    }
                    if (old == key) break;
                }
                h = (h + 1) & g.mask;
            }
        }
        // lanes of one cell: the lowest one adds them all, each takes its place among them
        uint32_t rank = 0u, total = 0u;
        int leader = lane;
        uint64_t todo = __ballot(have);
        while (todo) {
            const int l = __ffsll((unsigned long long)todo) - 1;
            const uint64_t same = __ballot(h == (uint32_t)__builtin_amdgcn_readlane(h, l));
            if (h == (uint32_t)__builtin_amdgcn_readlane(h, l)) {
                rank = lanes_below(same);
                total = (uint32_t)__popcll(same);
                leader = l;
            }
            todo &= ~same;
        }
        uint32_t first = 0u;
        if (have && lane == leader) first = atomicAdd(&g.cells[h].cnt, total);
        first = (uint32_t)__shfl((int)first, leader);
        if (have) slot_rank[i] = make_uint2(h, first + rank);
    }
    __syncthreads();
    if (threadIdx.x == 0) base = n_fresh ? atomicAdd(g.counts, n_fresh) : 0u;
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < n_fresh; j += blockDim.x) g.list[base + j] = fresh[j];
}

// Ranges of the listed cells: a workgroup scans 256 counts and reserves their
// range with one atomic (the ranges need not be in cell order).
__global__ __launch_bounds__(256) void nn_offset_kernel(NnGrid g)
{
    __shared__ uint32_t part[4];
    __shared__ uint32_t base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t n = g.counts[0];
    for (uint32_t j0 = blockIdx.x * 256u; j0 < n; j0 += gridDim.x * 256u) {
        const uint32_t j = j0 + threadIdx.x;
        const uint32_t h = j < n ? g.list[j] : 0u;
        const uint32_t c = j < n ? g.cells[h].cnt : 0u;
        uint32_t incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o);
            incl += (lane >= o) ? y : 0u;
        }
        if (lane == 63) part[wave] = incl;
        __syncthreads();
        if (threadIdx.x == 0) base = atomicAdd(g.counts + 32, part[0] + part[1] + part[2] + part[3]);
        __syncthreads();
        uint32_t off = base + incl - c;
        for (int w = 0; w < wave; ++w) off += part[w];
        if (j < n) g.cells[h].off = off;
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void nn_scatter_kernel(const float* __restrict__ ref, int64_t n, NnGrid g,
                                                         const uint2* __restrict__ slot_rank)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint2 s = slot_rank[i];
    g.pts[g.cells[s.x].off + s.y] = make_float4(ref[3 * i], ref[3 * i + 1], ref[3 * i + 2], 0.0f);
}

// The 27 cells, the query's own first, then those sharing a face, an edge, a
// corner: d + 1 along each axis, two bits a cell, and the cells with each d.
struct NnOrder {
    uint64_t d[3];
    uint32_t mask[3][3];
};
constexpr NnOrder nn_order()
{
    NnOrder o{};
    int n = 0;
    for (int away = 0; away <= 3; ++away)
        for (int z = 0; z < 3; ++z)
            for (int y = 0; y < 3; ++y)
                for (int x = 0; x < 3; ++x)
                    if ((x != 1) + (y != 1) + (z != 1) == away) {
                        o.d[0] |= (uint64_t)x << (2 * n);
                        o.d[1] |= (uint64_t)y << (2 * n);
                        o.d[2] |= (uint64_t)z << (2 * n);
                        o.mask[0][x] |= 1u << n;
                        o.mask[1][y] |= 1u << n;
                        o.mask[2][z] |= 1u << n;
                        ++n;
                    }
    return o;
}
constexpr NnOrder kNnOrder = nn_order();

// Points of cell (cx, cy, cz): [a, e).
__device__ inline void nn_range(const NnGrid& g, int cx, int cy, int cz, uint32_t& a, uint32_t& e)
{
    const uint64_t key = pack_key(cx, cy, cz);
    uint32_t h = hash_block(cx, cy, cz) & g.mask;
    a = e = 0u;
    for (uint32_t probe = 0; probe <= g.mask; ++probe) {
        const uint4 w = reinterpret_cast<const uint4*>(g.cells)[h];
        const uint64_t k = ((uint64_t)w.y << 32) | w.x;
        if (k == key) {
            a = w.z;
            e = w.z + w.w;
        }
        if (k == key || k == kKeyEmpty) break;
        h = (h + 1) & g.mask;
    }
}

// kNnLanes lanes per query, which take a cell's points in turn.  The query's
// own cell comes first; another cell is looked up only when its box is nearer
// than the best distance so far (and the radius), which leaves one or two of
// the 27 for a query near the surface.  Each query walks its own set of them,
// so that a wavefront takes as many rounds as its longest set and not one for
// each cell that some query needs.  The box distance is taken low by 2^-21 of
// the coordinate and the edge, more than the roundings of the cell coordinate
// and of the products here, so that a cell holding a nearer point is never
// left out and the minimum is that over all 27 cells.  Bound: the vector ALU,
// the rounds that only some of the queries need.  1.0 M random queries against
// 2.0 M vertices and the reverse, radius five voxels: 2036 us a call with every
// cell read, in three 4-byte loads a point, 400 with the cells by their boxes,
// 288 with a set a query and two lanes (one lane 303, four 344).
// The distances' sum: per-workgroup partials in FP64, added by nn_sum_kernel
// (one atomic a wavefront on the sum had serialised).
constexpr int kNnLanes = 2;

// The minimum of a query's lanes, two neighbours.
__device__ inline float nn_group_min(float x)
{
    static_assert(kNnLanes == 2, "one exchange");
    return fminf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false)));
}

__global__ __launch_bounds__(256) void nn_query_kernel(const float* __restrict__ q, int64_t n, NnGrid g, bool empty,
                                                       float radius, float* dist, double* partial)
{
    __shared__ double part[4];
    const uint32_t sub = threadIdx.x & (kNnLanes - 1);
    double mine = 0.0;
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kNnLanes; i < n;
         i += (int64_t)gridDim.x * blockDim.x / kNnLanes) {
        const float x[3] = {q[3 * i], q[3 * i + 1], q[3 * i + 2]};
        float best = __builtin_inff();
        if (!empty) {
            int c[3];
            float lo[3], hi[3];  // squared distance to the cells below and above along each axis
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                c[r] = nn_cell(x[r], g.inv);
                const float m = 0x1p-21f * (fabsf(x[r]) + g.edge);
                const float a = fmaxf(x[r] - (float)c[r] * g.edge - m, 0.0f);
                const float b = fmaxf((float)(c[r] + 1) * g.edge - x[r] - m, 0.0f);
                lo[r] = a * a;
                hi[r] = b * b;
            }
            // nothing beyond the radius counts
            const float cap = radius * radius * (1.0f + 0x1p-16f);
            auto look = [&](int cx, int cy, int cz) {
                uint32_t a, e;
                nn_range(g, cx, cy, cz, a, e);
#pragma unroll 4
                for (uint32_t k = a + sub; k < e; k += kNnLanes) {
                    const float4 p = g.pts[k];
                    const float ex = x[0] - p.x;
                    const float ey = x[1] - p.y;
                    const float ez = x[2] - p.z;
                    best = fminf(best, (ex * ex + ey * ey) + ez * ez);
                }
                best = nn_group_min(best);  // a group's lanes are here together
            };
            look(c[0], c[1], c[2]);
            // the other cells, those out of reach along one axis left out at once
            constexpr float low = 1.0f - 0x1p-20f;
            const float reach = fminf(best, cap);
            uint32_t left = ~1u;
#pragma unroll
            for (int r = 0; r < 3; ++r)
                left &= (kNnOrder.mask[r][1] | (lo[r] * low > reach ? 0u : kNnOrder.mask[r][0])) |
                        (hi[r] * low > reach ? 0u : kNnOrder.mask[r][2]);
            while (left != 0u) {
                const int j = __ffs((int)left) - 1;
                left &= left - 1u;
                int d[3];
                float away = 0.0f;
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const uint32_t w = j < 16 ? (uint32_t)kNnOrder.d[r] : (uint32_t)(kNnOrder.d[r] >> 32);
                    d[r] = (int)((w >> ((2 * j) & 31)) & 3u) - 1;
                    away += d[r] < 0 ? lo[r] : d[r] > 0 ? hi[r] : 0.0f;
                }
                if (away * low > fminf(best, cap)) continue;
                look(c[0] + d[0], c[1] + d[1], c[2] + d[2]);
            }
        }
        const float d = fminf(sqrtf(best), radius);
        if (sub == 0u) {
            if (dist) dist[i] = d;
            mine += (double)d;
        }
    }
    if (partial) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mine;
        __syncthreads();
        if (threadIdx.x == 0) partial[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
    }
}

// The partials' sum, by one workgroup.
__global__ __launch_bounds__(1024) void nn_sum_kernel(const double* __restrict__ partial, int64_t n, double* sum)
{
    __shared__ double part[16];
    double mine = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) mine += partial[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < 16; ++w) s += part[w];
        *sum = s;
    }
}

static uint32_t pow2_at_least(uint64_t x)
{
    uint32_t p = 1024;
    while (p < x && p < (1u << 30)) p <<= 1;
    return p;
}

}  // namespace sc

using namespace sc;

extern "C" {

sc_status sc_mesh_table(uint8_t* loops, uint8_t* ntri)
{
    if (!loops && !ntri) return SC_EINVAL;
    McTable T;
    if (!mc_build(T)) return SC_EDEVICE;
    if (loops) memcpy(loops, T.loops, sizeof(T.loops));
    if (ntri) memcpy(ntri, T.ntri, sizeof(T.ntri));
    return SC_OK;
}

sc_status sc_volume_mesh(sc_volume* vol, void* stream, float* tri_xyz, int32_t* tri_keys, int64_t cap, int64_t* n_tri)
{
    if (!vol || cap < 0 || !n_tri) return SC_EINVAL;
    sc_status st = mc_table_ready();
    if (st != SC_OK) return st;
    int64_t nb = 0;
    st = sc_volume_query(vol, stream, &nb, nullptr);
    if (st != SC_OK) return st;
    *n_tri = 0;
    if (nb == 0) return SC_OK;
    hipStream_t s = (hipStream_t)stream;
    const uint32_t n = (uint32_t)nb;
    const uint32_t wgs = (n + kScanGroup - 1u) / kScanGroup;
    Scratch buf;
    uint32_t* counts = nullptr;
    uint64_t *offsets = nullptr, *sums = nullptr, *d_total = nullptr;
    for (int pass = 0; pass < 2; ++pass) {
        Carve c{buf.p};
        counts = c.take<uint32_t>(n);
        offsets = c.take<uint64_t>(n);
        sums = c.take<uint64_t>(wgs);
        d_total = c.take<uint64_t>(1);
        if (pass == 0) buf = scratch_take(c.off);
        if (!buf.p) return SC_ENOMEM;
    }
    uint64_t total = 0;
    MeshOut out{tri_xyz, tri_keys, counts, offsets, sums, cap};
    mesh_kernel<false><<<n, 64, 0, s>>>(vol->dev, out);
    scan_local_kernel<<<wgs, 256, 0, s>>>(counts, offsets, sums, n);
    scan_sums_kernel<<<1, 256, 0, s>>>(sums, wgs, d_total);
    if (cap > 0 && (tri_xyz || tri_keys)) mesh_kernel<true><<<n, 64, 0, s>>>(vol->dev, out);
    bool ok = hipGetLastError() == hipSuccess;
    ok = ok && hipMemcpyAsync(&total, d_total, sizeof(total), hipMemcpyDeviceToHost, s) == hipSuccess;
    ok = ok && hipStreamSynchronize(s) == hipSuccess;
    scratch_give(buf, ok);
    if (!ok) return SC_EDEVICE;
    *n_tri = (int64_t)total;
    return SC_OK;
}

sc_status sc_mesh_vertices(const float* tri_xyz, const int32_t* tri_keys, int64_t n_tri, float* vert_xyz, int64_t cap,
                           int64_t* n_vert, void* stream)
{
    if (n_tri < 0 || cap < 0 || !n_vert || (n_tri > 0 && (!tri_xyz || !tri_keys)) || (cap > 0 && !vert_xyz) ||
        n_tri > ((int64_t)1 << 28))
        return SC_EINVAL;
    *n_vert = 0;
    if (n_tri == 0) return SC_OK;
    hipStream_t s = (hipStream_t)stream;
    const int64_t nv = 3 * n_tri;
    // at most three quarters full where every instance is a vertex of its own; a mesh fills about a sixth of that
    const uint32_t slots = pow2_at_least((uint64_t)(nv + nv / 3));
    Scratch buf;
    uint64_t* table = nullptr;
    unsigned long long* d_count = nullptr;  // the count, then the error word
    for (int pass = 0; pass < 2; ++pass) {
        Carve c{buf.p};
        table = c.take<uint64_t>(slots);
        d_count = c.take<unsigned long long>(2);
        if (pass == 0) buf = scratch_take(c.off);
        if (!buf.p) return SC_ENOMEM;
    }
    unsigned long long got[2] = {0, 0};
    fill_u64(table, kKeyEmpty, slots, s);
    fill_u64(reinterpret_cast<uint64_t*>(d_count), 0ull, 2, s);
    unique_vertex_kernel<<<(unsigned)((nv + kVertPerWg - 1) / kVertPerWg), 256, 0, s>>>(
        tri_xyz, tri_keys, nv, table, slots - 1, vert_xyz, cap, d_count, reinterpret_cast<int*>(d_count + 1));
    bool ok = hipGetLastError() == hipSuccess;
    ok = ok && hipMemcpyAsync(got, d_count, sizeof(got), hipMemcpyDeviceToHost, s) == hipSuccess;
    ok = ok && hipStreamSynchronize(s) == hipSuccess;
    scratch_give(buf, ok);
    if (!ok) return SC_EDEVICE;
    if (got[1]) return SC_ERANGE;
    *n_vert = (int64_t)got[0];
    return SC_OK;
}

sc_status sc_nn_distance(const float* ref, int64_t n_ref, const float* query, int64_t n_query, float radius,
                         float* dist, double* sum, void* stream)
{
    if (n_ref < 0 || n_query < 0 || (n_ref > 0 && !ref) || (n_query > 0 && !query) || !(radius > 0.0f) ||
        !(radius < 1.0e30f) || n_ref > ((int64_t)1 << 29) || n_query > ((int64_t)1 << 31))
        return SC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    if (n_query == 0) {
        if (sum) fill_u64(reinterpret_cast<uint64_t*>(sum), 0ull, 1, s);
        return hipStreamSynchronize(s) == hipSuccess ? SC_OK : SC_EDEVICE;
    }
    NnGrid g{};
    g.edge = radius * (1.0f + 1.0f / 64.0f);
    g.inv = 1.0f / g.edge;
    const uint32_t slots = pow2_at_least((uint64_t)(2 * std::max<int64_t>(n_ref, 1)));
    g.mask = slots - 1;
    const int64_t wgs = std::min<int64_t>((n_query * kNnLanes + 255) / 256, 1 << 22);
    Scratch buf;
    uint2* slot_rank = nullptr;
    double* partial = nullptr;
    for (int pass = 0; pass < 2; ++pass) {
        Carve c{buf.p};
        partial = c.take<double>(sum ? (size_t)wgs : 1);
        if (n_ref > 0) {
            g.cells = c.take<NnCell>(slots);
            g.pts = c.take<float4>((size_t)n_ref);
            slot_rank = c.take<uint2>((size_t)n_ref);
            g.list = c.take<uint32_t>((size_t)n_ref);
            g.counts = c.take<uint32_t>(64);
        }
        if (pass == 0) buf = scratch_take(c.off);
        if (!buf.p) return SC_ENOMEM;
    }
    if (n_ref > 0) {
        nn_clear_kernel<<<(unsigned)std::min<uint32_t>(slots / 256, 4096), 256, 0, s>>>(g);
        nn_count_kernel<<<(unsigned)((n_ref + 256 * kNnPer - 1) / (256 * kNnPer)), 256, 0, s>>>(ref, n_ref, g,
                                                                                               slot_rank);
        nn_offset_kernel<<<(unsigned)std::min<int64_t>((n_ref + 255) / 256, 1024), 256, 0, s>>>(g);
        nn_scatter_kernel<<<(unsigned)((n_ref + 255) / 256), 256, 0, s>>>(ref, n_ref, g, slot_rank);
    }
    nn_query_kernel<<<(unsigned)wgs, 256, 0, s>>>(query, n_query, g, n_ref == 0, radius, dist, sum ? partial : nullptr);
    if (sum) nn_sum_kernel<<<1, 1024, 0, s>>>(partial, wgs, sum);
    bool ok = hipGetLastError() == hipSuccess;
    ok = ok && hipStreamSynchronize(s) == hipSuccess;
    scratch_give(buf, ok);
    return ok ? SC_OK : SC_EDEVICE;
}

}  // extern "C"
