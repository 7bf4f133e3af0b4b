// Keyframe fusion (Sec. 3, "Keyframe Fusion"; Eq. 1).
//
//   depth_weight   w_z = cos(theta) Z^-2 per pixel, quantised to 2^-10, with
//                  rejection near depth discontinuities
//   warp_kernel    forward warp of every surviving pixel into the keyframe,
//                  p* = g(T*^-1, g(T_i, pi^-1(x, Z_i(x)))), accumulated at the
//                  nearest pixel of pi(p*) in exact int64 fixed point (w on the
//                  2^-10 grid, z on the 2^-20 m grid), so that colliding
//                  atomics cannot change a bit; Eq. 1's running weighted mean
//                  equals sum(w z) / sum(w)
//   color_prep     unsharp mask C + (C - G * C), G the binomial [1 4 6 4 1]/16
//                  kernel, exact in units of 1/256, and the re-blur measure's
//                  integer luminance sums (exact int64 per-tile partials)
//   blur_final     per-frame sums of the partials and w_b (inside the warp
//                  launch when fusing)
//   color_kernel   the keyframe depth and weight from the accumulators, then
//                  the back-warp of each keyframe pixel into every frame,
//                  bilinear sample of the sharpened colour, weight w_b * w_z,
//                  per-channel lower weighted median
//
// A fusion is three launches: colour prep and depth weight together (which
// also clears the accumulators and stores the relative poses, passed to it as
// arguments), warp (which also forms w_b from the colour-prep partials) and
// colour.
//
// Decisions are FP32 with the written operation order (-ffp-contract=off).
#include <string.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "internal.hpp"
#include "kernels.hpp"

namespace sc {

constexpr int kMaxFrames = 64;

struct FuseFrames {
    float Rf[kMaxFrames][12];  // forward: T*^-1 T_i, rows of R then t
    float Rb[kMaxFrames][12];  // backward: T_i^-1 T*
    const float* Z[kMaxFrames];    // depth, H x W
    const uint8_t* C[kMaxFrames];  // colour, H x W x 3
};

// Relative poses and images passed by value, kStageFrames frames per launch, so
// that no host staging buffer or copy is needed.
constexpr int kStageFrames = 32;
struct PoseChunk {
    float Rf[kStageFrames][12];
    float Rb[kStageFrames][12];
    const float* Z[kStageFrames];
    const uint8_t* C[kStageFrames];
};

// Source tiles (16 x 16 pixels of a frame) by the keyframe tile that their
// samples land near: up to `cap` items f << 20 | tile a keyframe tile, the
// others in `over` (room for every source tile).
struct WarpBins {
    uint32_t* count;  // per keyframe tile, then the length of `over`
    uint32_t* items;
    uint32_t* over;
    int32_t cap, tiles_x, tiles;
};

// Work of one fusion done beside the colour prep and the depth weight: frame
// 0's depth tiles clear the fixed-point accumulators of their pixels, and the
// first one stores the first `count` relative poses and images.
struct FuseInit {
    unsigned long long* acc;  // KW then KZ, 2 x H W
    FuseFrames* fr;
    // the first frame's images where the others follow them (n x H x W), else
    // null: an address from the table waits for a load of its own
    const float* Z0;
    const uint8_t* C0;
    WarpBins bins;  // emptied, if there are any
    int32_t count;
    PoseChunk poses;
};

// A frame's images: their addresses come from memory, so that the compiler has
// to be told that they are global ones.
typedef __attribute__((address_space(1))) const float FrameDepth;
typedef __attribute__((address_space(1))) const uint8_t FrameColor;

// An address that is the same in every lane, in scalar registers: a load that
// brings it is then waited for once and not before each load through it.
template <class T>
__device__ inline const T* uniform(const T* p)
{
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return (const T*)(((uint64_t)hi << 32) | lo);
}

__device__ inline bool zvalid(float z, float zmin, float zmax) { return z >= zmin && z <= zmax; }

__device__ inline void backproject(float u, float v, float z, const sc_intrinsics& in, float P[3])
{
    P[0] = ((u - in.cx) * z) / in.fx;
    P[1] = ((v - in.cy) * z) / in.fy;
    P[2] = z;
}

__device__ inline void xform(const float* T, const float P[3], float q[3])
{
#pragma unroll
    for (int r = 0; r < 3; ++r) q[r] = ((T[3 * r + 0] * P[0] + T[3 * r + 1] * P[1]) + T[3 * r + 2] * P[2]) + T[9 + r];
}

__device__ inline bool project(const sc_intrinsics& in, const float q[3], float& uf, float& vf, int& iu, int& iv)
{
    if (!(q[2] > 0.0f)) return false;
    uf = (in.fx * q[0]) / q[2] + in.cx;
    vf = (in.fy * q[1]) / q[2] + in.cy;
    const float fu = floorf(uf + 0.5f), fv = floorf(vf + 0.5f);
    if (!(fu >= 0.0f && fu <= (float)(in.width - 1) && fv >= 0.0f && fv <= (float)(in.height - 1))) return false;
    iu = (int)fu;
    iv = (int)fv;
    return true;
}

// project's pixel alone: the coordinate's rounding test on a one-ulp
// reciprocal (pixel_coord_fast), the correctly rounded division only near a
// rounding boundary.  The same pixels for depths below 2^43 m, where the depth
// sums' integers end.
__device__ inline bool project_pixel(const sc_intrinsics& in, const float q[3], int& iu, int& iv)
{
    if (!(q[2] > 0.0f)) return false;
    const float r = __builtin_amdgcn_rcpf(q[2]);
    const float wl = (float)(in.width - 1), hl = (float)(in.height - 1);
    const float fu = pixel_coord_fast(in.fx * q[0], q[2], r, in.cx, wl);
    const float fv = pixel_coord_fast(in.fy * q[1], q[2], r, in.cy, hl);
    if (!(fu >= 0.0f && fu <= wl && fv >= 0.0f && fv <= hl)) return false;
    iu = (int)fu;
    iv = (int)fv;
    return true;
}

// One frame's tile partials (4 exact int64 sums per tile) added up by a
// 256-thread workgroup, then w_b = 1 - max(blur_h, blur_v) in FP64 (the
// integer sums are exact, so the order of the additions does not matter).
__device__ inline void blur_reduce(const long long* p, int tiles, long long (*red)[4], double* wb)
{
    long long acc[4] = {0, 0, 0, 0};
    for (int t = threadIdx.x; t < tiles; t += blockDim.x)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += p[(size_t)t * 4 + k];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();  // `red` may still be read from the caller's own reduction
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) red[wave][k] = acc[k];
    __syncthreads();
    if (threadIdx.x == 0) {
        long long s[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
        const double bh = s[0] > 0 ? (double)(s[0] - s[1]) / (double)s[0] : 0.0;
        const double bv = s[2] > 0 ? (double)(s[2] - s[3]) / (double)s[2] : 0.0;
        *wb = 1.0 - (bh > bv ? bh : bv);
    }
}

// ---------------------------------------------------------------------------
// depth weight
// ---------------------------------------------------------------------------

// One 64 x 16 tile per workgroup: the back-projection of every pixel of the
// tile and a one-pixel halo is computed once into LDS (two divisions per
// pixel), and each pixel reads its four neighbours' points from there; the
// operations are those of the per-pixel definition, so the result is the
// same bit for bit.
constexpr int kDwTW = 64, kDwTH = 16;
constexpr int kDwLW = kDwTW + 2, kDwLH = kDwTH + 2;
constexpr int kDwStage = (kDwLW * kDwLH + 255) / 256;  // staged pixels per thread (256 threads)

struct DwLds {
    float x[kDwLH][kDwLW], y[kDwLH][kDwLW], z[kDwLH][kDwLW];
};

// Tile `tile` of frame f (depth Zf); `acc` (or null): the accumulators that frame 0's
// tiles clear.
__device__ inline void depth_weight_tile(FrameDepth* __restrict__ Zf, int f, int tile, const sc_intrinsics& in,
                                         const sc_fuse_params& p, int tiles_x, float* __restrict__ wz,
                                         unsigned long long* acc, DwLds& lds)
{
    auto& sx = lds.x;
    auto& sy = lds.y;
    auto& sz = lds.z;
    const int W = in.width, H = in.height;
    const int64_t np = (int64_t)W * H;
    const int u0 = (tile % tiles_x) * kDwTW, v0 = (tile / tiles_x) * kDwTH;
    // staging: every depth load of a thread issues before the divisions
    float zs[kDwStage];
#pragma unroll
    for (int k = 0; k < kDwStage; ++k) {
        const int q = (int)threadIdx.x + 256 * k;
        const int uu = u0 - 1 + q % kDwLW, vv = v0 - 1 + q / kDwLW;
        zs[k] = (q < kDwLW * kDwLH && uu >= 0 && uu < W && vv >= 0 && vv < H) ? Zf[(size_t)vv * W + uu] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < kDwStage; ++k) {
        const int q = (int)threadIdx.x + 256 * k;
        if (q < kDwLW * kDwLH) {
            const int i = q % kDwLW, j = q / kDwLW;
            const int uu = u0 - 1 + i, vv = v0 - 1 + j;
            float P[3] = {0.0f, 0.0f, 0.0f};
            if (uu >= 0 && uu < W && vv >= 0 && vv < H) backproject((float)uu, (float)vv, zs[k], in, P);
            sx[j][i] = P[0];
            sy[j][i] = P[1];
            sz[j][i] = P[2];
        }
    }
    __syncthreads();
    const int tx = threadIdx.x & (kDwTW - 1), ty = threadIdx.x / kDwTW;
    const int u = u0 + tx, i = tx + 1;
#pragma unroll 1
    for (int r = 0; r < kDwTH / 4; ++r) {
        const int v = v0 + ty + 4 * r, j = ty + 4 * r + 1;
        if (u >= W || v >= H) continue;
        float out = 0.0f;
        const float z = sz[j][i];
        if (zvalid(z, p.z_min, p.z_max) && u >= 1 && u <= W - 2 && v >= 1 && v <= H - 2) {
            const float zl = sz[j][i - 1], zr = sz[j][i + 1], zu = sz[j - 1][i], zd = sz[j + 1][i];
            const bool ok = zvalid(zl, p.z_min, p.z_max) && zvalid(zr, p.z_min, p.z_max) &&
                            zvalid(zu, p.z_min, p.z_max) && zvalid(zd, p.z_min, p.z_max);
            const float th = p.disc_rel * z;
            if (ok && !(fabsf(zl - z) > th) && !(fabsf(zr - z) > th) && !(fabsf(zu - z) > th) &&
                !(fabsf(zd - z) > th)) {
                // neighbours (u - 1, v), (u + 1, v), (u, v - 1), (u, v + 1)
                const float a0 = sx[j][i + 1] - sx[j][i - 1], a1 = sy[j][i + 1] - sy[j][i - 1], a2 = zr - zl;
                const float b0 = sx[j + 1][i] - sx[j - 1][i], b1 = sy[j + 1][i] - sy[j - 1][i], b2 = zd - zu;
                const float nx = a1 * b2 - a2 * b1;
                const float ny = a2 * b0 - a0 * b2;
                const float nz = a0 * b1 - a1 * b0;
                const float nn = (nx * nx + ny * ny) + nz * nz;
                if (nn > 0.0f) {
                    const float c = fabsf(nz) / sqrtf(nn);
                    const float w = c / (z * z);
                    out = rintf(w * kWeightScale) / kWeightScale;
                }
            }
        }
        wz[(size_t)f * np + (size_t)v * W + u] = out;
        if (acc && f == 0) {
            acc[(size_t)v * W + u] = 0ull;
            acc[np + (size_t)v * W + u] = 0ull;
        }
    }
}

__global__ __launch_bounds__(256) void depth_weight_kernel(const float* __restrict__ Z, int n, sc_intrinsics in,
                                                           sc_fuse_params p, int tiles_x, int tiles,
                                                           float* __restrict__ wz)
{
    __shared__ DwLds lds;
    const int f = blockIdx.y, tile = blockIdx.x;
    if (f >= n || tile >= tiles) return;
    depth_weight_tile((FrameDepth*)(Z + (size_t)f * in.width * in.height), f, tile, in, p, tiles_x, wz, nullptr, lds);
}

// ---------------------------------------------------------------------------
// depth fusion
// ---------------------------------------------------------------------------

// The warp by target tiles.  Workgroup k owns the 16 x 16 tile k of
// keyframe pixels (on a grid extended by kWpE tiles on each side) and, for
// each frame f, the source tile k shifted back by that frame's displacement
// d_f: the image centre back-projected at depth z_nom, moved into the
// keyframe and projected, rounded to whole pixels and clamped to +-kWpD.
// Every workgroup computes the same d_f, and a whole-pixel shift of the tile
// grid still covers each frame's pixels exactly once, so every sample is
// warped once whatever d_f is; d_f only decides how many land near the
// tile.  The samples are first added into an LDS window of keyframe pixels
// (the tile and kWpM pixels on each side); each window pixel that received
// any then goes to the device-wide accumulators with one pair of atomics,
// and samples that land outside the window go there directly.  The sums are
// exact integers, so the grouping does not change them.  The first n
// workgroups add up the frames' colour-prep partials instead.
constexpr int kWpT = 16, kWpM = 8, kWpL = kWpT + 2 * kWpM;
constexpr int kWpE = 4, kWpD = kWpE * kWpT;

__global__ __launch_bounds__(256) void warp_kernel(const float* __restrict__ wz, int n,
                                                   sc_intrinsics in, float z_nom, int tiles_x,
                                                   const FuseFrames* __restrict__ fr, unsigned long long* KW,
                                                   unsigned long long* KZ, const long long* __restrict__ parts,
                                                   int prep_tiles, double* wb)
{
    if ((int)blockIdx.x < n) {  // the frame's w_b, for the colour kernel
        __shared__ long long red[4][4];
        blur_reduce(parts + (size_t)blockIdx.x * prep_tiles * 4, prep_tiles, red, wb + blockIdx.x);
        return;
    }
    const int tile = (int)blockIdx.x - n;
    __shared__ unsigned long long lw[kWpL * kWpL], lz[kWpL * kWpL];
    __shared__ int2 shift[kMaxFrames];
    const int W = in.width, H = in.height;
    const int64_t np = (int64_t)W * H;
    for (int e = threadIdx.x; e < kWpL * kWpL; e += blockDim.x) {
        lw[e] = 0ull;
        lz[e] = 0ull;
    }
    if ((int)threadIdx.x < n) {
        const float cu = (float)(W / 2), cv = (float)(H / 2);
        float P[3], q[3];
        backproject(cu, cv, z_nom, in, P);
        xform(fr->Rf[threadIdx.x], P, q);
        int2 d = make_int2(0, 0);
        if (q[2] > 0.0f) {
            const float du = rintf((in.fx * q[0]) / q[2] + in.cx - cu);
            const float dv = rintf((in.fy * q[1]) / q[2] + in.cy - cv);
            // (a NaN compares false and leaves 0)
            if (fabsf(du) <= (float)kWpD) d.x = (int)du;
            else if (du > 0.0f) d.x = kWpD;
            else if (du < 0.0f) d.x = -kWpD;
            if (fabsf(dv) <= (float)kWpD) d.y = (int)dv;
            else if (dv > 0.0f) d.y = kWpD;
            else if (dv < 0.0f) d.y = -kWpD;
        }
        shift[threadIdx.x] = d;
    }
    __syncthreads();
    const int ku = (tile % tiles_x - kWpE) * kWpT, kv = (tile / tiles_x - kWpE) * kWpT;
    const int wx0 = ku - kWpM, wy0 = kv - kWpM;
    const int tx = (int)threadIdx.x & (kWpT - 1), ty = (int)threadIdx.x / kWpT;
    // frames in groups of kWpF: every load of a group issues before its samples are warped
    constexpr int kWpF = 4;
    for (int f0 = 0; f0 < n; f0 += kWpF) {
        float wg[kWpF], zg[kWpF];
#pragma unroll
        for (int j = 0; j < kWpF; ++j) {
            wg[j] = 0.0f;
            zg[j] = 0.0f;
            const int f = f0 + j;
            if (f < n) {
                const int2 d = shift[f];
                const int u = ku + tx - d.x, v = kv + ty - d.y;
                if (u >= 0 && u < W && v >= 0 && v < H) {
                    const size_t pix = (size_t)v * W + u;
                    wg[j] = wz[(size_t)f * np + pix];
                    zg[j] = ((FrameDepth*)fr->Z[f])[pix];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kWpF; ++j) {
            const int f = f0 + j;
            const float w = wg[j];
            if (!(w > 0.0f)) continue;  // also frames past n and pixels outside the image
            const int2 d = shift[f];
            const int u = ku + tx - d.x, v = kv + ty - d.y;
            float P[3], q[3];
            backproject((float)u, (float)v, zg[j], in, P);
            xform(fr->Rf[f], P, q);
            float uf, vf;
            int iu, iv;
            if (!project(in, q, uf, vf, iu, iv)) continue;
            const long long wk = (long long)rintf(w * kWeightScale);
            const long long zk = (long long)rintf(q[2] * 1048576.0f);
            const int lx = iu - wx0, ly = iv - wy0;
            if ((unsigned)lx < (unsigned)kWpL && (unsigned)ly < (unsigned)kWpL) {
                atomicAdd(&lw[ly * kWpL + lx], (unsigned long long)wk);
                atomicAdd(&lz[ly * kWpL + lx], (unsigned long long)(wk * zk));
            } else {
                const int64_t t = (int64_t)iv * W + iu;
                atomicAdd(KW + t, (unsigned long long)wk);
                atomicAdd(KZ + t, (unsigned long long)(wk * zk));
            }
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kWpL * kWpL; e += blockDim.x) {
        const unsigned long long a = lw[e];
        if (a != 0ull) {
            // only samples inside the image were added, so the pixel is too
            const int64_t t = (int64_t)(wy0 + e / kWpL) * W + (wx0 + e % kWpL);
            atomicAdd(KW + t, a);
            atomicAdd(KZ + t, lz[e]);
        }
    }
}

// The warp of groups of many frames.  The displacement of a frame's pixels
// follows their depths, and over many frames the camera moves far enough that
// one displacement a frame leaves most samples outside the windows (60 frames
// of a turning camera: 64 % of them, 160 of warp_kernel's 242 us in their
// atomics).  Here each 16 x 16 source tile of a frame goes by its own: a thread
// a source tile takes the depth at its centre (or at the first of four other
// pixels that has one), moves that point into the keyframe and appends the
// tile to the list of the keyframe tile it lands in (the nearest one up to a
// tile outside the image, its own place from there on, which spreads them).
// The assignment only decides where samples are added up.
__global__ __launch_bounds__(256) void warp_bin_kernel(int n, sc_intrinsics in, sc_fuse_params p,
                                                       const FuseFrames* __restrict__ fr, WarpBins b)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i >= n * b.tiles) return;
    const int f = i / b.tiles, tile = i - f * b.tiles;
    const int u0 = (tile % b.tiles_x) * 16, v0 = (tile / b.tiles_x) * 16;
    FrameDepth* Z = (FrameDepth*)fr->Z[f];
    int u[5], v[5];
    float z[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        u[k] = min(u0 + (k == 0 ? 8 : (k & 1) ? 3 : 12), in.width - 1);
        v[k] = min(v0 + (k == 0 ? 8 : (k & 2) ? 3 : 12), in.height - 1);
        z[k] = Z[(size_t)v[k] * in.width + u[k]];
    }
    float us = (float)u[0], vs = (float)v[0], zs = 0.5f * (p.z_min + p.z_max);
#pragma unroll
    for (int k = 4; k >= 0; --k)
        if (zvalid(z[k], p.z_min, p.z_max)) {
            us = (float)u[k];
            vs = (float)v[k];
            zs = z[k];
        }
    float P[3], q[3];
    backproject(us, vs, zs, in, P);
    xform(fr->Rf[f], P, q);
    int bx = u0 / 16, by = v0 / 16;
    if (q[2] > 0.0f) {
        const float x = (in.fx * q[0]) / q[2] + in.cx, y = (in.fy * q[1]) / q[2] + in.cy;
        if (x > -16.0f && x < (float)in.width + 16.0f && y > -16.0f && y < (float)in.height + 16.0f) {
            bx = (int)fminf(fmaxf(x, 0.0f), (float)(in.width - 1)) / 16;
            by = (int)fminf(fmaxf(y, 0.0f), (float)(in.height - 1)) / 16;
        }
    }
    const uint32_t item = (uint32_t)f << 20 | (uint32_t)tile;
    const int bin = by * b.tiles_x + bx;
    const uint32_t at = atomicAdd(b.count + bin, 1u);
    if (at < (uint32_t)b.cap) b.items[(size_t)bin * b.cap + at] = item;
    else b.over[atomicAdd(b.count + b.tiles, 1u)] = item;
}

// Workgroups [0, n): the frames' w_b, as in warp_kernel; then one a keyframe
// tile, which adds its list's samples into its LDS window and those outside the
// window to memory; then kWpOver for the source tiles beyond the lists, whose
// samples all go to memory.
// Bound: the vector ALU and the loads' latency, four source tiles at a time.
// 60 frames of 640x480: 0.9 % of the samples outside the windows, 110 us with
// warp_bin_kernel's 13 (242 us by a displacement a frame).
constexpr int kWpOver = 64;

static int warp_tiles(int W, int H) { return ((W + 15) / 16) * ((H + 15) / 16); }

// Whether n frames of W x H pixels are warped by their source tiles.  It costs
// a launch and one pass over the frames' tiles, and leaves a workgroup a
// keyframe tile, so few tiles in all or too few keyframe tiles for the CUs go
// by a displacement a frame.  Whole fusions of a room scan and of a turning
// camera, by displacements / by tiles: 640x480 9 frames 117 / 127 and 109 / 115
// us, 12 frames 132 / 142 and 127 / 127, 13 frames 142 / 149 and 138 / 134, 32
// frames 327 / 267 and 278 / 237; 1280x960 8 frames 266 / 258 and 241 / 220, 9
// frames 338 / 321 and 309 / 279 (with 8 at most the colours take another way);
// 320x240 (300 tiles) 16 frames 82 / 95 and 86 / 95, 64 frames 201 / 238 and
// 184 / 213.
static bool warp_by_tiles(int n, int W, int H)
{
    const int tiles = warp_tiles(W, H);
    return n > 8 && tiles >= 600 && (int64_t)n * tiles > 12 * 1200;
}

__global__ __launch_bounds__(256) void warp_bins_kernel(const float* __restrict__ wz, int n, sc_intrinsics in,
                                                        const FuseFrames* __restrict__ fr, unsigned long long* KW,
                                                        unsigned long long* KZ, const long long* __restrict__ parts,
                                                        int prep_tiles, double* wb, WarpBins b)
{
    __shared__ unsigned long long lw[kWpL * kWpL], lz[kWpL * kWpL];
    __shared__ uint32_t items[2 * kMaxFrames];
    if ((int)blockIdx.x < n) {
        __shared__ long long red[4][4];
        blur_reduce(parts + (size_t)blockIdx.x * prep_tiles * 4, prep_tiles, red, wb + blockIdx.x);
        return;
    }
    const int W = in.width, H = in.height;
    const size_t np = (size_t)W * H;
    const int tx = (int)threadIdx.x & 15, ty = (int)threadIdx.x >> 4;
    // this thread's sample of a source tile
    auto load = [&](uint32_t item, float& w, float& z) {
        const int f = (int)(item >> 20), tile = (int)(item & 0xFFFFFu);
        const int u = (tile % b.tiles_x) * 16 + tx, v = (tile / b.tiles_x) * 16 + ty;
        w = z = 0.0f;
        if (u < W && v < H) {
            const uint32_t pix = (uint32_t)(v * W + u);
            w = wz[f * np + pix];
            z = ((FrameDepth*)fr->Z[f])[pix];
        }
    };
    auto warp = [&](uint32_t item, float w, float z, int& iu, int& iv, long long& wk, long long& zk) {
        const int f = (int)(item >> 20), tile = (int)(item & 0xFFFFFu);
        float P[3], q[3];
        backproject((float)((tile % b.tiles_x) * 16 + tx), (float)((tile / b.tiles_x) * 16 + ty), z, in, P);
        xform(fr->Rf[f], P, q);
        wk = (long long)rintf(w * kWeightScale);
        zk = (long long)rintf(q[2] * 1048576.0f);
        return project_pixel(in, q, iu, iv);
    };
    auto add = [&](int iu, int iv, long long wk, long long zk) {
        const size_t t = (size_t)iv * W + iu;
        atomicAdd(KW + t, (unsigned long long)wk);
        atomicAdd(KZ + t, (unsigned long long)(wk * zk));
    };
    const int bin = (int)blockIdx.x - n;
    if (bin >= b.tiles) {
        const uint32_t m = b.count[b.tiles];
        for (uint32_t i = (uint32_t)(bin - b.tiles); i < m; i += kWpOver) {
            const uint32_t item = __builtin_amdgcn_readfirstlane(b.over[i]);
            float w, z;
            load(item, w, z);
            if (!(w > 0.0f)) continue;
            int iu, iv;
            long long wk, zk;
            if (warp(item, w, z, iu, iv, wk, zk)) add(iu, iv, wk, zk);
        }
        return;
    }
    const int m = (int)min(b.count[bin], (uint32_t)b.cap);
    if (m == 0) return;
    for (int e = threadIdx.x; e < m; e += blockDim.x) items[e] = b.items[(size_t)bin * b.cap + e];
    for (int e = threadIdx.x; e < kWpL * kWpL; e += blockDim.x) {
        lw[e] = 0ull;
        lz[e] = 0ull;
    }
    __syncthreads();
    const int wx0 = (bin % b.tiles_x) * 16 - kWpM, wy0 = (bin / b.tiles_x) * 16 - kWpM;
    constexpr int kWpF = 4;
    for (int i0 = 0; i0 < m; i0 += kWpF) {
        float wg[kWpF], zg[kWpF];
        uint32_t it[kWpF];
#pragma unroll
        for (int j = 0; j < kWpF; ++j) {
            it[j] = __builtin_amdgcn_readfirstlane(items[min(i0 + j, m - 1)]);
            load(it[j], wg[j], zg[j]);
            if (i0 + j >= m) wg[j] = 0.0f;
        }
#pragma unroll
        for (int j = 0; j < kWpF; ++j) {
            if (!(wg[j] > 0.0f)) continue;
            int iu, iv;
            long long wk, zk;
            if (!warp(it[j], wg[j], zg[j], iu, iv, wk, zk)) continue;
            const int lx = iu - wx0, ly = iv - wy0;
            if ((unsigned)lx < (unsigned)kWpL && (unsigned)ly < (unsigned)kWpL) {
                atomicAdd(&lw[ly * kWpL + lx], (unsigned long long)wk);
                atomicAdd(&lz[ly * kWpL + lx], (unsigned long long)(wk * zk));
            } else {
                add(iu, iv, wk, zk);
            }
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kWpL * kWpL; e += blockDim.x) {
        const unsigned long long a = lw[e];
        if (a != 0ull) {
            // only samples inside the image were added, so the pixel is too
            const int64_t t = (int64_t)(wy0 + e / kWpL) * W + (wx0 + e % kWpL);
            atomicAdd(KW + t, a);
            atomicAdd(KZ + t, lz[e]);
        }
    }
}

// ---------------------------------------------------------------------------
// colour pre-processing
// ---------------------------------------------------------------------------

__device__ inline int clampi(int a, int lo, int hi) { return a < lo ? lo : (a > hi ? hi : a); }

__device__ inline int luma(uint32_t px) { return (77 * (int)(px & 255u) + 150 * (int)((px >> 8) & 255u) + 29 * (int)(px >> 16) + 128) >> 8; }

// Colour pre-processing of one 64 x 16 tile of one frame.  The tile and a
// halo (2 pixels for the 5-tap binomial, 5 before and 4 after for the 9-tap
// re-blur box) are staged in LDS with coordinates clamped to the image, which
// is the edge rule of both filters.  The binomial runs separably on pixels
// packed as R | G << 16 and B: every channel's weighted sum stays below
// 16 * 16 * 255 < 2^16, so the 16-bit lanes never carry into each other and
// the sums are the per-channel integers.  Bound by the vector ALU: 60 frames
// of 640x480 with their depth weights took 178 us with a 64-bit word a pixel
// and 64-bit re-blur sums, now 164.  Each thread then produces four
// pixels of the unsharp mask and adds their re-blur terms to four integer
// sums, reduced over the workgroup and stored as the tile's partial sums (no
// atomics).
//   sums k = 0..3: sF_h, sV_h, sF_v, sV_v, the 9x-scaled horizontal and
//   vertical variation of the frame and of its re-blurred copy (the box
//   difference telescopes to two samples).
constexpr int kPrepTW = 64, kPrepTH = 16;
constexpr int kPrepLW = kPrepTW + 9, kPrepLH = kPrepTH + 9;
constexpr int kPrepHalo = 5;
constexpr int kPrepStage = (kPrepLW * kPrepLH + 255) / 256;  // staged pixels per thread (256 threads)

struct PrepLds {
    uint2 pix[kPrepLH][kPrepLW];
    uint2 hsum[kPrepTH + 4][kPrepTW];  // horizontal binomial of staged rows 3 .. 22
    uint8_t lum[kPrepLH][kPrepLW];  // luma <= 255; bytes keep the workgroup under 26.7 KB of LDS (six per CU)
    int red[4][4];
};

// a + 4 b + 6 c + 4 d + e in both words.
__device__ inline uint2 binomial(uint2 a, uint2 b, uint2 c, uint2 d, uint2 e)
{
    auto sum = [](uint32_t a0, uint32_t b0, uint32_t c0, uint32_t d0, uint32_t e0) {
        return (a0 + e0) + ((b0 + d0) << 2) + (c0 << 2) + (c0 << 1);
    };
    return make_uint2(sum(a.x, b.x, c.x, d.x, e.x), sum(a.y, b.y, c.y, d.y, e.y));
}

// kOutCh: 3 (packed RGB, the standalone output) or 4 (RGB and a zero, one
// 8-byte store per pixel; the layout the colour kernel gathers from).
template <int kOutCh>
__device__ inline void color_prep_tile(FrameColor* __restrict__ C, int f, int tile, int W, int H, int tiles_x,
                                       int tiles, uint16_t* __restrict__ out, long long* __restrict__ parts,
                                       PrepLds& lds)
{
    auto& pix = lds.pix;
    auto& hsum = lds.hsum;
    auto& lum = lds.lum;
    auto& red = lds.red;
    const int u0 = (tile % tiles_x) * kPrepTW, v0 = (tile / tiles_x) * kPrepTH;
    const int64_t np = (int64_t)W * H;
    // staging: every load of a thread issues before its first LDS store
    uint32_t st[kPrepStage];
#pragma unroll
    for (int k = 0; k < kPrepStage; ++k) {
        const int p = (int)threadIdx.x + 256 * k;
        st[k] = 0u;
        if (p < kPrepLW * kPrepLH) {
            const int i = p % kPrepLW, j = p / kPrepLW;
            const int uu = clampi(u0 - kPrepHalo + i, 0, W - 1), vv = clampi(v0 - kPrepHalo + j, 0, H - 1);
            FrameColor* q = C + 3 * ((size_t)vv * W + uu);
            st[k] = (uint32_t)q[0] | ((uint32_t)q[1] << 8) | ((uint32_t)q[2] << 16);
        }
    }
#pragma unroll
    for (int k = 0; k < kPrepStage; ++k) {
        const int p = (int)threadIdx.x + 256 * k;
        if (p < kPrepLW * kPrepLH) {
            const int i = p % kPrepLW, j = p / kPrepLW;
            const uint32_t px = st[k];
            pix[j][i] = make_uint2((px & 255u) | ((px << 8) & 0xFF0000u), px >> 16);
            lum[j][i] = (uint8_t)luma(px);
        }
    }
    __syncthreads();
    for (int p = threadIdx.x; p < (kPrepTH + 4) * kPrepTW; p += blockDim.x) {
        const int c = p % kPrepTW, jr = p / kPrepTW;
        const uint2* row = &pix[jr + kPrepHalo - 2][c + kPrepHalo - 2];
        hsum[jr][c] = binomial(row[0], row[1], row[2], row[3], row[4]);
    }
    __syncthreads();
    const int tx = threadIdx.x & (kPrepTW - 1), ty = threadIdx.x / kPrepTW;
    // at most 9 * 255 a pixel, 1,024 pixels a tile: 32 bits
    int acc[4] = {0, 0, 0, 0};
    const int u = u0 + tx, i = tx + kPrepHalo;
#pragma unroll 1
    for (int r = 0; r < kPrepTH / 4; ++r) {
        const int y = ty + 4 * r, v = v0 + y, j = y + kPrepHalo;
        if (u >= W || v >= H) continue;
        // staged row j + b is hsum row y + 2 + b
        const uint2 S = binomial(hsum[y][tx], hsum[y + 1][tx], hsum[y + 2][tx], hsum[y + 3][tx], hsum[y + 4][tx]);
        const uint2 c0 = pix[j][i];
        const uint32_t sh[3] = {(uint32_t)clampi((int)((c0.x & 0xFFFFu) << 9) - (int)(S.x & 0xFFFFu), 0, 65280),
                                (uint32_t)clampi((int)((c0.x >> 16) << 9) - (int)(S.x >> 16), 0, 65280),
                                (uint32_t)clampi((int)(c0.y << 9) - (int)S.y, 0, 65280)};
        const size_t px = (size_t)f * np + (size_t)v * W + u;
        if (kOutCh == 4) {
            *reinterpret_cast<uint2*>(out + 4 * px) = make_uint2(sh[0] | (sh[1] << 16), sh[2]);
        } else {
            uint16_t* o = out + 3 * px;
            o[0] = (uint16_t)sh[0];
            o[1] = (uint16_t)sh[1];
            o[2] = (uint16_t)sh[2];
        }
        const int y0 = lum[j][i];
        if (u >= 1) {
            const int dF = 9 * abs(y0 - lum[j][i - 1]);
            const int dB = abs(lum[j][i + 4] - lum[j][i - 5]);
            acc[0] += dF;
            acc[1] += max(dF - dB, 0);
        }
        if (v >= 1) {
            const int dF = 9 * abs(y0 - lum[j - 1][i]);
            const int dB = abs(lum[j + 4][i] - lum[j - 5][i]);
            acc[2] += dF;
            acc[3] += max(dF - dB, 0);
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) red[wave][k] = acc[k];
    __syncthreads();
    if (threadIdx.x < 4) {
        const int k = threadIdx.x;
        parts[((size_t)f * tiles + tile) * 4 + k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
    }
}

__global__ __launch_bounds__(256) void color_prep_kernel(const uint8_t* __restrict__ rgb, int n, int W, int H,
                                                         int tiles_x, int tiles, uint16_t* __restrict__ out,
                                                         long long* __restrict__ parts)
{
    __shared__ PrepLds lds;
    const int f = blockIdx.y, tile = blockIdx.x;
    if (f >= n || tile >= tiles) return;
    color_prep_tile<3>((FrameColor*)(rgb + (size_t)f * W * H * 3), f, tile, W, H, tiles_x, tiles, out, parts, lds);
}

// A fusion's colour prep (four channels) and depth weight in one launch: of a
// frame's workgroups the first prep_tiles take the colour tiles, the others
// the depth tiles.  Neither needs the other, and each alone waits for its loads with the
// CUs half empty at its end: 640x480, 5 frames 16.2 + 11.5 us in two launches,
// now 21 in one; 60 frames 104 + 72 us, now 164.
__global__ __launch_bounds__(256) void fuse_front_kernel(sc_intrinsics in, sc_fuse_params p, int prep_x,
                                                         int prep_tiles, int dw_x,
                                                         uint16_t* __restrict__ cs, long long* __restrict__ parts,
                                                         float* __restrict__ wz, const FuseInit init)
{
    __shared__ union {
        PrepLds prep;
        DwLds dw;
    } lds;
    const int f = blockIdx.y;
    if ((int)blockIdx.x < prep_tiles) {
        const uint8_t* C = init.C0 ? init.C0 + (size_t)f * in.width * in.height * 3
                                   : f < init.count ? init.poses.C[f] : init.fr->C[f];
        color_prep_tile<4>((FrameColor*)uniform(C), f, blockIdx.x, in.width, in.height, prep_x, prep_tiles, cs, parts, lds.prep);
        return;
    }
    const int tile = (int)blockIdx.x - prep_tiles;
    if (f == 0 && tile == 0) {
        for (int i = threadIdx.x; i < init.count * 12; i += blockDim.x) {
            init.fr->Rf[i / 12][i % 12] = init.poses.Rf[i / 12][i % 12];
            init.fr->Rb[i / 12][i % 12] = init.poses.Rb[i / 12][i % 12];
        }
        for (int i = threadIdx.x; i < init.count; i += blockDim.x) init.fr->Z[i] = init.poses.Z[i];
    }
    if (f == 0 && init.bins.count && threadIdx.x < 5) {
        // the tile's four keyframe tiles (64 x 16 pixels), and the overflow's length
        const int bx = 4 * (tile % dw_x) + (int)threadIdx.x, by = tile / dw_x;
        if (threadIdx.x < 4 && bx < init.bins.tiles_x) init.bins.count[by * init.bins.tiles_x + bx] = 0u;
        if (threadIdx.x == 4 && tile == 0) init.bins.count[init.bins.tiles] = 0u;
    }
    const float* Z = init.Z0 ? init.Z0 + (size_t)f * in.width * in.height
                             : f < init.count ? init.poses.Z[f] : init.fr->Z[f];
    depth_weight_tile((FrameDepth*)uniform(Z), f, tile, in, p, dw_x, wz, init.acc, lds.dw);
}

// One workgroup per frame (standalone colour pre-processing).
__global__ __launch_bounds__(256) void blur_final_kernel(const long long* __restrict__ parts, int n, int tiles,
                                                         double* wb)
{
    __shared__ long long red[4][4];
    const int f = blockIdx.x;
    if (f >= n) return;
    blur_reduce(parts + (size_t)f * tiles * 4, tiles, red, wb + f);
}

// ---------------------------------------------------------------------------
// colour fusion
// ---------------------------------------------------------------------------

// The keyframe pixel's channel is the weighted median of its observations
// rounded to 8 bits.  Rounding is monotone, so that is the weighted median of
// the rounded observations, and of observations equal after rounding any will
// do: an observation is four bytes (three 8-bit channels) and its weight on
// the 2^-20 grid, and the median the smallest value up to which the weights
// reach half their total.
//
// Up to eight frames (N = their number) a wavefront takes 64 consecutive
// keyframe pixels through everything, a lane a pixel: its depth from the
// fixed-point accumulators (W* = sum(w), Z* = sum(w z) / sum(w), rounded once
// to FP32), the back-warp into each frame, whose lanes read neighbouring
// pixels, and the median from the observations' sums of weights at or below
// each, all in registers.  With more frames the eight wavefronts of a
// workgroup share the 64 pixels: each takes every eighth frame, the
// observations meet in LDS by frame, and a wavefront takes a channel's median
// by a bisection of the 256 values.
// Bound: the vector ALU (about 150 instructions a pixel and frame).  One thread
// a (pixel, frame), its frame's neighbours in other workgroups and n
// comparisons of (value, frame) each with 64-bit sums: 640x480, 5 frames 20.4
// us, 60 frames 611 us, now 14 and 132 us (5 frames through LDS, every
// wavefront forming the depths: 17.3).
constexpr int kColorWaves = 8;

// Keyframe pixel idx: its point (and Z*) and W*; W* = 0 without depth.
__device__ inline float color_point(const unsigned long long* __restrict__ KW,
                                    const unsigned long long* __restrict__ KZ, int idx, const sc_intrinsics& in,
                                    float P[3])
{
    P[0] = P[1] = P[2] = 0.0f;
    // np <= 16384^2 < 2^31: pixel indices and their division in 32 bits
    const long long kw = idx < in.width * in.height ? (long long)KW[idx] : 0ll;
    if (kw <= 0) return 0.0f;
    const int v = idx / in.width, u = idx - v * in.width;
    const float zk = (float)(((double)(long long)KZ[idx] / (double)kw) * 0x1p-20);
    backproject((float)u, (float)v, zk, in, P);
    return (float)((double)kw / 1024.0);
}

// Frame i's observation of point P: 8-bit channels and weight (0: none).
__device__ inline uint2 color_observe(const float* __restrict__ wz,
                                      const uint16_t* __restrict__ cs, const double* __restrict__ wb, int i,
                                      const sc_intrinsics& in, float occ_rel, const FuseFrames* __restrict__ fr,
                                      bool live, const float P[3])
{
    const int W = in.width, H = in.height;
    uint2 o = make_uint2(0u, 0u);
    float q[3], uf, vf;
    int iu, iv;
    xform(fr->Rb[i], P, q);
    if (!live || !project(in, q, uf, vf, iu, iv)) return o;
    const float x0 = floorf(uf), y0 = floorf(vf);
    if (!(x0 >= 0.0f && x0 + 1.0f <= (float)(W - 1) && y0 >= 0.0f && y0 + 1.0f <= (float)(H - 1))) return o;
    const size_t base = (size_t)i * (W * H);
    const float wzi = wz[base + (size_t)iv * W + iu];
    const float zi = ((FrameDepth*)fr->Z[i])[(size_t)iv * W + iu];
    const float ax = uf - x0, ay = vf - y0;
    const int ix = (int)x0, iy = (int)y0;
    // four channels of 16 bits per pixel, 8-byte aligned
    const uint2* C0 = reinterpret_cast<const uint2*>(cs) + base + (size_t)iy * W + ix;
    const uint2* C1 = C0 + W;
    const uint2 p00 = C0[0], p10 = C0[1], p01 = C1[0], p11 = C1[1];
    const float wcs = rintf(((float)wb[i] * wzi) * 1048576.0f);
    if (!(wzi > 0.0f && fabsf(zi - q[2]) <= occ_rel * q[2] && wcs > 0.0f)) return o;
    auto ch = [](uint2 p, int k) {
        return (float)(k == 0 ? (p.x & 0xFFFFu) : k == 1 ? (p.x >> 16) : (p.y & 0xFFFFu));
    };
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float c00 = ch(p00, k), c10 = ch(p10, k);
        const float c01 = ch(p01, k), c11 = ch(p11, k);
        const float top = c00 + ax * (c10 - c00);
        const float bot = c01 + ax * (c11 - c01);
        const float val = rintf((top + ay * (bot - top)) / 256.0f);
        o.x |= (uint32_t)fminf(fmaxf(val, 0.0f), 255.0f) << (8 * k);
    }
    o.y = (uint32_t)wcs;
    return o;
}

__device__ inline void color_store(int idx, bool any, float w, float z, uint32_t rgb, float* Zs, float* Ws,
                                   uint8_t* rgba)
{
    Ws[idx] = any ? w : 0.0f;
    Zs[idx] = any ? z : 0.0f;
    const uint32_t c = any ? rgb | 0xFF000000u : 0u;
    if (((uintptr_t)rgba & 3u) == 0u) {
        reinterpret_cast<uint32_t*>(rgba)[idx] = c;
    } else {
        for (int k = 0; k < 4; ++k) rgba[4 * (size_t)idx + k] = (uint8_t)(c >> (8 * k));
    }
}

// Channel `sh` of N observations, its sums in T.
template <int N, class T>
__device__ inline uint32_t median_regs(const uint2 (&o)[N], int sh, T total)
{
    uint32_t best = 255u;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t v = (o[i].x >> sh) & 255u;
        T s = 0;
#pragma unroll
        for (int l = 0; l < N; ++l) s += ((o[l].x >> sh) & 255u) <= v ? o[l].y : 0u;
        if (2 * s >= total) best = min(best, v);
    }
    return best;
}

template <int N>
__global__ __launch_bounds__(256) void color_kernel(const float* __restrict__ wz,
                                                    const uint16_t* __restrict__ cs, const double* __restrict__ wb,
                                                    sc_intrinsics in, float occ_rel,
                                                    const FuseFrames* __restrict__ fr,
                                                    const unsigned long long* __restrict__ KW,
                                                    const unsigned long long* __restrict__ KZ, float* Zs, float* Ws,
                                                    uint8_t* rgba)
{
    const int idx = (int)(blockIdx.x * 256 + threadIdx.x);
    float P[3];
    const float w = color_point(KW, KZ, idx, in, P);
    uint2 o[N];
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = color_observe(wz, cs, wb, i, in, occ_rel, fr, w > 0.0f, P);
    uint64_t total = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) total += o[i].y;
    // the total bounds every sum: in 32 bits where twice it fits
    uint32_t rgb = 0u;
    const bool small = __ballot(total >= (1ull << 31)) == 0ull;
#pragma unroll
    for (int sh = 0; sh < 24; sh += 8)
        rgb |= (small ? median_regs<N, uint32_t>(o, sh, (uint32_t)total) : median_regs<N, uint64_t>(o, sh, total))
               << sh;
    if (idx < in.width * in.height) color_store(idx, total != 0, w, P[2], rgb, Zs, Ws, rgba);
}

// Channel `sh` of the n observations in LDS, its sums in T.
template <class T>
__device__ inline uint32_t median_lds(const uint2* obs, int n, int lane, int sh, T total)
{
    uint32_t lo = 0u, hi = 255u;
#pragma unroll 1
    for (int step = 0; step < 8; ++step) {
        const uint32_t mid = (lo + hi) >> 1;
        T s = 0;
#pragma unroll 4
        for (int l = 0; l < n; ++l) {
            const uint2 o = obs[l * 64 + lane];
            s += ((o.x >> sh) & 255u) <= mid ? o.y : 0u;
        }
        const bool up = 2 * s >= total;
        hi = up ? mid : hi;
        lo = up ? lo : mid + 1u;
    }
    return hi;
}

__global__ __launch_bounds__(64 * kColorWaves) void color_many_kernel(
    const float* __restrict__ wz, const uint16_t* __restrict__ cs,
    const double* __restrict__ wb, int n, sc_intrinsics in, float occ_rel, const FuseFrames* __restrict__ fr,
    const unsigned long long* __restrict__ KW, const unsigned long long* __restrict__ KZ, float* Zs, float* Ws,
    uint8_t* rgba)
{
    extern __shared__ uint2 obs[];  // [frame][pixel]
    __shared__ uint8_t med[3][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int idx = (int)blockIdx.x * 64 + lane;
    float P[3];
    const float w = color_point(KW, KZ, idx, in, P);
    for (int i = wave; i < n; i += kColorWaves)
        obs[i * 64 + lane] = color_observe(wz, cs, wb, i, in, occ_rel, fr, w > 0.0f, P);
    __syncthreads();
    if (wave < 3) {
        uint64_t total = 0;
        for (int l = 0; l < n; ++l) total += obs[l * 64 + lane].y;
        med[wave][lane] =
            (uint8_t)(__ballot(total >= (1ull << 31)) == 0ull
                          ? median_lds<uint32_t>(obs, n, lane, 8 * wave, (uint32_t)total)
                          : median_lds<uint64_t>(obs, n, lane, 8 * wave, total));
    }
    __syncthreads();
    if (wave != 0 || idx >= in.width * in.height) return;
    bool any = false;  // some frame observed the pixel
    for (int l = 0; l < n; ++l) any = any || obs[l * 64 + lane].y != 0u;
    color_store(idx, any, w, P[2],
                (uint32_t)med[0][lane] | ((uint32_t)med[1][lane] << 8) | ((uint32_t)med[2][lane] << 16), Zs, Ws, rgba);
}

// ---------------------------------------------------------------------------
// workspace
// ---------------------------------------------------------------------------

struct FuseWs {
    std::mutex mu;
    int device = -1;
    size_t cap_px = 0, cap_frames = 0;
    float* wz = nullptr;
    uint16_t* cs = nullptr;
    unsigned long long* acc = nullptr;   // KW, KZ
    long long* parts = nullptr;          // 4 per colour-prep tile and frame
    size_t cap_parts = 0;
    uint32_t* bins = nullptr;            // source tiles by keyframe tile (bins_words), or null
    size_t cap_bins = 0;
    double* wb = nullptr;
    FuseFrames* d_fr = nullptr;
};

static FuseWs g_ws;

// Colour-prep tiles of one W x H frame.
static int prep_tiles_x(int W) { return (W + kPrepTW - 1) / kPrepTW; }
static int prep_tiles(int W, int H) { return prep_tiles_x(W) * ((H + kPrepTH - 1) / kPrepTH); }

// Words of tile lists of n frames of W x H pixels.
static size_t bins_words(int n, int W, int H)
{
    return warp_by_tiles(n, W, H) ? (size_t)warp_tiles(W, H) * (1 + 3 * (size_t)n) + 1 : 0;
}

// At least bins_words of every W x H <= px and n W H <= total (W, H >= 3,
// n <= kMaxFrames): a W x H image has at most (W + 15) (H + 15) / 256 tiles, W
// + H is at most W H / 3 + 3, so at most 6 W H / 256 + 2 tiles.
static size_t bins_bound(size_t px, size_t total)
{
    return (6 * px + 18 * total) / 256 + 6 * kMaxFrames + 4;
}

// np pixels per frame, frames frames, parts int64 colour-prep partials.  The
// tile lists come with the images, for whatever fits those, so that no later
// call allocates for them (one under capture cannot); without memory for them
// the warp goes without.
static sc_status ws_reserve(size_t np, size_t frames, size_t parts)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return SC_EDEVICE;
    if (g_ws.device != dev) {
        // a different device: start over (old buffers belong to another device)
        g_ws.cap_px = g_ws.cap_frames = 0;
        g_ws.wz = nullptr;
        g_ws.cs = nullptr;
        g_ws.acc = nullptr;
        g_ws.parts = nullptr;
        g_ws.cap_parts = 0;
        g_ws.bins = nullptr;
        g_ws.cap_bins = 0;
        g_ws.wb = nullptr;
        g_ws.d_fr = nullptr;
        g_ws.device = dev;
    }
    if (!g_ws.d_fr) {
        if (!device_alloc(&g_ws.d_fr, sizeof(FuseFrames))) return SC_ENOMEM;
        if (!device_alloc(&g_ws.wb, sizeof(double) * kMaxFrames)) return SC_ENOMEM;
    }
    if (np * frames > g_ws.cap_px * g_ws.cap_frames || np > g_ws.cap_px) {
        if (hipDeviceSynchronize() != hipSuccess) return SC_EDEVICE;
        (void)hipFree(g_ws.wz);
        (void)hipFree(g_ws.cs);
        (void)hipFree(g_ws.acc);
        const size_t px = std::max(np, g_ws.cap_px);
        const size_t fr = std::max(frames, g_ws.cap_frames);
        g_ws.wz = nullptr;
        g_ws.cs = nullptr;
        g_ws.acc = nullptr;
        g_ws.cap_px = g_ws.cap_frames = 0;
        if (!device_alloc(&g_ws.wz, sizeof(float) * px * fr)) return SC_ENOMEM;
        if (!device_alloc(&g_ws.cs, sizeof(uint16_t) * 4 * px * fr)) return SC_ENOMEM;
        if (!device_alloc(&g_ws.acc, sizeof(unsigned long long) * 2 * px)) return SC_ENOMEM;
        g_ws.cap_px = px;
        g_ws.cap_frames = fr;
        (void)hipFree(g_ws.bins);
        g_ws.bins = nullptr;
        g_ws.cap_bins = bins_bound(px, px * fr);
        if (!device_alloc(&g_ws.bins, sizeof(uint32_t) * g_ws.cap_bins)) {
            (void)hipGetLastError();
            g_ws.bins = nullptr;
            g_ws.cap_bins = 0;
        }
    }
    if (parts > g_ws.cap_parts) {
        if (hipDeviceSynchronize() != hipSuccess) return SC_EDEVICE;
        (void)hipFree(g_ws.parts);
        g_ws.parts = nullptr;
        g_ws.cap_parts = 0;
        if (!device_alloc(&g_ws.parts, sizeof(long long) * parts)) return SC_ENOMEM;
        g_ws.cap_parts = parts;
    }
    return SC_OK;
}

// Fusion parameters a fusion accepts: z_min at least 2^-5 m keeps every
// depth weight w_z <= 1 / z_min^2 at most 2^10, so a colour weight on the
// 2^-20 grid stays below 2^31 and fits the 32 bits it is held in.
static bool fuse_params_valid(const sc_fuse_params* p)
{
    return p && p->z_min >= 0x1p-5f && p->z_max >= p->z_min && p->z_max < 1e6f && p->disc_rel >= 0.0f &&
           p->occ_rel >= 0.0f;
}

static bool intr_valid(const sc_intrinsics* in)
{
    return in && in->width >= 3 && in->height >= 3 && in->fx > 0.0f && in->fy > 0.0f && in->width <= 16384 &&
           in->height <= 16384;
}

// Overlap counts (valid, visible) of one frame with a reference view, FP64
// in the written order; each thread counts kOverlapPix pixels, a workgroup
// reduces in LDS and adds its two totals with one atomic each.
struct OverlapArgs {
    double R[9], t[3], Rr[9], tr[3];
    double fx, fy, cx, cy;
    float z_min, z_max;
    int32_t width, height;
};

constexpr int kOverlapPix = 16;

__global__ void overlap_clear_kernel(uint32_t* counts)
{
    if (threadIdx.x < 2) counts[threadIdx.x] = 0u;
}

__global__ __launch_bounds__(256) void overlap_kernel(const float* __restrict__ depth, OverlapArgs a,
                                                      uint32_t* counts)
{
    __shared__ uint32_t red[2][256];
    const int64_t n = (int64_t)a.width * a.height;
    const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * kOverlapPix;
    uint32_t valid = 0u, visible = 0u;
    for (int k = 0; k < kOverlapPix; ++k) {
        const int64_t i = i0 + k;
        if (i >= n) break;
        const float zf = depth[i];
        if (!(zf >= a.z_min && zf <= a.z_max)) continue;
        ++valid;
        const int u = (int)(i % a.width), v = (int)(i / a.width);
        const double z = (double)zf;
        const double p[3] = {(((double)u - a.cx) / a.fx) * z, (((double)v - a.cy) / a.fy) * z, z};
        double w[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) w[r] = ((a.R[3 * r] * p[0] + a.R[3 * r + 1] * p[1]) + a.R[3 * r + 2] * p[2]) + a.t[r];
        const double d[3] = {w[0] - a.tr[0], w[1] - a.tr[1], w[2] - a.tr[2]};
        double q[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) q[c] = (a.Rr[c] * d[0] + a.Rr[3 + c] * d[1]) + a.Rr[6 + c] * d[2];
        if (q[2] > 0.0) {
            const double fu = floor(((a.fx * q[0]) / q[2] + a.cx) + 0.5);
            const double fv = floor(((a.fy * q[1]) / q[2] + a.cy) + 0.5);
            visible += (fu >= 0.0 && fu <= (double)(a.width - 1) && fv >= 0.0 && fv <= (double)(a.height - 1)) ? 1u : 0u;
        }
    }
    red[0][threadIdx.x] = valid;
    red[1][threadIdx.x] = visible;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < (unsigned)o) {
            red[0][threadIdx.x] += red[0][threadIdx.x + o];
            red[1][threadIdx.x] += red[1][threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (red[0][0]) atomicAdd(counts, red[0][0]);
        if (red[1][0]) atomicAdd(counts + 1, red[1][0]);
    }
}

static void rel_pose(const sc_pose& A, const sc_pose& B, float out[12])
{
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) {
            const double x = (A.R[0 * 3 + r] * B.R[0 * 3 + c] + A.R[1 * 3 + r] * B.R[1 * 3 + c]) + A.R[2 * 3 + r] * B.R[2 * 3 + c];
            out[3 * r + c] = (float)x;
        }
        const double y = (A.R[0 * 3 + r] * (B.t[0] - A.t[0]) + A.R[1 * 3 + r] * (B.t[1] - A.t[1])) +
                         A.R[2 * 3 + r] * (B.t[2] - A.t[2]);
        out[9 + r] = (float)y;
    }
}

static int dw_tiles_x(int W) { return (W + kDwTW - 1) / kDwTW; }
static int dw_tiles(int W, int H) { return dw_tiles_x(W) * ((H + kDwTH - 1) / kDwTH); }

// Relative poses and images of frames first .. first + count - 1 into the
// device table.
__global__ void stage_poses_kernel(PoseChunk c, int first, int count, FuseFrames* fr)
{
    for (int i = threadIdx.x; i < count * 12; i += blockDim.x) {
        fr->Rf[first + i / 12][i % 12] = c.Rf[i / 12][i % 12];
        fr->Rb[first + i / 12][i % 12] = c.Rb[i / 12][i % 12];
    }
    for (int i = threadIdx.x; i < count; i += blockDim.x) {
        fr->Z[first + i] = c.Z[i];
        fr->C[first + i] = c.C[i];
    }
}

// Device buffers of one fusion: per-frame weights, sharpened colour, the
// fixed-point accumulators, colour-prep partials, w_b and the relative poses.
struct FuseBufs {
    float* wz;
    uint16_t* cs;
    unsigned long long* acc;
    long long* parts;
    double* wb;
    FuseFrames* fr;
    uint32_t* bins;  // bins_words, or null
};

static WarpBins warp_bins(uint32_t* words, int n, const sc_intrinsics& in)
{
    WarpBins b;
    b.tiles_x = (in.width + 15) / 16;
    b.tiles = warp_tiles(in.width, in.height);
    b.cap = 2 * n;
    b.count = words;
    b.items = words + b.tiles + 1;
    b.over = b.items + (size_t)b.tiles * b.cap;
    return b;
}

// The fusion kernels of one keyframe.  The relative poses of the first
// kStageFrames frames travel in the first launch; those of later
// frames are stored by stage_poses_kernel launches enqueued first.
static void launch_fuse(const FuseBufs& b, const float* const* depth, const uint8_t* const* rgb, const sc_pose* poses,
                        int n_frames, int ref, const sc_intrinsics& in, const sc_fuse_params& params, float* kf_depth,
                        float* kf_weight, uint8_t* kf_rgba, hipStream_t s)
{
    const int64_t np = (int64_t)in.width * in.height;
    FuseInit init;
    init.acc = b.acc;
    init.fr = b.fr;
    const WarpBins bins = warp_by_tiles(n_frames, in.width, in.height) && b.bins ? warp_bins(b.bins, n_frames, in)
                                                                                : WarpBins{};
    init.bins = bins;
    init.Z0 = depth[0];
    init.C0 = rgb[0];
    for (int i = 1; i < n_frames; ++i) {
        if (depth[i] != depth[0] + i * np) init.Z0 = nullptr;
        if (rgb[i] != rgb[0] + i * np * 3) init.C0 = nullptr;
    }
    auto stage = [&](int i, int j) {
        rel_pose(poses[ref], poses[i], init.poses.Rf[j]);
        rel_pose(poses[i], poses[ref], init.poses.Rb[j]);
        init.poses.Z[j] = depth[i];
        init.poses.C[j] = rgb[i];
    };
    for (int i0 = kStageFrames; i0 < n_frames; i0 += kStageFrames) {
        const int cnt = std::min(kStageFrames, n_frames - i0);
        for (int j = 0; j < cnt; ++j) stage(i0 + j, j);
        stage_poses_kernel<<<1, 256, 0, s>>>(init.poses, i0, cnt, b.fr);
    }
    init.count = std::min(kStageFrames, n_frames);
    for (int j = 0; j < init.count; ++j) stage(j, j);
    const int pt = prep_tiles(in.width, in.height), dt = dw_tiles(in.width, in.height);
    fuse_front_kernel<<<dim3((unsigned)(pt + dt), (unsigned)n_frames), 256, 0, s>>>(
        in, params, prep_tiles_x(in.width), pt, dw_tiles_x(in.width), b.cs, b.parts, b.wz, init);
    if (bins.count) {
        warp_bin_kernel<<<(unsigned)(((int64_t)n_frames * bins.tiles + 255) / 256), 256, 0, s>>>(n_frames, in, params,
                                                                                                 b.fr, bins);
        warp_bins_kernel<<<(unsigned)(n_frames + bins.tiles + kWpOver), 256, 0, s>>>(
            b.wz, n_frames, in, b.fr, b.acc, b.acc + np, b.parts, pt, b.wb, bins);
    } else {
        // target tiles over the image and kWpE more on each side
        const int wtx = (in.width + kWpT - 1) / kWpT + 2 * kWpE, wty = (in.height + kWpT - 1) / kWpT + 2 * kWpE;
        const float z_nom = 0.5f * (params.z_min + params.z_max);
        warp_kernel<<<(unsigned)(n_frames + wtx * wty), 256, 0, s>>>(b.wz, n_frames, in, z_nom, wtx, b.fr, b.acc,
                                                                     b.acc + np, b.parts, pt, b.wb);
    }
    const unsigned long long *KW = b.acc, *KZ = b.acc + np;
    auto color = [&](auto n) {
        color_kernel<decltype(n)::value><<<(unsigned)((np + 255) / 256), 256, 0, s>>>(
            b.wz, b.cs, b.wb, in, params.occ_rel, b.fr, KW, KZ, kf_depth, kf_weight, kf_rgba);
    };
    switch (n_frames) {
    case 1: color(std::integral_constant<int, 1>{}); break;
    case 2: color(std::integral_constant<int, 2>{}); break;
    case 3: color(std::integral_constant<int, 3>{}); break;
    case 4: color(std::integral_constant<int, 4>{}); break;
    case 5: color(std::integral_constant<int, 5>{}); break;
    case 6: color(std::integral_constant<int, 6>{}); break;
    case 7: color(std::integral_constant<int, 7>{}); break;
    case 8: color(std::integral_constant<int, 8>{}); break;
    default:
        color_many_kernel<<<(unsigned)((np + 63) / 64), 64 * kColorWaves, sizeof(uint2) * 64 * (size_t)n_frames, s>>>(
            b.wz, b.cs, b.wb, n_frames, in, params.occ_rel, b.fr, KW, KZ, kf_depth, kf_weight, kf_rgba);
    }
}

// ---------------------------------------------------------------------------
// allocation-free fusion: every buffer in one fixed device array
// ---------------------------------------------------------------------------

// Scratch of kf_fuse_noalloc.  In host code `scratch` names a host-side
// stand-in, never device memory: its device address is looked up once per
// device with hipGetSymbolAddress and only that address is passed on.  Every
// call on a device shares that device's copy, so calls that overlap on one
// device race.
// 76 MiB for the images and 1 KiB for the frames' addresses decide what a call
// takes; the source tiles' lists (under a hundredth of the images of a call
// that large) come after them.
constexpr size_t kScratchImages = (size_t(76) << 20) + sizeof(FuseFrames::Z) + sizeof(FuseFrames::C);
constexpr size_t kScratchBytes = kScratchImages + (size_t(2) << 20);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static unsigned char* g_scratch_dev[kMaxDevices];

// The current device's address of `scratch`, looked up on the first call on
// that device (with the device current).
static sc_status scratch_address(unsigned char** out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SC_EDEVICE;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SC_EDEVICE;
        g_scratch_dev[dev] = static_cast<unsigned char*>(p);
    }
    *out = g_scratch_dev[dev];
    return SC_OK;
}

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Places the fusion buffers of np pixels x frames frames in one region
// starting at base (may be null to measure); returns the bytes used.
static size_t fuse_layout(unsigned char* base, size_t np, size_t frames, size_t parts, FuseBufs& b)
{
    size_t off = 0;
    auto take = [&](size_t bytes) {
        unsigned char* p = base ? base + off : nullptr;
        off = align256(off + bytes);
        return p;
    };
    b.fr = reinterpret_cast<FuseFrames*>(take(sizeof(FuseFrames)));
    b.wb = reinterpret_cast<double*>(take(sizeof(double) * kMaxFrames));
    b.acc = reinterpret_cast<unsigned long long*>(take(sizeof(unsigned long long) * 2 * np));
    b.parts = reinterpret_cast<long long*>(take(sizeof(long long) * parts));
    b.wz = reinterpret_cast<float*>(take(sizeof(float) * np * frames));
    b.cs = reinterpret_cast<uint16_t*>(take(sizeof(uint16_t) * 4 * np * frames));
    return off;
}

// The frames of n x H x W (x 3) arrays.
static bool frame_rows(const float* depth, const uint8_t* rgb, int n, const sc_intrinsics* in, const float** Z,
                       const uint8_t** C)
{
    if (!depth || !rgb || n <= 0 || n > kMaxFrames || !intr_valid(in)) return false;
    const size_t np = (size_t)in->width * in->height;
    for (int i = 0; i < n; ++i) {
        Z[i] = depth + i * np;
        C[i] = rgb + i * np * 3;
    }
    return true;
}

}  // namespace sc

using namespace sc;

extern "C" {

sc_status sc_depth_weight(const float* depth, int32_t n_frames, const sc_intrinsics* intr, const sc_fuse_params* params,
                          float* wz_out, void* stream)
{
    if (!depth || !wz_out || n_frames <= 0 || n_frames > 65535 || !intr_valid(intr) || !params) return SC_EINVAL;
    const int tiles = dw_tiles(intr->width, intr->height);
    depth_weight_kernel<<<dim3((unsigned)tiles, (unsigned)n_frames), 256, 0, (hipStream_t)stream>>>(
        depth, n_frames, *intr, *params, dw_tiles_x(intr->width), tiles, wz_out);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

sc_status sc_color_prep(const uint8_t* rgb, int32_t n_frames, int32_t width, int32_t height, uint16_t* sharp_out,
                        double* wb_out, void* stream)
{
    if (!rgb || !sharp_out || !wb_out || n_frames <= 0 || n_frames > kMaxFrames || width < 2 || height < 2 ||
        width > 16384 || height > 16384)
        return SC_EINVAL;
    std::lock_guard<std::mutex> lk(g_ws.mu);
    const sc_status st =
        ws_reserve((size_t)width * height, (size_t)n_frames, 4 * (size_t)prep_tiles(width, height) * n_frames);
    if (st != SC_OK) return st;
    const int tiles = prep_tiles(width, height);
    color_prep_kernel<<<dim3((unsigned)tiles, (unsigned)n_frames), 256, 0, (hipStream_t)stream>>>(
        rgb, n_frames, width, height, prep_tiles_x(width), tiles, sharp_out, g_ws.parts);
    blur_final_kernel<<<n_frames, 256, 0, (hipStream_t)stream>>>(g_ws.parts, n_frames, tiles, wb_out);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

sc_status kf_fuse_frames(const float* const* depth, const uint8_t* const* rgb, const sc_pose* poses, int32_t n_frames,
                         int32_t ref, const sc_intrinsics* intr, const sc_fuse_params* params, float* kf_depth,
                         float* kf_weight, uint8_t* kf_rgba, void* stream)
{
    if (!depth || !rgb || !poses || n_frames <= 0 || n_frames > kMaxFrames || ref < 0 || ref >= n_frames ||
        !intr_valid(intr) || !fuse_params_valid(params) || !kf_depth || !kf_weight || !kf_rgba)
        return SC_EINVAL;
    for (int i = 0; i < n_frames; ++i)
        if (!depth[i] || !rgb[i]) return SC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const sc_intrinsics in = *intr;
    const int64_t np = (int64_t)in.width * in.height;
    std::lock_guard<std::mutex> lk(g_ws.mu);
    sc_status st = ws_reserve((size_t)np, (size_t)n_frames, 4 * (size_t)prep_tiles(in.width, in.height) * n_frames);
    if (st != SC_OK) return st;
    uint32_t* bins = bins_words(n_frames, in.width, in.height) <= g_ws.cap_bins ? g_ws.bins : nullptr;
    const FuseBufs b{g_ws.wz, g_ws.cs, g_ws.acc, g_ws.parts, g_ws.wb, g_ws.d_fr, bins};
    launch_fuse(b, depth, rgb, poses, n_frames, ref, in, *params, kf_depth, kf_weight, kf_rgba, s);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

sc_status kf_fuse(const float* depth, const uint8_t* rgb, const sc_pose* poses, int32_t n_frames, int32_t ref,
                  const sc_intrinsics* intr, const sc_fuse_params* params, float* kf_depth, float* kf_weight,
                  uint8_t* kf_rgba, void* stream)
{
    const float* Z[kMaxFrames];
    const uint8_t* C[kMaxFrames];
    if (!frame_rows(depth, rgb, n_frames, intr, Z, C)) return SC_EINVAL;
    return kf_fuse_frames(Z, C, poses, n_frames, ref, intr, params, kf_depth, kf_weight, kf_rgba, stream);
}

sc_status kf_fuse_noalloc(const float* depth, const uint8_t* rgb, const sc_pose* poses, int32_t n_frames, int32_t ref,
                          const sc_intrinsics* intr, const sc_fuse_params* params, float* kf_depth, float* kf_weight,
                          uint8_t* kf_rgba, void* stream)
{
    const float* Z[kMaxFrames];
    const uint8_t* C[kMaxFrames];
    if (!frame_rows(depth, rgb, n_frames, intr, Z, C) || !poses || ref < 0 || ref >= n_frames ||
        !fuse_params_valid(params) || !kf_depth || !kf_weight || !kf_rgba)
        return SC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const sc_intrinsics in = *intr;
    const size_t np = (size_t)in.width * in.height;
    const size_t parts = 4 * (size_t)prep_tiles(in.width, in.height) * n_frames;
    FuseBufs b;
    size_t bytes = fuse_layout(nullptr, np, (size_t)n_frames, parts, b);
    if (bytes > kScratchImages) return SC_ESCRATCH;
    unsigned char* base = nullptr;
    const sc_status st = scratch_address(&base);
    if (st != SC_OK) return st;
    fuse_layout(base, np, (size_t)n_frames, parts, b);
    const size_t lists = sizeof(uint32_t) * bins_words(n_frames, in.width, in.height);
    b.bins = lists > 0 && bytes + lists <= kScratchBytes ? reinterpret_cast<uint32_t*>(base + bytes) : nullptr;
    launch_fuse(b, Z, C, poses, n_frames, ref, in, *params, kf_depth, kf_weight, kf_rgba, s);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

sc_status sc_overlap(const float* depth, const sc_intrinsics* intr, const sc_pose* T_frame, const sc_pose* T_ref,
                     float z_min, float z_max, uint32_t* counts, void* stream)
{
    if (!depth || !intr || !T_frame || !T_ref || !counts || intr->width <= 0 || intr->height <= 0 ||
        intr->width > 16384 || intr->height > 16384 || !(intr->fx > 0.0f) || !(intr->fy > 0.0f))
        return SC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    OverlapArgs a;
    memcpy(a.R, T_frame->R, sizeof(a.R));
    memcpy(a.t, T_frame->t, sizeof(a.t));
    memcpy(a.Rr, T_ref->R, sizeof(a.Rr));
    memcpy(a.tr, T_ref->t, sizeof(a.tr));
    a.fx = intr->fx;
    a.fy = intr->fy;
    a.cx = intr->cx;
    a.cy = intr->cy;
    a.z_min = z_min;
    a.z_max = z_max;
    a.width = intr->width;
    a.height = intr->height;
    overlap_clear_kernel<<<1, 64, 0, s>>>(counts);
    const int64_t n = (int64_t)intr->width * intr->height;
    const int64_t per_wg = 256 * kOverlapPix;
    overlap_kernel<<<(unsigned)((n + per_wg - 1) / per_wg), 256, 0, s>>>(depth, a, counts);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

}  // extern "C"
