// Adjoint of integration.  After integrating keyframes k at poses T_k into a
// field (running weighted average, Sec. 3; quantities of Sec. 4.3), every
// voxel holds D = (W0 D0 + sum_k w_k d_k) / W with d_k = Z_k(u_k) - p_z and
// W = W0 + sum_k w_k (the colour likewise).  With the pixel and band
// decisions held fixed:
//   dL/dZ_k(u)  = sum_{v -> u} (w_k / W) dL/dD(v)
//   dL/dC_k(u)  = sum_{v -> u} (w_k / W) dL/dC(v)
//   dL/dxi_k    = sum_v (w_k / W) dL/dD(v) (0, 0, 1, p_y, -p_x, 0)
//   dL/dD0(v)   = (W0 / W) dL/dD(v),   dL/dC0(v) = (W0 / W) dL/dC(v)
// for a right perturbation T_k Exp(xi) (p = Exp(-xi) T_k^-1 x_v, so
// dp/drho = -I, dp/dphi = [p]_x and d d_k / d xi = -d p_z / d xi).
//
// The keyframes run in chunks through the batched candidate stage, which
// leaves every block a keyframe may touch with the mask of those keyframes;
// a persistent pass then visits each candidate block once, loads its weights
// and upstream gradients, walks its keyframes, scatters the pixel gradients
// and accumulates the pose terms per workgroup in LDS.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "kernels.hpp"

namespace sc {

// A wavefront collects the pixel gradients of a (block, keyframe) in LDS, in a
// window of kAdjWin x kAdjWin pixels around the block's projected centre, and
// adds the window's touched rows to memory: neighbouring lanes then carry
// neighbouring pixels, and the voxels behind one another share an addition.
// Entry (r, c) of the window is pixel origin + r W + c of the image, whatever
// its place in it; a pixel whose entry lies outside goes to memory directly.
// The depth plane is FP64: a pixel's voxels lie on both sides of the surface,
// their terms cancel, and block sums in FP32 would add to what the additions
// to memory lose.
constexpr int kAdjWin = 22;  // a block of 8 cm spans 15 pixels of a 320-wide image at 1.5 m

template <int CM>
constexpr int adj_win_floats()
{
    return kAdjWin * kAdjWin * (CM == SC_COLOR_F32 ? 5 : 2);
}

// LDS of a workgroup: the pose terms of the chunk, then a window a wavefront
// (depth, then colour as pixels lie in memory).
template <int CM>
static size_t adj_lds(int n_ops)
{
    return sizeof(double) * 3 * (size_t)n_ops + sizeof(float) * 4 * adj_win_floats<CM>();
}

// Adds entries [begin, end) of a window plane with kLen entries a row to `out`
// (row r at out + r pitch) and clears them.
template <int kLen, class T>
__device__ inline void window_flush(T* win, int begin, int end, float* out, int pitch, int lane)
{
    for (int e0 = begin; e0 < end; e0 += 256) {
        T x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = e0 + 64 * q + lane;
            x[q] = e < end ? win[e] : (T)0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = e0 + 64 * q + lane;
            if (x[q] != (T)0) {
                const int r = e / kLen;
                atomicAdd(out + (int64_t)r * pitch + (e - r * kLen), (float)x[q]);
                win[e] = (T)0;
            }
        }
    }
}

// Bound: the memory's additions.  One a touched voxel and value, straight to
// memory: 16 keyframes of 320x240 with FP32 colour 639 us, now 184 (and the
// blocks from 32 counters instead of one; four wavefronts a SIMD with 18
// spilled registers, 190 against 221 us with three and none).
template <int CM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void adjoint_kernel(const OpDesc* __restrict__ ops, VolDev v, CandDev cd,
                                                      const float* __restrict__ gD, const float* __restrict__ gC,
                                                      float* grad_depth, float* grad_color, float* grad_D0,
                                                      float* grad_C0, double* acc_xi, int n_ops)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double* const s_acc = reinterpret_cast<double*>(smem);  // pose terms 2, 3, 4 of each keyframe of the chunk
    float* const wins = reinterpret_cast<float*>(s_acc + 3 * n_ops);
    const int lane = threadIdx.x & 63;
    const int wave = (int)bcast(threadIdx.x >> 6);
    double* const win_z = reinterpret_cast<double*>(wins + wave * adj_win_floats<CM>());
    float* const win_c = reinterpret_cast<float*>(win_z + kAdjWin * kAdjWin);
    for (int i = threadIdx.x; i < 3 * n_ops; i += blockDim.x) s_acc[i] = 0.0;
    for (int i = threadIdx.x; i < 4 * adj_win_floats<CM>(); i += blockDim.x) wins[i] = 0.0f;
    __syncthreads();
    const uint32_t n = cd.counters[4];
    const uint32_t worker = blockIdx.x * (blockDim.x >> 6) + (uint32_t)wave;
    const uint32_t n_workers = gridDim.x * (blockDim.x >> 6);
    RangeCursor cur;
    range_init(cur, worker, n, n_workers);
    for (;;) {
        const uint32_t i = range_pop(cur, cd.cursors + kCursorSet, n, n_workers, lane);
        if (i >= n) break;
        const uint32_t h = bcast(cd.sorted[i]);
        const uint64_t key = bcast64(cd.skey[i]);
        const int slot = (int)bcast((uint32_t)cd.sslot[i]);
        int bx, by, bz;
        unpack_key(key, bx, by, bz);
        // a candidate block the forward never allocated holds no touched voxel
        const size_t sb = (size_t)max(slot, 0);
        const float* blk = v.pool + sb * v.stride;
        float Wv[8], g[8], gc[3][8], sw[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int x = lane + 64 * j;
            Wv[j] = (slot >= 0) ? blk[kPoolW + x] : 0.0f;
            g[j] = (slot >= 0) ? gD[sb * kBlockVox + x] : 0.0f;
#pragma unroll
            for (int c = 0; c < 3; ++c) gc[c][j] = (gC && slot >= 0) ? gC[(sb * 3 + c) * kBlockVox + x] : 0.0f;
            sw[j] = 0.0f;
        }
        OpWalk walk{cd.mask + (size_t)h * cd.words, cd.words, 0, bcast64(cd.mask[(size_t)h * cd.words])};
        for (int o = walk_next(walk); o >= 0; o = walk_next(walk)) {
            const OpDesc& op = ops[o];
            float q[3];
            double qz;
            block_origin(op, v.s, bx, by, bz, q, qz);
            const float kx = (float)(lane & 7), ky = (float)(lane >> 3);
            RingGeom geo;
#pragma unroll
            for (int r = 0; r < 3; ++r) geo.base[r] = (q[r] + kx * op.a[0][r]) + ky * op.a[1][r];
            uint32_t pix[8];
            float w[8];
            bool t[8];
            auto test = [&](auto packed) {
                constexpr bool kPacked = decltype(packed)::value;
                RingFetch<CM> f[2];
                ring_fetch<CM, kPacked>(op, geo, 0, f[0]);
                ring_fetch<CM, kPacked>(op, geo, 4, f[1]);
                ring_decide<CM, kPacked>(f[0], v.mu, w, t);
                ring_decide<CM, kPacked>(f[1], v.mu, w + 4, t + 4);
#pragma unroll
                for (int j = 0; j < 8; ++j) pix[j] = f[j >> 2].pix[j & 3];
            };
            if (CM == SC_COLOR_RGBA8 && op.packed) test(std::true_type{});
            else test(std::false_type{});
            bool any = false;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                t[j] = t[j] && Wv[j] > 0.0f;
                any = any || t[j];
            }
            if (__ballot(any) == 0ull) continue;
            // the window about the centre's pixel (clamped, also from a NaN)
            const int W = op.width;
            const float rW = __builtin_amdgcn_rcpf(op.wf);
            int origin;
            {
                float m[3];
#pragma unroll
                for (int r = 0; r < 3; ++r) m[r] = q[r] + 3.5f * (op.a[0][r] + op.a[1][r] + op.a[2][r]);
                const float rz = __builtin_amdgcn_rcpf(m[2]);
                const int u0 = (int)fminf(fmaxf(op.fx * m[0] * rz + op.cx, -64.0f), 16448.0f) - kAdjWin / 2;
                const int v0 = (int)fminf(fmaxf(op.fy * m[1] * rz + op.cy, -64.0f), 16448.0f) - kAdjWin / 2;
                origin = (int)bcast((uint32_t)(v0 * W + u0));
            }
            const size_t first = (size_t)op.kf * ((size_t)W * op.height);  // the keyframe's first pixel
            uint32_t rows = 0u;  // of the window, touched by this lane
            float j2 = 0.0f, j3 = 0.0f, j4 = 0.0f;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (!t[j]) continue;
                const float px = geo.base[0] + op.za[j][0];
                const float py = geo.base[1] + op.za[j][1];
                const float a = w[j] / Wv[j];
                const float gg = g[j] * a;
                const int d = (int)pix[j] - origin;
                // d < 22 * 16384, so the product's error is far below half a pixel's 1 / (2 W)
                const int r = (int)(((float)d + 0.5f) * rW), c = d - r * W;
                if ((unsigned)d < (unsigned)(kAdjWin * W) && c < kAdjWin) {
                    const int e = r * kAdjWin + c;
                    atomicAdd(win_z + e, (double)gg);
                    if (CM == SC_COLOR_F32 && grad_color) {
                        atomicAdd(win_c + 3 * e + 0, gc[0][j] * a);
                        atomicAdd(win_c + 3 * e + 1, gc[1][j] * a);
                        atomicAdd(win_c + 3 * e + 2, gc[2][j] * a);
                    }
                    rows |= 1u << r;
                } else {
                    const size_t at = first + pix[j];
                    atomicAdd(grad_depth + at, gg);
                    if (CM == SC_COLOR_F32 && grad_color) {
                        atomicAdd(grad_color + 3 * at + 0, gc[0][j] * a);
                        atomicAdd(grad_color + 3 * at + 1, gc[1][j] * a);
                        atomicAdd(grad_color + 3 * at + 2, gc[2][j] * a);
                    }
                }
                sw[j] += w[j];
                j2 += gg;
                j3 += gg * py;
                j4 -= gg * px;
            }
            // the three sums over the wavefront, halving what a lane holds in
            // the first two steps: they end in lanes 0, 16 and 32
            const bool b5 = lane & 32, b4 = lane & 16;
            const double t2 = (double)j2, t3 = (double)j3, t4 = (double)j4;
            double a0 = (b5 ? t4 : t2) + __shfl_xor(b5 ? t2 : t4, 32);
            double a1 = (b5 ? 0.0 : t3) + __shfl_xor(b5 ? t3 : 0.0, 32);
            double sum = (b4 ? a1 : a0) + __shfl_xor(b4 ? a0 : a1, 16);
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) rows |= (uint32_t)__shfl_xor((int)rows, off);
            if ((lane & 15) == 0 && lane < 48) atomicAdd(s_acc + 3 * o + (lane >> 4), sum);
            rows = bcast(rows);
            if (rows == 0u) continue;
            wave_lds_sync();
            const int r0 = __ffs((int)rows) - 1, r1 = 32 - __clz((int)rows);  // rows [r0, r1)
            const int64_t at = (int64_t)first + origin;
            window_flush<kAdjWin>(win_z, r0 * kAdjWin, r1 * kAdjWin, grad_depth + at, W, lane);
            if (CM == SC_COLOR_F32 && grad_color)
                window_flush<3 * kAdjWin>(win_c, 3 * r0 * kAdjWin, 3 * r1 * kAdjWin, grad_color + 3 * at, 3 * W, lane);
            wave_lds_sync();
        }
        // dL/dD0 = dL/dD (W - sum_k w_k) / W: grad_D0 first collects
        // sum_k w_k over the chunks (exact in FP32 on the 2^-10 weight grid
        // below 2^14, one wavefront per block and launch), and the final
        // kernel forms W0 = W - sum_k w_k exactly before one division, so a
        // small W0 / W is not the difference of two nearly equal products
        if (slot >= 0 && grad_D0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int x = lane + 64 * j;
                if (sw[j] > 0.0f) grad_D0[sb * kBlockVox + x] += sw[j];
            }
        }
        retire_candidate(cd, v, h, 0, lane);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * n_ops; i += blockDim.x)
        if (s_acc[i] != 0.0) atomicAdd(acc_xi + i, s_acc[i]);
}

// grad_D0 holds sum_k w_k per voxel while the chunks run; it starts at 0.
__global__ void adjoint_prior_init_kernel(int64_t n_blocks, float* grad_D0)
{
    const int64_t b = blockIdx.x;
    for (int x = threadIdx.x; x < kBlockVox; x += blockDim.x) grad_D0[b * kBlockVox + x] = 0.0f;
}

// dL/dD0 = dL/dD W0 / W and dL/dC0 = dL/dC W0 / W with W0 = W - sum_k w_k
// (exact), where W > 0; 0 elsewhere (an empty voxel stays empty whatever D0
// holds).
__global__ void adjoint_prior_final_kernel(VolDev v, int64_t n_blocks, const float* gD, const float* gC,
                                           float* grad_D0, float* grad_C0)
{
    const int64_t b = blockIdx.x;
    const float* blk = v.pool + (size_t)b * v.stride;
    for (int x = threadIdx.x; x < kBlockVox; x += blockDim.x) {
        const float W = blk[kPoolW + x];
        const bool live = W > 0.0f;
        const float f = live ? (W - grad_D0[b * kBlockVox + x]) / W : 0.0f;
        grad_D0[b * kBlockVox + x] = live ? gD[b * kBlockVox + x] * f : 0.0f;
        if (grad_C0)
            for (int c = 0; c < 3; ++c)
                grad_C0[(b * 3 + c) * kBlockVox + x] = (live && gC) ? gC[(b * 3 + c) * kBlockVox + x] * f : 0.0f;
    }
}

__global__ void xi_final_kernel(double* acc, int n, float* out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        out[6 * (i / 3) + 2 + i % 3] += (float)acc[i];
        acc[i] = 0.0;
    }
}

}  // namespace sc

using namespace sc;

extern "C" {

sc_status tsdf_integrate_backward(sc_volume* vol, const sc_keyframe* kfs, int32_t n_kf, const sc_intrinsics* intr,
                                  const sc_pose* T, const float* grad_D, const float* grad_C, float* grad_depth,
                                  float* grad_color, float* grad_xi, float* grad_D0, float* grad_C0, void* stream)
{
    if (!vol || !kfs || n_kf <= 0 || !intr || intr->width <= 0 || intr->height <= 0 || !(intr->fx > 0.0f) ||
        !(intr->fy > 0.0f) || intr->width > 16384 || intr->height > 16384 || !T || !grad_D || !grad_depth ||
        !grad_xi)
        return SC_EINVAL;
    if ((grad_C != nullptr) != (grad_color != nullptr)) return SC_EINVAL;
    if (grad_C0 && (!grad_D0 || !grad_C)) return SC_EINVAL;
    if (grad_color && vol->p.color_mode != SC_COLOR_F32) return SC_EINVAL;
    if (stream_host_blocks(vol) > 0) return SC_EINVAL;  // the forward's blocks must all be on the device
    for (int i = 0; i < n_kf; ++i)
        if (!keyframe_ok(&kfs[i])) return SC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    int64_t nb = 0;
    int32_t sticky = 0;
    sc_status st = sc_volume_query(vol, s, &nb, &sticky);
    if (st != SC_OK) return st;
    if (sticky != SC_OK) return sticky;
    if (grad_D0 && nb > 0) adjoint_prior_init_kernel<<<(unsigned)nb, 256, 0, s>>>(nb, grad_D0);
    const int chunk = std::min(vol->p.max_batch_ops, kAdjChunk);
    const bool f32 = vol->p.color_mode == SC_COLOR_F32;
    for (int k0 = 0; k0 < n_kf; k0 += chunk) {
        const int cnt = std::min(chunk, n_kf - k0);
        OpDesc* ops = stage_begin(vol);
        if (!ops) return SC_EDEVICE;
        // op.kf is the keyframe's index in the call: it addresses the pixel gradients
        for (int j = 0; j < cnt; ++j) make_op(vol, &kfs[k0 + j], intr, &T[k0 + j], +1, k0 + j, &ops[j]);
        const bool dirty = vol->cand_dirty;
        vol->cand_dirty = true;
        st = run_candidates(vol, ops, cnt, intr, s);
        if (st != SC_OK) return st;
        const int grid = vol->n_cu * 4;
        if (f32)
            adjoint_kernel<SC_COLOR_F32><<<grid, 256, adj_lds<SC_COLOR_F32>(cnt), s>>>(
                vol->d_ops, vol->dev, vol->cand, grad_D, grad_C, grad_depth, grad_color, grad_D0, grad_C0,
                vol->adj_acc, cnt);
        else
            adjoint_kernel<SC_COLOR_RGBA8><<<grid, 256, adj_lds<SC_COLOR_RGBA8>(cnt), s>>>(
                vol->d_ops, vol->dev, vol->cand, grad_D, nullptr, grad_depth, nullptr, grad_D0, nullptr,
                vol->adj_acc, cnt);
        if (hipPeekAtLastError() != hipSuccess) return SC_EDEVICE;
        vol->cand_dirty = dirty;
        xi_final_kernel<<<(3 * cnt + 255) / 256, 256, 0, s>>>(vol->adj_acc, 3 * cnt, grad_xi + 6 * (size_t)k0);
    }
    if (grad_D0 && nb > 0)
        adjoint_prior_final_kernel<<<(unsigned)nb, 256, 0, s>>>(vol->dev, nb, grad_D, grad_C, grad_D0, grad_C0);
    return hipGetLastError() == hipSuccess ? SC_OK : SC_EDEVICE;
}

}  // extern "C"
