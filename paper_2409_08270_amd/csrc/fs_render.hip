// Novel-view mask rendering (paper Sec. 3.4 "Depth-guided Novel View Mask
// Rendering" and the supplement's "Quantization in novel view mask").
//
// For every object e, the Gaussians labelled e (row e of S) are composited on
// their own, front to back, with the compositing rules of the accumulation
// pass: rho_e = sum of alpha*T (the object's alpha mask) and
// D_e = sum of alpha*T*z / rho_e (its depth where it is visible). The mask
// label is then either
//   depth-guided: the object with rho_e > tau of least D_e (0 if none), or
//   argmax:       argmax over all objects (background included) of rho_e.
//
// One workgroup renders one tile; each of its four waves owns an 8x8 block of
// pixels and works by itself, without barriers. The objects are taken kObj at a
// time, with one walk over the tile's depth-ordered list for all of them: a lane
// takes one of 64 list entries, reads its membership bits for those objects, and
// only if there are any gathers the record and tests whether its support can reach
// the box of the block's live pixels. What is left goes to LDS, and the entries of
// each object are one ballot: a scalar loop over its bits composites them in list
// order into that object's registers (an entry of two objects is composited in
// each). Each object's arithmetic is the same sequence of operations as compositing
// it alone.
//
// What bounds it: the chain of the steps (two LDS reads, then 21 vector and 16 scalar
// instructions per entry and object, most of them one after the other) with too few waves to
// hide it, as tiles differ in their lists. Counters: vector issue in 0.42 of the SIMDs' cycles
// and 2.7 of 5 waves resident for 8 views of 800x600 of a 500k-Gaussian scene with 10 classes
// (1.90 ms), 0.55 and 3.8 for 40 views of 1008x756 of 700k Gaussians (9.45 ms). Having every
// pixel walk all the tile's entries of any of 8 objects, with a barrier per 256 entries and a
// divergent branch per object, took 13.5 ms for the 8 views. 16 objects a walk: with 8 the same
// scene takes 2.4 ms and 4 views of 1008x756 of 1M Gaussians with 64 classes 15.1 ms against
// 9.1 ms; with 32 the state of the objects (three registers each) leaves two waves per SIMD, 3.3
// and 14.4 ms. Five waves per SIMD (96 registers, 16 spilled outside the steps) against four: 1.85
// and 2.04 ms (these before the depth of an entry that a lane does not take was left out of
// its sum, which took the 1.85 to 1.90).
//
// The steps are per (entry, object), so Gaussians in many objects at once cost more than
// they would with one walk that forms an alpha for all of them: 4 views of 800x600 of 300k
// Gaussians, each in 1, 4, 8 and all of 16 objects, take 2.2, 3.6, 4.7 and 6.0 ms (such a
// walk 4.6, 5.8, 5.0 and 4.4 ms). A second loop in here for dense groups of entries spills
// 158 more registers, in the steps of both.
//
// The membership bits come from one 16-bit word per (group of kObj objects,
// Gaussian), built from S beforehand with reads that are contiguous along the
// Gaussians, so that staging an entry gathers one word per group instead of
// one row of S per object.
#include "fs_internal.h"

namespace fs {
namespace {

constexpr int kObj = 16;  // objects composited in one walk of a tile's list
using Memb = uint16_t;    // a Gaussian's membership bits for the objects of one walk

// memb[q][g], bit k: Gaussian g belongs to object e_first + kObj q + k
__global__ void k_member_bits(const uint8_t *__restrict__ S, int64_t n, int32_t e_first, int32_t E,
                               Memb *__restrict__ memb)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    for (int q = 0, e0 = e_first; e0 < E; ++q, e0 += kObj) {
        uint32_t bits = 0;
        for (int k = 0; k < kObj && e0 + k < E; ++k) bits |= (S[(int64_t)(e0 + k) * n + g] != 0 ? 1u : 0u) << k;
        memb[(int64_t)q * n + g] = (Memb)bits;
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 5))) void k_render(const float4 *__restrict__ rec, const uint32_t *__restrict__ vals,
                                                const uint2 *__restrict__ ranges, const ViewDev *__restrict__ views,
                                                int32_t n_views, const Memb *__restrict__ memb, int64_t n, int32_t E,
                                                AccParams P, float tau, int32_t mode, uint8_t *__restrict__ labels,
                                                float *__restrict__ rho_out, float *__restrict__ depth_out,
                                                int64_t n_pixels)
{
#pragma clang fp contract(off)
    // per wave, entry j: s_rec[2 j] = (u, v, p', r), s_rec[2 j + 1] = (s', lo, thr, z), with the
    // LDL^T factors p, s in log2 units
    __shared__ float4 s_rec[4][2 * 64];

    const uint32_t tile = blockIdx.x;
    const int view = find_view_of_tile(views, n_views, tile);
    const ViewDev &C = views[view];
    const uint32_t local = tile - C.tile_base;
    const int tx = (int)(local % (uint32_t)C.tiles_x), ty = (int)(local / (uint32_t)C.tiles_x);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int bpr = P.tile_w >> 3;  // 8x8 blocks per tile row
    const int x0 = tx * P.tile_w + (w % bpr) * 8, y0 = ty * P.tile_h + (w / bpr) * 8;
    const int x = x0 + (lane & 7), y = y0 + (lane >> 3);
    const bool inside = x < C.W && y < C.H;
    const int64_t pix = (int64_t)C.mask_off + (int64_t)y * C.W + x;
    const float pxc = (float)x + 0.5f, pyc = (float)y + 0.5f;
    const float LOG2E = 1.4426950408889634f;
    const uint2 rg = ranges[tile];
    const int64_t rec_base = (int64_t)C.elem_off;
    float4 *const recs = s_rec[w];
    const float a_max = fminf(P.alpha_max, 1.0f);

    int best = 0;
    float best_d = 3.0e38f, best_rho = -1.0f;
    const int e_first = mode == 1 ? 0 : 1;
    for (int e0 = e_first; e0 < E; e0 += kObj) {
        const Memb *__restrict__ mq = memb + (int64_t)((e0 - e_first) / kObj) * n;
        const int ne = min(kObj, E - e0);
        float T[kObj], rho[kObj], dz[kObj];
#pragma unroll
        for (int k = 0; k < kObj; ++k) {
            T[k] = 1.0f;
            rho[k] = 0.0f;
            dz[k] = 0.0f;
        }
        // bit k: this pixel still composites object e0 + k; alive: the same for any pixel of the wave
        uint32_t live = inside ? ((1u << ne) - 1u) : 0u;
        uint32_t alive = __ballot(inside) ? ((1u << ne) - 1u) : 0u;
        // ids are read two groups of 64 ahead, their membership bits one
        uint32_t g1 = rg.x + lane < rg.y ? vals[rg.x + lane] : 0u;
        uint32_t g2 = rg.x + 64u + lane < rg.y ? vals[rg.x + 64u + lane] : 0u;
        uint32_t m1 = rg.x + lane < rg.y ? mq[g1] : 0u;
        for (uint32_t base = rg.x; base < rg.y && alive; base += 64) {
            const uint32_t g = g1;
            uint32_t mbits = m1 & alive;
            g1 = g2;
            m1 = base + 64u + lane < rg.y ? mq[g1] : 0u;
            if (base + 128u + lane < rg.y) g2 = vals[base + 128u + lane];
            if (__ballot(mbits != 0u) == 0ull) continue;
            // columns bx.. and rows by.. of the wave's live pixels (lane = 8 * row + column)
            const unsigned long long lm = __ballot(live != 0u);
            uint32_t cols = (uint32_t)(lm | (lm >> 32));
            cols |= cols >> 16;
            cols = (cols | (cols >> 8)) & 0xFFu;
            const float bx0 = (float)(__ffs((int)cols) - 1), bx1 = (float)(31 - __clz((int)cols));
            const float by0 = (float)((__ffsll((long long)lm) - 1) >> 3), by1 = (float)((63 - __clzll((long long)lm)) >> 3);
            if (mbits) {
                const float4 r0 = rec[(rec_base + g) * 2];
                const float4 r1 = rec[(rec_base + g) * 2 + 1];
                const float lo = fmaxf(__builtin_amdgcn_logf(r1.y), -200.0f);
                if (block_hit(r0.x, r0.y, r0.z, r0.w, r1.x, (float)x0, (float)y0, reach_limit(P, lo), bx0, bx1, by0, by1)) {
                    recs[2 * lane] = make_float4(r0.x, r0.y, -0.5f * LOG2E * r0.z, r0.w);
                    recs[2 * lane + 1] = make_float4(-0.5f * LOG2E * r1.x, lo, P.cut2 + lo, r1.z);
                } else {
                    mbits = 0u;
                }
            }
            __builtin_amdgcn_wave_barrier();
            uint32_t left = 0;  // objects with a live pixel after this group of entries
#pragma unroll
            for (int k = 0; k < kObj; ++k) {
                if (!((alive >> k) & 1u)) continue;
                unsigned long long todo = __ballot((mbits >> k) & 1u);
                bool on = (live >> k) & 1u;
                float Tk = T[k], rk = rho[k], dk = dz[k];
                while (todo) {
                    const int j = __ffsll((long long)todo) - 1;
                    todo &= todo - 1ull;
                    const float4 q = recs[2 * j];
                    const float4 q2 = recs[2 * j + 1];
                    const float dx = pxc - q.x, dy = pyc - q.y;
                    const float e = fmaf(q.w, dy, dx);
                    const float pw = fmaf(q.z * e, e, fmaf(q2.x * dy, dy, q2.y));
                    const float av = fminf(a_max, __builtin_amdgcn_exp2f(pw));
                    // alpha = 0 leaves T and rho as they are, and with z = 0 the depth sum (a
                    // depth may be infinite)
                    const bool hit = on && pw >= q2.z && av >= P.alpha_min;
                    const float alpha = hit ? av : 0.0f, z = hit ? q2.w : 0.0f;
                    const float Tn = fmaf(-Tk, alpha, Tk);
                    const float wv = alpha * Tk;
                    const bool stop = alpha > 0.0f && Tn < P.t_min;  // the entry is not added, the pixel ends
                    if (__builtin_expect(__ballot(stop) != 0ull, 0)) {
                        if (!stop) {
                            rk = fmaf(alpha, Tk, rk);
                            dk = fmaf(wv, z, dk);
                            Tk = Tn;
                        }
                        on = on && !stop;
                        if (__ballot(on) == 0ull) break;
                    } else {
                        rk = fmaf(alpha, Tk, rk);
                        dk = fmaf(wv, z, dk);
                        Tk = Tn;
                    }
                }
                T[k] = Tk;
                rho[k] = rk;
                dz[k] = dk;
                live = on ? live : (live & ~(1u << k));
                if (__ballot(on)) left |= 1u << k;
            }
            alive = left;
            __builtin_amdgcn_wave_barrier();  // the records are read before the next group's are written
        }
#pragma unroll
        for (int k = 0; k < kObj; ++k) {
            if (k >= ne) break;
            const int eo = e0 + k;
            const float d = rho[k] > 0.0f ? dz[k] / rho[k] : 3.0e38f;
            if (inside) {
                const int64_t o = (int64_t)eo * n_pixels + pix;
                if (rho_out) rho_out[o] = rho[k];
                if (depth_out) depth_out[o] = d;
            }
            if (mode == 1) {
                if (rho[k] > best_rho) {
                    best_rho = rho[k];
                    best = eo;
                }
            } else if (rho[k] > tau && d < best_d) {
                best_d = d;
                best = eo;
            }
        }
    }
    if (inside) labels[pix] = (uint8_t)best;
}

}  // namespace

hipError_t launch_render(hipStream_t s, const float *rec, const uint32_t *vals, const uint32_t *ranges,
                         const ViewDev *views, int32_t n_views, uint32_t n_tiles, const uint8_t *S, int64_t n,
                         int32_t E, const AccParams &p, float tau, int32_t mode, uint8_t *labels, float *rho,
                         float *depth, int64_t n_pixels, uint8_t *memb)
{
    if (n_tiles == 0) return hipSuccess;
    if (n > 0) {
        hipLaunchKernelGGL(k_member_bits, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, S, n,
                           mode == 1 ? 0 : 1, E, (Memb *)memb);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_render, dim3(n_tiles), dim3(256), 0, s, reinterpret_cast<const float4 *>(rec), vals,
                       reinterpret_cast<const uint2 *>(ranges), views, n_views, (const Memb *)memb, n, E, p, tau, mode, labels, rho,
                       depth, n_pixels);
    return hipGetLastError();
}

int64_t render_member_bytes(int64_t n, int32_t E, int32_t mode)
{
    const int e_first = mode == 1 ? 0 : 1;
    return (int64_t)sizeof(Memb) * n * (int64_t)((E - e_first + kObj - 1) / kObj);
}

}  // namespace fs
