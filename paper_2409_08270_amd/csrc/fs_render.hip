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
// pixels. The objects are taken kObj at a time, with one walk over the tile's
// depth-ordered list for all of them: a lane takes one list entry, reads its
// membership bits for those objects, and only if there are any gathers the record and
// tests whether its support can reach the box of a block's live pixels. What is left goes
// to LDS, and the entries of each object are one ballot: a scalar loop over its bits
// composites them in list order into that object's registers (an entry of two objects is
// composited in each). Each object's arithmetic is the same sequence of operations as
// compositing it alone.
//
// Either each wave walks the list by itself, 64 entries at a time and without barriers, or
// (SHARED, by the rule of shared_walk) the waves share the walk, 256 entries at a time, and an
// entry is read and staged once for all the waves that it reaches.
//
// What bounds it: the chain of the steps (two LDS reads, then 19 vector and 14 scalar
// instructions per entry and object, most of them one after the other) with too few waves to
// hide it, as tiles differ in their lists; in large scenes the reading of the entries. Having
// every pixel walk all the tile's entries of any of 8 objects, with a barrier per 256 entries and
// a divergent branch per object, took 13.5 ms for 8 views of 800x600 of a 500k-Gaussian scene with
// 10 classes; this takes 1.85. 16 objects a walk: with 8 the same scene takes 2.4 ms and 4 views
// of 1008x756 of 1M Gaussians with 64 classes 15.1 ms against 9.1 ms (5.5 shared); with 32 the
// state of the objects (three registers each) leaves two waves per SIMD, 3.3 and 14.4 ms. Waves on
// their own: five per SIMD (96 registers, 16 spilled outside the steps) against four, 1.85 and
// 2.04 ms. Shared: four (five spill 72 registers, 29 ms instead of 22 for 4 views of 1297x840 of 3M
// Gaussians with 64 classes); 320 or 1024 staged entries are within 4% of 576.
//
// The steps are per (entry, object), so Gaussians in many objects at once cost more than
// they would with one walk that forms an alpha for all of them: 4 views of 800x600 of 300k
// Gaussians, each in 1, 4, 8 and all of 16 objects, take 2.1, 3.4, 4.5 and 5.8 ms (such a
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

constexpr int kObj = 16;          // objects composited in one walk of a tile's list
constexpr uint32_t kStage = 576;  // most entries that a shared walk stages
using Memb = uint16_t;            // a Gaussian's membership bits for the objects of one walk

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

// the live pixels of a wave (lane = 8 * row + column): columns x0.. x1, rows y0.. y1 (one is live)
struct Box {
    int x0, x1, y0, y1;
};
__device__ __forceinline__ Box box_of(unsigned long long lm)
{
    uint32_t cols = (uint32_t)(lm | (lm >> 32));
    cols |= cols >> 16;
    cols = (cols | (cols >> 8)) & 0xFFu;
    return Box{__ffs((int)cols) - 1, 31 - __clz((int)cols), (__ffsll((long long)lm) - 1) >> 3, (63 - __clzll((long long)lm)) >> 3};
}

// block_hit over a box of the 8x8 block with corner (bx, by)
__device__ __forceinline__ bool box_hit(float u, float v, float p, float r, float s, int bx, int by, float lim, const Box &b)
{
    return block_hit(u, v, p, r, s, (float)bx, (float)by, lim, (float)b.x0, (float)b.x1, (float)b.y0, (float)b.y1);
}

// a box as one word, a byte each; kNoBox: no live pixel
constexpr uint32_t kNoBox = 0xFFu;
__device__ __forceinline__ uint32_t pack_box(bool live)
{
    const unsigned long long lm = __ballot(live);
    if (lm == 0ull) return kNoBox;
    const Box b = box_of(lm);
    return (uint32_t)b.x0 | (uint32_t)b.x1 << 8 | (uint32_t)b.y0 << 16 | (uint32_t)b.y1 << 24;
}
__device__ __forceinline__ Box unpack_box(uint32_t w)
{
    return Box{(int)(w & 0xFFu), (int)((w >> 8) & 0xFFu), (int)((w >> 16) & 0xFFu), (int)(w >> 24)};
}

template <bool SHARED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SHARED ? 4 : 5, SHARED ? 4 : 5))) void k_render(
    const float4 *__restrict__ rec_in, const uint32_t *__restrict__ vals, const uint2 *__restrict__ ranges,
    const ViewDev *__restrict__ views, int32_t n_views, const Memb *__restrict__ memb, int64_t n, int32_t E, AccParams P,
    float tau, int32_t mode, uint8_t *__restrict__ labels, float *__restrict__ rho_out, float *__restrict__ depth_out,
    int64_t n_pixels)
{
#pragma clang fp contract(off)
    // staged entry j: s_rec[2 j] = (u, v, p', r), s_rec[2 j + 1] = (s', lo, thr, z), with the
    // LDL^T factors p, s in log2 units. SHARED: s_in[j] = membership bits | the waves it reaches << 16;
    // else each wave has 64 entries of its own
    __shared__ float4 s_rec[2 * (SHARED ? kStage : 256u)];
    __shared__ uint32_t s_in[SHARED ? kStage : 1u];
    __shared__ uint32_t s_cnt[2][4], s_alive[4], s_box[4];

    const uint32_t tile = blockIdx.x;
    const int view = find_view_of_tile(views, n_views, tile);
    const ViewDev &C = views[view];
    const uint32_t local = tile - C.tile_base;
    const int tx = (int)(local % (uint32_t)C.tiles_x), ty = (int)(local / (uint32_t)C.tiles_x);
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int bpr = P.tile_w >> 3;  // 8x8 blocks per tile row
    const int x0 = tx * P.tile_w + (w % bpr) * 8, y0 = ty * P.tile_h + (w / bpr) * 8;
    const int x = x0 + (lane & 7), y = y0 + (lane >> 3);
    const bool inside = x < C.W && y < C.H;
    const int64_t pix = (int64_t)C.mask_off + (int64_t)y * C.W + x;
    const float pxc = (float)x + 0.5f, pyc = (float)y + 0.5f;
    const float LOG2E = 1.4426950408889634f;
    const float4 *__restrict__ rec = rec_in + 2 * (int64_t)C.elem_off;
    const uint2 rg = ranges[tile];
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

        auto staged0 = [&](const float4 &r0) { return make_float4(r0.x, r0.y, -0.5f * LOG2E * r0.z, r0.w); };
        auto staged1 = [&](const float4 &r1, float lo) { return make_float4(-0.5f * LOG2E * r1.x, lo, P.cut2 + lo, r1.z); };

        auto publish = [&]() {
            const uint32_t box = pack_box(live != 0u);
            if (lane == 0) {
                s_alive[w] = alive;
                s_box[w] = box;
            }
        };
        // SHARED: the objects that any wave still composites and (lane i) wave i's live box, as
        // published; entries staged; which of s_cnt's halves is in use
        uint32_t alive_b = (1u << ne) - 1u, boxes = 0, fill = 0, par = 0;
        if constexpr (SHARED) {
            __syncthreads();  // the walk before has been read
            publish();
            __syncthreads();
            boxes = s_box[lane & 3];
        }
        // list entries are taken kStep at a time, one per lane; ids are read two steps ahead, their
        // membership bits one
        constexpr uint32_t kStep = SHARED ? 256u : 64u;
        const uint32_t me = SHARED ? (uint32_t)tid : (uint32_t)lane;
        uint32_t g1 = rg.x + me < rg.y ? vals[rg.x + me] : 0u;
        uint32_t g2 = rg.x + kStep + me < rg.y ? vals[rg.x + kStep + me] : 0u;
        uint32_t m1 = rg.x + me < rg.y ? mq[g1] : 0u;
        for (uint32_t base = rg.x; base < rg.y && (SHARED || alive); base += kStep, par ^= 1u) {
            const uint32_t g = g1;
            uint32_t mbits = m1 & (SHARED ? alive_b : alive);
            g1 = g2;
            m1 = base + kStep + me < rg.y ? mq[g1] : 0u;
            if (base + 2u * kStep + me < rg.y) g2 = vals[base + 2u * kStep + me];
            uint32_t seen = 0;
            if constexpr (!SHARED) {
                if (__ballot(mbits != 0u) == 0ull) continue;
                const Box box = box_of(__ballot(live != 0u));
                if (mbits) {
                    const float4 r0 = rec[2 * (int64_t)g];
                    const float4 r1 = rec[2 * (int64_t)g + 1];
                    const float lo = fmaxf(__builtin_amdgcn_logf(r1.y), -200.0f);
                    if (box_hit(r0.x, r0.y, r0.z, r0.w, r1.x, x0, y0, reach_limit(P, lo), box)) {
                        s_rec[128 * w + 2 * lane] = staged0(r0);
                        s_rec[128 * w + 2 * lane + 1] = staged1(r1, lo);
                    } else {
                        mbits = 0u;
                    }
                }
                __builtin_amdgcn_wave_barrier();
            } else {
                uint32_t waves = 0;  // those that the entry reaches
                float4 q0, q1;
                if (mbits) {
                    const float4 r0 = rec[2 * (int64_t)g];
                    const float4 r1 = rec[2 * (int64_t)g + 1];
                    const float lo = fmaxf(__builtin_amdgcn_logf(r1.y), -200.0f);
                    const float lim = reach_limit(P, lo);
#pragma unroll 1
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t box = __builtin_amdgcn_readlane(boxes, i);
                        if (box != kNoBox && box_hit(r0.x, r0.y, r0.z, r0.w, r1.x, tx * P.tile_w + (i % bpr) * 8,
                                                     ty * P.tile_h + (i / bpr) * 8, lim, unpack_box(box)))
                            waves |= 1u << i;
                    }
                    q0 = staged0(r0);
                    q1 = staged1(r1, lo);
                }
                const unsigned long long bm = __ballot(waves != 0u);
                if (lane == 0) s_cnt[par][w] = (uint32_t)__popcll(bm);
                __syncthreads();  // every wave has composited what was staged before
                uint32_t at = fill, total = 0;
                alive_b = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t c = s_cnt[par][i];
                    if (i < w) at += c;
                    total += c;
                    alive_b |= s_alive[i];
                }
                boxes = s_box[lane & 3];
                fill = __builtin_amdgcn_readfirstlane(fill + total);
                alive_b = __builtin_amdgcn_readfirstlane(alive_b);
                if (waves) {
                    const uint32_t j = at + (uint32_t)__popcll(bm & ((1ull << lane) - 1ull));
                    s_rec[2 * j] = q0;
                    s_rec[2 * j + 1] = q1;
                    s_in[j] = mbits | waves << 16;
                }
                if (alive_b == 0u) break;
                // s_cnt's halves are used in turn and nothing was published, so the next entries can be
                // read at once
                if (fill <= kStage - 256u && base + 256u < rg.y) continue;
                __syncthreads();  // the staged entries are there
                seen = __builtin_amdgcn_readlane(boxes, w);
            }
            // the staged entries, 64 at a time
            for (uint32_t c = 0; c < (SHARED ? fill : 64u); c += 64) {
                const float4 *const recs = s_rec + (SHARED ? 2 * c : 128 * w);
                if constexpr (SHARED) {
                    if (!alive) break;
                    const uint32_t in = c + lane < fill ? s_in[c + lane] : 0u;
                    mbits = (in >> (16 + w)) & 1u ? in & alive : 0u;
                    const uint32_t box = pack_box(live != 0u);
                    if (box != seen && mbits) {  // fewer live pixels than the entries were tested against
                        const float4 q = recs[2 * lane], q2 = recs[2 * lane + 1];
                        if (!box_hit(q.x, q.y, -q.z, q.w, -q2.x, x0, y0, reach_limit(P, q2.y) * (0.5f * LOG2E),
                                     unpack_box(box)))
                            mbits = 0u;
                    }
                    if (__ballot(mbits != 0u) == 0ull) continue;
                }
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
                        const float av = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(pw), 0.0f, a_max);  // a minimum: 2^pw >= 0
                        // alpha = 0 leaves T and rho as they are, and with z = 0 the depth sum (a
                        // depth may be infinite)
                        const bool hit = on && pw >= q2.z && av >= P.alpha_min;
                        const float alpha = hit ? av : 0.0f, z = hit ? q2.w : 0.0f;
                        const float Tn = fmaf(-Tk, alpha, Tk);
                        const float wv = alpha * Tk;
                        // the entry is not added, the pixel ends (with alpha = 0, Tn = T >= t_min)
                        const bool stop = Tn < P.t_min;
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
            }
            if constexpr (SHARED) {
                fill = 0;
                publish();
            } else {
                __builtin_amdgcn_wave_barrier();  // the records are read before the next step's are written
            }
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

// Whether a tile's waves share the walk over its list. Reading the entries (id, membership, record)
// is then done once per tile instead of once per wave, which pays where most entries read are not
// composited: lists long for their objects. In ms, on their own / shared, views of
//   one object: 300k Gaussians 800x600 0.32/0.29 (4 views), 2M 2400x1800 3.3/1.4;
//   one walk: 300k 800x600 0.99/1.23 (4), 500k 800x600 1.87/2.2 (8), 700k 1008x756 3.2/3.2 (8),
//   1M 800x600 2.24/2.13 (4), 1M 2400x1800 1.84/1.17, but 1M 320x240 4.3/4.8, which leaves CUs idle;
//   several: 300k 2 walks 1.05/1.25 (800x600, 4), 400k 2 walks 1.81/1.99 (640x480, 4), 500k 2 walks
//   1.99/1.90 (2400x1800), 250k 4 walks 2.35/2.05 (800x600, 4), 3M 4 walks 75/22 (1297x840, 4), 300k
//   13 walks 7.0/4.0 (800x600, 4).
bool shared_walk(int64_t n, int32_t objects, uint32_t n_tiles)
{
    const int64_t walks = (objects + kObj - 1) / kObj;
    if (objects == 1) return n >= 400000;
    return n * walks >= 1000000 && (walks > 1 || n_tiles >= 1024);
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
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(n_tiles), dim3(256), 0, s, reinterpret_cast<const float4 *>(rec), vals,
                           reinterpret_cast<const uint2 *>(ranges), views, n_views, (const Memb *)memb, n, E, p, tau,
                           mode, labels, rho, depth, n_pixels);
    };
    if (!shared_walk(n, E - (mode == 1 ? 0 : 1), n_tiles)) go(k_render<false>);
    else go(k_render<true>);
    return hipGetLastError();
}

int64_t render_member_bytes(int64_t n, int32_t E, int32_t mode)
{
    const int e_first = mode == 1 ? 0 : 1;
    return (int64_t)sizeof(Memb) * n * (int64_t)((E - e_first + kObj - 1) / kObj);
}

}  // namespace fs
