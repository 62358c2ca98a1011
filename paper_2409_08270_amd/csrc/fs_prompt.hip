// Point-prompt propagation (paper Sec. 4.1 "2D mask generation and
// association" and the supplement's "Binary Mask Association"): each point
// prompt on a reference view is back-projected to the world at a given depth,
// the k Gaussian centres nearest to it (L2) are found, the one of least
// positive depth in the reference view is chosen, and its centre is projected
// into every view, giving the associated prompt of each view.
//
// One grid row (blockIdx.y) per prompt. A wave keeps its k smallest keys sorted across its lanes:
// of 64 new keys those below its k-th are taken, one by one, each by a ballot (its place) and
// a shift of the lanes above. The waves of a block merge their lists the same way; the second
// kernel merges the blocks' lists of one prompt and looks at the k candidates in parallel.
// What bounds it: latency (16 prompts on 200k centres read 2.4 MB from L2). A k-list per thread in
// scratch memory with k block-wide minima per block, and the candidates one after the other, took
// 165 + 57 us for 16 prompts, k = 10 and 200k centres; this takes 23 + 11 us
// (64 prompts, k = 32 and 1M centres: 5290 + 395 us and 115 + 17 us). Centres that lie in falling order
// of their distance make every one a new nearest: one prompt on 1M of them took 124 us a call with the
// thread's lists, 317 with waves that took each key in the order it came in, and takes 90 with the
// rounds and lanes visited out of order (77 on centres in no order).
//
// Compiled without floating-point contraction: the distances and depths decide
// which Gaussians are chosen, and they are evaluated in binary32 in a fixed
// order, so an independent implementation with the same order makes the same
// choice.
#include "fs_internal.h"

namespace fs {
namespace {

constexpr int kMaxK = 32;

struct PromptCam {
    float R[9], t[3], fx, fy, cx, cy;
};

// world point of pixel (px, py) at camera depth d: R^T (d * K^-1 [px, py, 1] - t)
__device__ __forceinline__ void back_project(const PromptCam &c, float px, float py, float d, float &X, float &Y,
                                             float &Z)
{
#pragma clang fp contract(off)
    const float xc = d * ((px - c.cx) / c.fx) - c.t[0];
    const float yc = d * ((py - c.cy) / c.fy) - c.t[1];
    const float zc = d - c.t[2];
    X = (c.R[0] * xc + c.R[3] * yc) + c.R[6] * zc;
    Y = (c.R[1] * xc + c.R[4] * yc) + c.R[7] * zc;
    Z = (c.R[2] * xc + c.R[5] * yc) + c.R[8] * zc;
}

// key = (float bits of the squared distance) << 32 | id: non-negative floats
// order like their bit patterns, ties go to the smaller id
__device__ __forceinline__ unsigned long long dist_key(float X, float Y, float Z, float mx, float my, float mz,
                                                       uint32_t id)
{
#pragma clang fp contract(off)
    const float dx = mx - X, dy = my - Y, dz = mz - Z;
    const float d2 = (dx * dx + dy * dy) + dz * dz;
    return ((unsigned long long)__float_as_uint(d2) << 32) | id;
}

__device__ __forceinline__ unsigned long long read_lane(unsigned long long v, int lane)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
    return ((unsigned long long)hi << 32) | lo;
}

// the value of the lane before (lane 0 keeps its own)
__device__ __forceinline__ unsigned long long lane_before(unsigned long long v)
{
    const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
    const uint32_t l = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, 0x138, 0xF, 0xF, false);  // wave_shr:1
    const uint32_t h = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, 0x138, 0xF, 0xF, false);
    return ((unsigned long long)h << 32) | l;
}

// Takes the lanes' keys into the wave's list: lane i < k holds its i-th smallest key so far
// (~0 where there are fewer, and in the lanes from k on). Every lane of the wave calls it.
__device__ __forceinline__ void wave_take(unsigned long long &list, int k, unsigned long long key)
{
    const int lane = threadIdx.x & 63;
    unsigned long long kth = read_lane(list, k - 1);
    unsigned long long todo = __ballot(key < kth);
    for (bool top = false; todo; top = !top) {  // from both ends: few are taken also if they rise or fall
        const int j = top ? 63 - __clzll((long long)todo) : __ffsll((long long)todo) - 1;
        const unsigned long long c = read_lane(key, j);
        const int pos = __popcll(__ballot(list < c));
        const unsigned long long up = lane_before(list);
        list = lane < pos || lane >= k ? list : (lane == pos ? c : up);
        kth = read_lane(list, k - 1);
        todo &= ~(1ull << j) & __ballot(key < kth);
    }
}

// Calls f(r) once for every r in [0, n), stepping through the range by the golden section. A
// key below all those before it costs the wave an insertion, and centres that lie in the order
// of their distance (falling with the index) would be inserted one by one: in this order only
// about log n rounds hold nearer ones than those before.
template <class F>
__device__ __forceinline__ void golden_order(uint32_t n, F f)
{
    const uint32_t m = n > 1 ? 1u << (32 - __clz((int)(n - 1))) : n;  // a power of two, so any odd step visits all
    const uint32_t step = (uint32_t)(((uint64_t)m * 2654435769u) >> 32) | 1u;
    for (uint32_t i = 0, r = 0; i < m; ++i, r = (r + step) & (m - 1))
        if (r < n) f(r);
}

// the waves' lists merged into that of wave 0
__device__ __forceinline__ void block_merge(unsigned long long &list, int k, unsigned long long (*s_lists)[kMaxK])
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane < k) s_lists[w][lane] = list;
    __syncthreads();
    if (w == 0)
        for (int i = 1; i < 4; ++i) wave_take(list, k, lane < k ? s_lists[i][lane] : ~0ull);
}

__global__ __launch_bounds__(256) void k_knn_partial(GaussPtrs g, int64_t n, PromptCam ref,
                                                     const float *__restrict__ prompts, int32_t k,
                                                     unsigned long long *__restrict__ part)
{
    __shared__ unsigned long long s_lists[4][kMaxK];
    const float *pr = prompts + 3 * (int64_t)blockIdx.y;
    float X, Y, Z;
    back_project(ref, pr[0], pr[1], pr[2], X, Y, Z);
    unsigned long long list = ~0ull;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int lane = threadIdx.x & 63;
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x - lane;  // the wave's
    // four centres per lane in flight; the same rounds for every lane of a wave
    golden_order(first < n ? (uint32_t)((n - first + 4 * stride - 1) / (4 * stride)) : 0u, [&](uint32_t r) {
        const int64_t at = first + (int64_t)r * 4 * stride + lane;
        float x[4], y[4], z[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = at + q * stride;
            x[q] = i < n ? g.mx[i] : 0.0f;
            y[q] = i < n ? g.my[i] : 0.0f;
            z[q] = i < n ? g.mz[i] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = at + q * stride;
            wave_take(list, k, i < n ? dist_key(X, Y, Z, x[q], y[q], z[q], (uint32_t)i) : ~0ull);
        }
    });
    block_merge(list, k, s_lists);
    if (threadIdx.x < (unsigned)k) part[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * k + threadIdx.x] = list;
}

__global__ __launch_bounds__(256) void k_knn_final(const unsigned long long *__restrict__ part, int32_t n_part,
                                                   GaussPtrs g, PromptCam ref, int32_t k,
                                                   const ViewDev *__restrict__ views, int32_t n_views, float znear,
                                                   long long *__restrict__ out_ids, float *__restrict__ out_uv,
                                                   uint8_t *__restrict__ out_vis)
{
    __shared__ unsigned long long s_lists[4][kMaxK];
    __shared__ long long s_chosen;
    const int64_t prompt = blockIdx.x;
    const int lane = threadIdx.x & 63;
    part += prompt * n_part;
    out_ids += prompt * (1 + k);
    out_uv += prompt * n_views * 2;
    out_vis += prompt * n_views;
    unsigned long long list = ~0ull;
    const int first = threadIdx.x - lane;
    golden_order(first < n_part ? (uint32_t)((n_part - first + 255) / 256) : 0u, [&](uint32_t r) {
        const int i = first + (int)r * 256 + lane;
        wave_take(list, k, i < n_part ? part[i] : ~0ull);
    });
    block_merge(list, k, s_lists);
    if (threadIdx.x < 64) {
        // among the k nearest centres, the one of least positive depth in the reference view
        // (ties to the smaller id): positive floats order like their bit patterns
        const bool have = lane < k && list != ~0ull;
        const uint32_t id = (uint32_t)(list & 0xFFFFFFFFull);
        unsigned long long best = ~0ull;
        if (have) {
            const float z = ((ref.R[6] * g.mx[id] + ref.R[7] * g.my[id]) + ref.R[8] * g.mz[id]) + ref.t[2];
            if (z > 0.0f) best = ((unsigned long long)__float_as_uint(z) << 32) | id;
        }
        if (lane < k) out_ids[1 + lane] = have ? (long long)id : -1;
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long o = __shfl_xor(best, off);
            best = o < best ? o : best;
        }
        if (lane == 0) {
            const long long c = best == ~0ull ? -1 : (long long)(best & 0xFFFFFFFFull);
            out_ids[0] = c;
            s_chosen = c;
        }
    }
    __syncthreads();
    const long long c = s_chosen;
    for (int v = threadIdx.x; v < n_views; v += blockDim.x) {
        float u = 0.0f, w = 0.0f;
        uint8_t vis = 0;
        if (c >= 0) {
            const ViewDev &C = views[v];
            const float mx = g.mx[c], my = g.my[c], mz = g.mz[c];
            const float x = ((C.R[0] * mx + C.R[1] * my) + C.R[2] * mz) + C.t[0];
            const float y = ((C.R[3] * mx + C.R[4] * my) + C.R[5] * mz) + C.t[1];
            const float z = ((C.R[6] * mx + C.R[7] * my) + C.R[8] * mz) + C.t[2];
            if (z > znear) {
                u = C.fx * (x / z) + C.cx;
                w = C.fy * (y / z) + C.cy;
                vis = (u >= 0.0f && u < (float)C.W && w >= 0.0f && w < (float)C.H) ? 1 : 0;
            }
        }
        out_uv[2 * v] = u;
        out_uv[2 * v + 1] = w;
        out_vis[v] = vis;
    }
}

}  // namespace

int prompt_max_k() { return kMaxK; }

hipError_t launch_prompt(hipStream_t s, const GaussPtrs &g, int64_t n, const ViewDev *views, int32_t n_views,
                         const ViewDev &ref_host, const float *prompts, int32_t n_prompts, int32_t k, float znear,
                         unsigned long long *part, int32_t n_part_blocks, long long *out_ids, float *out_uv,
                         uint8_t *out_vis)
{
    if (n_prompts == 0) return hipSuccess;
    PromptCam rc;
    for (int i = 0; i < 9; ++i) rc.R[i] = ref_host.R[i];
    for (int i = 0; i < 3; ++i) rc.t[i] = ref_host.t[i];
    rc.fx = ref_host.fx;
    rc.fy = ref_host.fy;
    rc.cx = ref_host.cx;
    rc.cy = ref_host.cy;
    hipLaunchKernelGGL(k_knn_partial, dim3((unsigned)n_part_blocks, (unsigned)n_prompts), dim3(256), 0, s, g, n, rc,
                       prompts, k, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_knn_final, dim3((unsigned)n_prompts), dim3(256), 0, s, part, n_part_blocks * k, g, rc, k,
                       views, n_views, znear, out_ids, out_uv, out_vis);
    return hipGetLastError();
}

}  // namespace fs
