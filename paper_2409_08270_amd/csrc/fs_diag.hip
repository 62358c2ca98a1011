// Per-Gaussian diagnostics of a solved scene (the supplement's "Scene
// segmentation extension", its count of the objects each Gaussian contributes
// to, and the fewer-masks ablation of Sec. 4.8):
//   contrib[c]  Gaussians with exactly c objects e whose A[g][e] exceeds
//               rel_eps times the row's total (c = 0 also holds unseen rows);
//   member[m]   Gaussians that belong to exactly m rows of S (m > 1 happens
//               only for a negative bias, where the subsets may overlap);
//   overlap[e]  |S_e and gt = e|, |S_e|, |gt = e| against per-Gaussian labels,
//               from which a caller forms the IoU of each object.
// One read of A, S and gt. A block works through several row tiles (fs_rows.h) and adds its
// histograms once to one of up to 8 global copies (the host adds those up): atomics on one
// address take about 18 ns each, one after the other. A row tile's labels are read as dwords, 4 rows of one
// object per lane; an object's members are counted from wave masks. 1M rows of 17 classes: 161 us
// with a block per 240 rows and a row per thread, 48 us now (58 with 1792 blocks, which leave a CU
// waiting for one tile after the other; 138 with 4096 blocks and one copy).
#include "fs_rows.h"

namespace fs {
namespace {

constexpr int kDiagLds = 2304;     // most doubles of staged rows
constexpr int kDiagBlocks = 4096;

// 1 in each byte of x that is not zero
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t x)
{
    return ((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u) >> 7;
}

__global__ __launch_bounds__(256) void k_diag_rows(const float *__restrict__ A_hi, const float *__restrict__ A_lo,
                                                   const uint8_t *__restrict__ S, const int32_t *__restrict__ gt,
                                                   int64_t n, int32_t E, RowTile tl, double rel_eps, int64_t stripe,
                                                   int32_t n_stripes,
                                                   unsigned long long *__restrict__ contrib,
                                                   unsigned long long *__restrict__ member,
                                                   unsigned long long *__restrict__ overlap)
{
    extern __shared__ double s_a[];
    __shared__ uint32_t s_c[kMaxDiagE + 1], s_m[kMaxDiagE + 1], s_o[3 * kMaxDiagE];
    __shared__ uint32_t s_rowm[256];  // memberships of each row of the tile
    const int tid = threadIdx.x, lane = tid & 63, rs = tl.rows + 1, gs = 1 << tl.gsh;
    for (int i = tid; i <= E; i += 256) s_c[i] = s_m[i] = 0;
    for (int i = tid; i < 3 * E; i += 256) s_o[i] = 0;
    const bool vec = aligned16(A_hi) && aligned16(A_lo);
    const unsigned long long mine = (gs == 64 ? ~0ull : (1ull << gs) - 1ull) << (lane & ~(gs - 1));
    const bool head = (lane & (gs - 1)) == 0;
    const int items = E << tl.gsh;
    const int64_t tiles = (n + tl.rows - 1) / tl.rows;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t r0 = tile * tl.rows;
        const int R = (int)min((int64_t)tl.rows, n - r0);
        __syncthreads();  // the previous tile's rows have been read
        s_rowm[tid] = 0;
        if (A_hi)
            stage_rows(s_a, r0, R, E, tl,
                       [&](int64_t i, int m, double (&v)[4]) { load_a4(A_hi, A_lo, vec, i, m, v); });
        else
            __syncthreads();
        if (A_hi && tid < tl.rows && ((tid & (gs - 1)) << 2) + (tid >> tl.gsh) < R) {
            const double thr = rel_eps * row_total(s_a, tid, E, tl);
            int c = 0;
#pragma unroll 8
            for (int e = 0; e < E; ++e) c += s_a[e * rs + tid] > thr ? 1 : 0;
            atomicAdd(&s_c[c], 1u);
        }
        if (S) {
            for (int i0 = tid - lane; i0 < items; i0 += 256) {  // wave by wave: the masks need every lane
                const int i = min(i0 + lane, items - 1);
                const int e = i >> tl.gsh, g = i & (gs - 1);
                const int left = i0 + lane < items ? R - 4 * g : 0;
                const uint8_t *p = S + (int64_t)e * n + r0 + 4 * g;
                uint32_t x = 0;
                if (left >= 4) {
                    x = load_bytes4(p);
                } else {
                    for (int j = 0; j < left; ++j) x |= (uint32_t)p[j] << (8 * j);
                }
                const uint32_t nz = nonzero_bytes(x);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((nz >> (8 * j)) & 1u) atomicAdd(&s_rowm[4 * g + j], 1u);
                if (gt) {
                    uint32_t members = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        members += (uint32_t)__popcll(__ballot((nz >> (8 * j)) & 1u) & mine);
                    if (head && members) atomicAdd(&s_o[3 * e + 1], members);
                }
            }
            __syncthreads();
            if (tid < R) {
                atomicAdd(&s_m[s_rowm[tid]], 1u);
                const int32_t truth = gt ? gt[r0 + tid] : -1;
                if (truth >= 0 && truth < E) {
                    atomicAdd(&s_o[3 * truth + 2], 1u);
                    if (S[(int64_t)truth * n + r0 + tid] != 0) atomicAdd(&s_o[3 * truth], 1u);
                }
            }
        }
    }
    __syncthreads();
    const int64_t copy = stripe * (blockIdx.x % (uint32_t)n_stripes);
    for (int i = tid; i <= E; i += 256) {
        if (contrib && s_c[i]) atomicAdd(&contrib[copy + i], (unsigned long long)s_c[i]);
        if (member && s_m[i]) atomicAdd(&member[copy + i], (unsigned long long)s_m[i]);
    }
    for (int i = tid; i < 3 * E; i += 256)
        if (overlap && s_o[i]) atomicAdd(&overlap[copy + i], (unsigned long long)s_o[i]);
}

unsigned diag_blocks(int64_t n, RowTile tl)
{
    const int64_t tiles = (n + tl.rows - 1) / tl.rows;
    return (unsigned)(tiles < kDiagBlocks ? tiles : kDiagBlocks);
}

}  // namespace

// The blocks queue at a copy's addresses, and every copy is cleared, read back and added up: the
// two balance near copies^2 = 8 * blocks / words. Calls of 5000 rows (contributions alone, 256
// classes, 625 blocks) take 40 us with 2 copies and 52 with 8, of 1.5M (17 classes, 4096 blocks)
// 67 and 59.
int32_t diag_stripes(int64_t n, int32_t E, int64_t words)
{
    const int64_t blocks = diag_blocks(n, row_tile(E, kDiagLds));
    int32_t s = 1;
    while (s < 8 && 4 * s * s * words <= 8 * blocks) s *= 2;
    return s;
}

hipError_t launch_diag_rows(hipStream_t s, const float *A_hi, const float *A_lo, const uint8_t *S, const int32_t *gt,
                            int64_t n, int32_t E, double rel_eps, int64_t stripe, int32_t n_stripes,
                            unsigned long long *contrib, unsigned long long *member, unsigned long long *overlap)
{
    if (n == 0) return hipSuccess;
    const RowTile tl = row_tile(E, kDiagLds);
    const unsigned blocks = diag_blocks(n, tl);
    const size_t lds = (size_t)E * (tl.rows + 1) * 8;
    hipLaunchKernelGGL(k_diag_rows, dim3(blocks), dim3(256), lds, s, A_hi, A_lo, S, gt, n, E, tl, rel_eps, stripe,
                       n_stripes, contrib, member, overlap);
    return hipGetLastError();
}

}  // namespace fs
