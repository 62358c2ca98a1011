// a7: closed-form assignment (paper Sec. 3.2 Eq. (7) and the background
// bias of "Regularized ILP for Noise Reduction"; Sec. 3.3 Eq. (8); Listing 1
// of the supplement). For Gaussian g and object t: a = A[g][t], o = sum of the other
// objects' contributions, (o_n, a_n) = (o, a) / max(o + a, 1e-12);
// S[t][g] = a_n > o_n + gamma (ties go to "others", the first index of the
// argmax); margin = |a_n - o_n - gamma|.
//
// The row total is formed once and reused for every object (the reuse the
// paper calls dynamic programming), in float64 from A_hi + A_lo: o = total - a
// is then exact to about 1e-16 of the row sum.
//
// Memory: row tiles of fs_rows.h. What bounds it: HBM. 3M rows of 64 classes with margins move
// 2.5 GB in 544 us, 4.6 TB/s (a copy reaches 4.75); with one element per lane and two divisions
// each 800 us. Small tiles keep seven or eight blocks on a CU: 4160 staged doubles take twice as long
// as 2304. 2568 give 5, 9, 18 to 19, 36 to 39 and 70 to 77 classes the next larger tile: 1.5M rows of
// 36 classes take 169 us (122 without margins) instead of 226 (183).
#include "fs_rows.h"

namespace fs {
namespace {

constexpr int kLdsDoubles = 2568;  // most staged doubles: 20 KiB, seven blocks per CU

// log2 of the most groups of 4 rows per tile: 256 rows; fewer, down to 64, for a block on each of
// 256 CUs, and 512 where 1024 blocks are left with them (with 2 classes 256 rows only fill half of a
// block's threads: 1.5M rows with margins take 16.4 us instead of 27.7; with 512 rows 5000 rows
// would take 5.8 us instead of 4.9)
int32_t max_groups(int64_t n)
{
    int32_t g = n >= (1 << 19) ? 7 : 6;
    while (g > 4 && n < ((int64_t)256 << (g + 2))) --g;
    return g;
}

// WIDE: the rows come from the float64 totals `wide`; A_hi and A_lo are set from them on the
// way, and the labels use the values they then hold.
// Rows are taken one per thread, in K rounds (tiles of at most 256 K rows).
template <bool WIDE, int K>
__global__ __launch_bounds__(256) void k_assign(float *__restrict__ A_hi, float *__restrict__ A_lo, int64_t n,
                                                int32_t E, RowTile tl, float gamma, uint8_t *__restrict__ S,
                                                float *__restrict__ margin, unsigned long long *__restrict__ status,
                                                const double *__restrict__ wide)
{
    // as large as this launch needs, for more blocks per CU
    extern __shared__ double s_a[];
    double *const s_tot = s_a + E * (tl.rows + 1);
    uint32_t *const s_members = reinterpret_cast<uint32_t *>(s_tot + tl.rows);
    __shared__ uint32_t s_cnt[3];
    const int64_t r0 = tile_of_block() * tl.rows;
    const int R = (int)min((int64_t)tl.rows, n - r0);
    const int tid = threadIdx.x, rs = tl.rows + 1;
    if (tid < 3) s_cnt[tid] = 0;
    const bool vec = aligned16(A_hi) && aligned16(A_lo) && aligned16(wide);
    stage_rows(s_a, r0, R, E, tl, [&](int64_t i, int m, double (&v)[4]) {
        if constexpr (WIDE) {
            float hi[4], lo[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                wide_split(j < m ? wide[i + j] : 0.0, hi[j], lo[j]);
                v[j] = (double)hi[j] + (double)lo[j];
            }
            if (vec && m == 4) {
                *reinterpret_cast<float4 *>(A_hi + i) = make_float4(hi[0], hi[1], hi[2], hi[3]);
                *reinterpret_cast<float4 *>(A_lo + i) = make_float4(lo[0], lo[1], lo[2], lo[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (j >= m) break;
                    A_hi[i + j] = hi[j];
                    A_lo[i + j] = lo[j];
                }
            }
        } else {
            load_a4(A_hi, A_lo, vec, i, m, v);
        }
    });
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int pos = tid + 256 * k;
        if (pos >= tl.rows) break;
        const double tot = row_total(s_a, pos, E, tl);
        s_tot[pos] = tot;
        s_members[pos] = 0;
        const int r = ((pos & ((1 << tl.gsh) - 1)) << 2) + (pos >> tl.gsh);  // the row at this position
        if (tot == 0.0 && r < R) atomicAdd(&s_cnt[0], 1u);
    }
    __syncthreads();
    const double gd = (double)gamma;
    uint32_t low = 0;
    for (int i = tid; i < E << tl.gsh; i += 256) {
        const int t = i >> tl.gsh, g = i & ((1 << tl.gsh) - 1);
        const int left = R - 4 * g;  // valid rows from this thread's first
        if (left <= 0) continue;
        uint32_t lab = 0;
        float m4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int pos = (j << tl.gsh) + g;
            double an, on;
            normalise(s_a[t * rs + pos], s_tot[pos], an, on);
            const bool in = j < left && an > on + gd;
            const double m = fabs(an - on - gd);
            lab |= (in ? 1u : 0u) << (8 * j);
            m4[j] = (float)m;
            if (in) atomicAdd(&s_members[pos], 1u);
            if (j < left && m < 1e-4) low++;
        }
        const int64_t o = (int64_t)t * n + r0 + 4 * g;
        if (left >= 4) {
            store_bytes4(S + o, lab);
            if (margin) store_floats4(margin + o, make_float4(m4[0], m4[1], m4[2], m4[3]));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j >= left) break;
                S[o + j] = (uint8_t)(lab >> (8 * j));
                if (margin) margin[o + j] = m4[j];
            }
        }
    }
    if (low) atomicAdd(&s_cnt[2], low);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tid + 256 * k < tl.rows && s_members[tid + 256 * k] > 1) atomicAdd(&s_cnt[1], 1u);
    __syncthreads();
    if (tid == 0) {
        if (s_cnt[0]) status_add(status, ST_UNSEEN, (unsigned long long)s_cnt[0]);
        if (s_cnt[1]) status_add(status, ST_MULTI, (unsigned long long)s_cnt[1]);
        if (s_cnt[2]) status_add(status, ST_LOWMARGIN, (unsigned long long)s_cnt[2]);
    }
}

}  // namespace

hipError_t launch_assign(hipStream_t s, float *A_hi, float *A_lo, int64_t n, int32_t E, float gamma, uint8_t *S,
                         float *margin, unsigned long long *status, const double *wide)
{
    if (n == 0) return hipSuccess;
    const RowTile tl = row_tile(E, kLdsDoubles, max_groups(n));
    const int64_t blocks = (n + tl.rows - 1) / tl.rows;
    const size_t lds = (size_t)E * (tl.rows + 1) * 8 + (size_t)tl.rows * 12;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), lds, s, A_hi, A_lo, n, E, tl, gamma, S, margin, status,
                           wide);
    };
    if (wide) go(tl.rows > 256 ? k_assign<true, 2> : k_assign<true, 1>);
    else go(tl.rows > 256 ? k_assign<false, 2> : k_assign<false, 1>);
    return hipGetLastError();
}

}  // namespace fs
