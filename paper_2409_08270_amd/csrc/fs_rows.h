// Row tiles of A, shared by the assignment, the bias sweep and the diagnostics.
//
// A is row-major [n][E] (one row per Gaussian) and what these kernels write or read beside it
// (labels, margins) is [E][n]. A block of 256 threads takes R = 4 * 2^gsh consecutive rows,
// stages them in LDS as float64 (A_hi + A_lo) with loads that run along the rows, and then works
// object by object: a thread takes 4 consecutive rows of one object, so that a byte per row goes
// out as one dword and a float per row as 16 bytes, and consecutive lanes write consecutive
// addresses.
//
// LDS layout: element (row r, object e) at e * row_stride + row_pos(r). The four rows of a thread
// lie a quarter of the tile apart, so consecutive lanes read consecutive doubles, and the odd
// stride spreads the staging's writes (consecutive e) over the banks.
#pragma once

#include <string.h>

#include "fs_internal.h"

namespace fs {

struct RowTile {
    int32_t gsh;   // log2 of the 4-row groups per tile
    int32_t rows;  // 4 << gsh
};

// Largest tile whose staged rows fit `doubles` of LDS: at most 4 << max_gsh rows, at least 4.
inline RowTile row_tile(int32_t E, int32_t doubles, int32_t max_gsh = 6)
{
    RowTile t{max_gsh, 4 << max_gsh};
    while (t.gsh > 0 && (int64_t)E * (t.rows + 1) > doubles) {
        t.gsh -= 1;
        t.rows >>= 1;
    }
    return t;
}

// Tile of this workgroup. Workgroups go to the chip's 8 XCDs in turn; this gives each XCD one
// contiguous run of tiles, so that neighbouring tiles' partial lines of the [E][n] outputs meet in
// one L2.
__device__ __forceinline__ int64_t tile_of_block()
{
    const uint32_t nb = gridDim.x, x = blockIdx.x & 7u;
    return (int64_t)x * (nb >> 3) + min(x, nb & 7u) + (blockIdx.x >> 3);
}

__device__ __forceinline__ int row_pos(int r, int gsh) { return ((r & 3) << gsh) + (r >> 2); }

// Stages rows [r0, r0 + R) (R <= t.rows valid ones, the rest as zeros). get4(i, m, v) gives the
// m (1 to 4) elements from element i of the row-major A; i is a multiple of 4. Ends with a barrier.
template <class Get4>
__device__ __forceinline__ void stage_rows(double *s_a, int64_t r0, int R, int E, RowTile t, Get4 get4)
{
    const int tid = threadIdx.x, rs = t.rows + 1;
    const int64_t base = r0 * E;  // r0 is a multiple of 4
    // (r, e) of element i advance with i
    int r = 4 * tid / E, e = 4 * tid - r * E;
    const int qd = 1024 / E, qm = 1024 - qd * E;
    const int total = t.rows * E, valid = R * E;
    for (int i = 4 * tid; i < total; i += 1024) {
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        if (i < valid) get4(base + i, min(4, valid - i), v);
        int rj = r, ej = e;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            s_a[ej * rs + row_pos(rj, t.gsh)] = v[j];
            if (++ej == E) {
                ej = 0;
                ++rj;
            }
        }
        r += qd;
        e += qm;
        if (e >= E) {
            e -= E;
            ++r;
        }
    }
    __syncthreads();
}

__device__ __forceinline__ bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// m (1 to 4) floats from p, 16 bytes at once where p allows it (`vec`: the array is 16-byte aligned)
__device__ __forceinline__ float4 load_floats4(const float *p, int m, bool vec)
{
    if (vec && m == 4) return *reinterpret_cast<const float4 *>(p);
    return make_float4(p[0], m > 1 ? p[1] : 0.0f, m > 2 ? p[2] : 0.0f, m > 3 ? p[3] : 0.0f);
}

// A_hi + A_lo (A_lo may be NULL)
__device__ __forceinline__ void load_a4(const float *A_hi, const float *A_lo, bool vec, int64_t i, int m, double (&v)[4])
{
    const float4 h = load_floats4(A_hi + i, m, vec);
    const float4 l = A_lo ? load_floats4(A_lo + i, m, vec) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    v[0] = (double)h.x + (double)l.x;
    v[1] = (double)h.y + (double)l.y;
    v[2] = (double)h.z + (double)l.z;
    v[3] = (double)h.w + (double)l.w;
}

// total of the row at position pos, in order e = 0, 1, ...; unrolled so that several LDS reads
// are in flight
__device__ __forceinline__ double row_total(const double *s_a, int pos, int E, RowTile t)
{
    const int rs = t.rows + 1;
    double tot = 0.0;
#pragma unroll 8
    for (int e = 0; e < E; ++e) tot += s_a[e * rs + pos];
    return tot;
}

// a / s and o / s from one reciprocal (s in the range of sums of A, at least 1e-12): the same
// refinement that a division uses, without the scaling that only extreme exponents need
__device__ __forceinline__ void divide2(double a, double o, double s, double &qa, double &qo)
{
    double r = __builtin_amdgcn_rcp(s);
    r = fma(r, fma(-s, r, 1.0), r);
    r = fma(r, fma(-s, r, 1.0), r);
    qa = a * r;
    qa = fma(fma(-s, qa, a), r, qa);
    qo = o * r;
    qo = fma(fma(-s, qo, o), r, qo);
}

// (a_n, o_n) of an object's share a of a row with total tot
__device__ __forceinline__ void normalise(double a, double tot, double &an, double &on)
{
    double o = tot - a;
    if (o < 0.0) o = 0.0;
    divide2(a, o, fmax(a + o, 1e-12), an, on);
}

// 4 consecutive bytes / floats at any address of their own alignment
__device__ __forceinline__ uint32_t load_bytes4(const uint8_t *p)
{
    uint32_t v;
    memcpy(&v, p, 4);
    return v;
}
__device__ __forceinline__ void store_bytes4(uint8_t *p, uint32_t v) { memcpy(p, &v, 4); }
__device__ __forceinline__ void store_floats4(float *p, const float4 v) { memcpy(p, &v, 16); }

}  // namespace fs
