// Interactive follow-ups of the assignment (paper Sec. 3.2 "Regularized ILP
// for Noise Reduction", Sec. 4.2 and Sec. 4.4 "Object Removal"): once A is
// known, the background bias gamma can be swept at the cost of reading A once,
// and the Gaussians of an object are extracted or removed by stream compaction.
#include "fs_rows.h"

namespace fs {
namespace {

constexpr int kSweepLds = 4352;       // doubles of staged rows
constexpr int kSweepCounters = 4096;  // n_gamma * E counters per block

// S[k][t][g] = a_n > o_n + gamma_k for every gamma of the sweep, from one read
// of A (same arithmetic as the single assignment); counts[k][t] += members
// (counts may be NULL). Row tiles of fs_rows.h: a thread holds 4 rows of one object
// and writes a dword per bias. A comparison's result is a wave-wide mask, so an object's
// members are counted with scalar bit counts of its lanes' part of the masks.
// What bounds it: the comparisons (float64, one per label) and the label bytes, 448 MB in 158 us
// for 700k rows, 10 classes and 64 biases (560 us with one byte per lane and store). Larger tiles
// than the assignment's give each wave one object up to 16 classes, so that its members are counted
// by scalar instructions: 228 against 273 us a call with 2304 doubles; 4352 of them leave 16 rows at 256
// classes. With many classes a wave writes runs of 16 to 64 bytes of many label rows, and neighbouring
// tiles complete each other's lines: with tiles taken in turn by the XCDs those lines went to memory
// in parts, 700k rows of 128 classes and 32 biases 5.8 ms, 256 and 16 10.4 ms (2.7 and 4.2 with one
// row per lane); in runs of tiles per XCD 2.0 and 2.5 ms, and 64 classes x 64 biases 1.4 ms instead
// of 2.2.
__global__ __launch_bounds__(256) void k_assign_sweep(const float *__restrict__ A_hi, const float *__restrict__ A_lo,
                                                      int64_t n, int32_t E, RowTile tl,
                                                      const float *__restrict__ gammas, int32_t n_gamma,
                                                      uint8_t *__restrict__ S,
                                                      unsigned long long *__restrict__ counts)
{
    // the staged rows, then the counters (as large as this launch needs, for more blocks per CU)
    extern __shared__ double s_a[];
    uint32_t *const s_cnt = reinterpret_cast<uint32_t *>(s_a + E * (tl.rows + 1));
    __shared__ double s_tot[256];
    __shared__ double s_g[64];
    const int64_t r0 = tile_of_block() * tl.rows;
    const int R = (int)min((int64_t)tl.rows, n - r0);
    const int tid = threadIdx.x, rs = tl.rows + 1;
    if (counts)
        for (int i = tid; i < n_gamma * E; i += 256) s_cnt[i] = 0;
    if (tid < n_gamma) s_g[tid] = (double)gammas[tid];
    const bool vec = aligned16(A_hi) && aligned16(A_lo);
    stage_rows(s_a, r0, R, E, tl,
               [&](int64_t i, int m, double (&v)[4]) { load_a4(A_hi, A_lo, vec, i, m, v); });
    if (tid < tl.rows) s_tot[tid] = row_total(s_a, tid, E, tl);
    __syncthreads();
    const int lane = tid & 63, gs = 1 << tl.gsh;
    // the lanes of this lane's object, and whether it is their first
    const unsigned long long mine = (gs == 64 ? ~0ull : (1ull << gs) - 1ull) << (lane & ~(gs - 1));
    const bool head = (lane & (gs - 1)) == 0;
    const int items = E << tl.gsh;
    const int64_t step = (int64_t)E * n;
    // units of work: 64 items for one bias, items first; each wave takes a quarter of the units
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int units = ((items + 63) >> 6) * n_gamma;
    int u = units * w / 4;
    const int u_end = units * (w + 1) / 4;
    while (u < u_end) {
        const int i0 = u / n_gamma * 64, k0 = u % n_gamma;
        const int k1 = min(n_gamma, k0 + u_end - u);
        u += k1 - k0;
        const int i = min(i0 + lane, items - 1);
        const int t = i >> tl.gsh, g = i & (gs - 1);
        const int left = i0 + lane < items ? R - 4 * g : 0;
        double an[4], on[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int pos = (j << tl.gsh) + g;
            normalise(s_a[t * rs + pos], s_tot[pos], an[j], on[j]);
            if (j >= left) an[j] = __builtin_nan("");  // rows past the end: never a member
        }
        uint8_t *out = S ? S + (int64_t)t * n + r0 + 4 * g + k0 * step : nullptr;
        for (int k = k0; k < k1; ++k) {
            const double gk = s_g[k];
            bool in[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) in[j] = an[j] > on[j] + gk;
            if (S) {
                const uint32_t lab = (in[0] ? 1u : 0u) | (in[1] ? 0x100u : 0u) | (in[2] ? 0x10000u : 0u) |
                                     (in[3] ? 0x1000000u : 0u);
                if (left >= 4) {
                    store_bytes4(out, lab);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (j < left) out[j] = (uint8_t)(lab >> (8 * j));
                }
                out += step;
            }
            if (counts) {
                uint32_t members = 0;
                if (gs == 64) {  // the whole wave holds one object: scalar counts
#pragma unroll
                    for (int j = 0; j < 4; ++j) members += (uint32_t)__popcll(__ballot(in[j]));
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) members += (uint32_t)__popcll(__ballot(in[j]) & mine);
                }
                if (head && members) atomicAdd(&s_cnt[k * E + t], members);
            }
        }
    }
    if (!counts) return;
    __syncthreads();
    for (int i = tid; i < n_gamma * E; i += 256)
        if (s_cnt[i]) atomicAdd(&counts[i], (unsigned long long)s_cnt[i]);
}

// Compaction in tiles of kCompactTile Gaussians: the kept ones of each tile are counted, the counts
// scanned, and the copy finds each kept Gaussian's place from its tile's bits. Neither a flag
// nor a position per Gaussian goes through memory, only a bit (so the caller may reuse `select` as soon
// as the count is known). What is left is the copy of the 11 arrays, at the
// rate of a large copy (13 us for 90% of 700k), two short launches and the wait for the count: 63 ->
// 57 us a call.
constexpr int kCompactRounds = kCompactTile / 256;

__device__ __forceinline__ bool keeps(const uint8_t *__restrict__ select, int64_t i, int64_t n, int32_t keep_selected)
{
    return i < n && (select[i] != 0) == (keep_selected != 0);
}

__global__ __launch_bounds__(256) void k_select_sums(const uint8_t *__restrict__ select, int64_t n,
                                                     int32_t keep_selected, uint32_t *__restrict__ sums,
                                                     unsigned long long *__restrict__ bits)
{
    __shared__ uint32_t s_cnt[4];
    const int64_t base = (int64_t)blockIdx.x * kCompactTile + threadIdx.x;
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < kCompactRounds; ++r) {
        const unsigned long long m = __ballot(keeps(select, base + r * 256, n, keep_selected));
        // every tile has all its words, also past n
        if ((threadIdx.x & 63) == 0) bits[((int64_t)blockIdx.x * kCompactRounds + r) * 4 + (threadIdx.x >> 6)] = m;
        c += (uint32_t)__popcll(m);
    }
    if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
}

struct Soa11 {
    const float *in[11];
    float *out[11];
};

__global__ __launch_bounds__(256) void k_compact(Soa11 a, const unsigned long long *__restrict__ bits,
                                                 const uint32_t *__restrict__ offs, int64_t *__restrict__ index_map)
{
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t base = (int64_t)blockIdx.x * kCompactTile + threadIdx.x;
    const unsigned long long *tile_bits = bits + (int64_t)blockIdx.x * kCompactRounds * 4;
    uint32_t at = offs[blockIdx.x];
#pragma unroll
    for (int r = 0; r < kCompactRounds; ++r) {
        uint32_t p = at;
        unsigned long long m = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned long long b = tile_bits[r * 4 + j];
            const uint32_t c = (uint32_t)__popcll(b);
            if (j < w) p += c;
            if (j == w) m = b;
            at += c;
        }
        p += (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if ((m >> lane) & 1ull) {
            const int64_t i = base + r * 256;
#pragma unroll
            for (int k = 0; k < 11; ++k) a.out[k][p] = a.in[k][i];
            if (index_map) index_map[p] = i;
        }
    }
}

unsigned grid_of(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

int sweep_max_gammas(int32_t E) { return kSweepCounters / E < 64 ? kSweepCounters / E : 64; }

hipError_t launch_assign_sweep(hipStream_t s, const float *A_hi, const float *A_lo, int64_t n, int32_t E,
                               const float *gammas_dev, int32_t n_gamma, uint8_t *S, unsigned long long *counts)
{
    if (n == 0 || n_gamma == 0) return hipSuccess;
    const RowTile tl = row_tile(E, kSweepLds);
    const int64_t blocks = (n + tl.rows - 1) / tl.rows;
    const size_t lds = (size_t)E * (tl.rows + 1) * 8 + (counts ? (size_t)n_gamma * E * 4 : 0);
    hipLaunchKernelGGL(k_assign_sweep, dim3((unsigned)blocks), dim3(256), lds, s, A_hi, A_lo, n, E, tl, gammas_dev,
                       n_gamma, S, counts);
    return hipGetLastError();
}

hipError_t launch_select_sums(hipStream_t s, const uint8_t *select, int64_t n, int32_t keep_selected, uint32_t *sums,
                              unsigned long long *bits)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_select_sums, dim3(grid_of(n, kCompactTile)), dim3(256), 0, s, select, n, keep_selected, sums,
                       bits);
    return hipGetLastError();
}

hipError_t launch_compact(hipStream_t s, const float *const in[11], float *const out[11],
                          const unsigned long long *bits, int64_t n, const uint32_t *offs, int64_t *index_map)
{
    if (n == 0) return hipSuccess;
    Soa11 a;
    for (int k = 0; k < 11; ++k) {
        a.in[k] = in[k];
        a.out[k] = out[k];
    }
    hipLaunchKernelGGL(k_compact, dim3(grid_of(n, kCompactTile)), dim3(256), 0, s, a, bits, offs, index_map);
    return hipGetLastError();
}

}  // namespace fs
