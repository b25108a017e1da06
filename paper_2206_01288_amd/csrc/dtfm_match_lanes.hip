// Eq. 3 for stages of at most 8 devices: a lane takes two blocks of a candidate by the min-max programme over
// column subsets that the 64-device kernels use (g[S] = min over c in S of max(g[S - c], w[row][c]), row by row; the table in
// registers with compile-time indices, the two blocks in the halves of each). Its length does not depend on the data: 1016
// maxima and 448 minima for two blocks of 8 rows in every lane, 18 vector instructions of a wavefront a block with the gathers, where the searches
// of k_match16, four blocks a wavefront, take 200 to 300. Codes (2 + rank, N <= 128: at most 8130) are halves in the order of the
// integers; the table of them is in LDS. Whole evaluations, by k_match and k_match16 (this way): 4000 allocations of 9 stages of 8
// 120 (63) us, 30,000 of 5 stages of 8 177 (57), 30,000 of 16 stages of 8 2719 (1496), 4000 of 8 stages of 4 53 (30).
#include "dtfm_fast64_device.h"

#include <math.h>

namespace {

constexpr int LANES_THREADS = 256;

template <int D>
__global__ void __launch_bounds__(LANES_THREADS)
k_match_lanes(const uint16_t *__restrict__ Wcode, const double *__restrict__ rank_val, const int32_t *__restrict__ perm, int N,
              int D_pp, double *__restrict__ ghat, uint32_t P, int inc_j, int inc_jp, int pairs)
{
    extern __shared__ uint16_t table[];   // rows N + 2 (N + 1) codes apart: not all in the same banks
    __shared__ uint16_t ends[120];        // the stages of every pair of the launch
    const int stride = N + 2 - (N & 1);
    for (int e = threadIdx.x; e < N * N; e += LANES_THREADS) {
        const int d = e / N;
        table[d * stride + (e - d * N)] = Wcode[e];
    }
    for (int t = threadIdx.x; t < pairs; t += LANES_THREADS) {
        int j1, j2;
        dtfm_match_pair(t, D_pp, inc_j, inc_jp, j1, j2);
        ends[t] = (uint16_t)(j1 << 8 | j2);
    }
    __syncthreads();
    const uint32_t couples = ((uint32_t)pairs + 1u) / 2u, last = (uint32_t)N - 1u;
    const size_t items = (size_t)P * couples;
    for (size_t it = (size_t)blockIdx.x * LANES_THREADS + threadIdx.x; it < items; it += (size_t)gridDim.x * LANES_THREADS) {
        const size_t p = it / couples;
        const int t0 = 2 * (int)(it - p * couples), t1 = min(t0 + 1, pairs - 1);   // an odd one out is matched twice
        const int e0 = ends[t0], e1 = ends[t1];
        const int32_t *row = perm + p * N;
        uint32_t dev[2][D], col[2][D];
#pragma unroll
        for (int i = 0; i < D; i++) {
            dev[0][i] = min((uint32_t)row[(e0 >> 8) * D + i], last) * (uint32_t)stride;
            dev[1][i] = min((uint32_t)row[(e1 >> 8) * D + i], last) * (uint32_t)stride;
            col[0][i] = min((uint32_t)row[(e0 & 255) * D + i], last);
            col[1][i] = min((uint32_t)row[(e1 & 255) * D + i], last);
        }
        uint32_t G[1 << D];
#pragma unroll
        for (int r = 0; r < D; r++) {
            uint32_t w[D];
#pragma unroll
            for (int c = 0; c < D; c++) w[c] = pack2(table[dev[0][r] + col[0][c]], table[dev[1][r] + col[1][c]]);
#pragma unroll
            for (int i = 0; i < BINOM8[r + 1]; i++) {
                const int S = LAYER.s[r + 1][i];
                if (S >> D) continue;   // the sets of the first D columns
                uint32_t acc = 0;
                bool first = true;
#pragma unroll
                for (int c = 0; c < D; c++) {
                    if (!(S & (1 << c))) continue;
                    const uint32_t m = r == 0 ? w[c] : pk_max<true>(G[S ^ (1 << c)], w[c]);
                    acc = first ? m : pk_min<true>(acc, m);
                    first = false;
                }
                G[S] = acc;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const uint32_t g = G[(1 << D) - 1];
        const double v0 = rank_val[(g & 0xFFFFu) - 2u], v1 = rank_val[(g >> 16) - 2u];
        double *to = ghat + p * (size_t)(D_pp * D_pp);
        to[(e0 >> 8) * D_pp + (e0 & 255)] = v0;
        to[(e0 & 255) * D_pp + (e0 >> 8)] = v0;
        to[(e1 >> 8) * D_pp + (e1 & 255)] = v1;
        to[(e1 & 255) * D_pp + (e1 >> 8)] = v1;
    }
}

}  // namespace

int dtfm_match_lanes_enqueue(const dtfm_problem *pr, const int32_t *perm, size_t rows, int pairs, double *ghat, int inc_j, int inc_jp,
                             hipStream_t st)
{
    const int N = pr->N, D = pr->D_dp;
    auto kern = D == 1 ? k_match_lanes<1> : D == 2 ? k_match_lanes<2> : D == 3 ? k_match_lanes<3> : D == 4 ? k_match_lanes<4>
              : D == 5 ? k_match_lanes<5> : D == 6 ? k_match_lanes<6> : D == 7 ? k_match_lanes<7> : k_match_lanes<8>;
    const size_t items = rows * (size_t)((pairs + 1) / 2), blocks = (items + LANES_THREADS - 1) / LANES_THREADS;
    const unsigned grid = (unsigned)(blocks < 2048 ? blocks : 2048);   // a table is loaded for many blocks
    hipLaunchKernelGGL(kern, dim3(grid), dim3(LANES_THREADS), (size_t)N * (N + 2) * sizeof(uint16_t), st, pr->W_code, pr->rank_val, perm,
                       N, pr->D_pp, ghat, (uint32_t)rows, inc_j, inc_jp, pairs);
    DTFM_HIP(hipGetLastError());
    return DTFM_OK;
}
