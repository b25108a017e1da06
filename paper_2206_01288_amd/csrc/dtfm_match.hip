// Eq. 3 for stages of more than 16 devices: bottleneck perfect matchings on bit masks.
//
// The optimum of a block (the rows: devices of one stage, the columns: of another) is one of its entries and depends on
// their order only, so the ranks of the weights stand for them. Written in base 127 a rank has one to three digits; each
// digit of every entry is a byte of a table of its own (code). A wavefront takes a block, lane = column:
//   digits     the lane gathers the leading digits of its column, a byte an entry (24, 32, 48 or 64 rows: 8 or 16 registers),
//              and the optimum's digit T is sought: the smallest one within which a perfect matching exists.
//   masks      one subtraction compares four bytes with a threshold, so the rows that the column reaches within it are a mask
//              a lane of 32 or 64 bits after 24 or 48 instructions. An alternating-path search then takes a handful of instructions a
//              level, whatever the number of rows in it: the columns reached are the lanes whose mask meets the set of rows
//              (one ballot), the rows matched to them the lanes whose column is among those (another).
//   thresholds start at the digit of the wavefront's last block (or of the edge that a trial changes; the first block: at
//              the usual digit of the problem's blocks, dtfm_match_prepare) and go up after a failed search, down after a
//              success, in growing steps until both bounds are known. A matching stays valid when the threshold rises, and loses
//              the edges above it when it falls, so a step repairs a few rows; where a step down leaves more than a few of
//              them free, they bid again before they are searched for one by one. Networks whose links are all of their own have
//              their optimum at a small digit: with a first threshold of 31 and no second bids 1000 allocations of 8 stages of
//              64 took 217 us (the searches by smallest entries before this kernel 183), now 126; of 8 of 33 128 (76), now 88.
//   ranks      the entries with digit T (some 33 of 4096 on 1024 devices) are told apart by their ranks: a lane lists those of
//              its column, and the rows that the matching below T leaves free are inserted by searches that, when stuck,
//              admit the smallest listed entry from a reached row to a column not yet reached. Reached rows own one column
//              fewer than they need, so the optimum is no smaller; an alternating path to a free column exists within a
//              threshold iff a larger matching does (Berge): the last one admitted is the optimum. Where a lane's list is
//              too short for its entries, their next digits are gathered and searched first.
// The result is mapped back through rank_val: no rounding is involved, and the way taken does not change the value.
// Evaluation of 4096 candidates of 16 stages of 64: 4258 -> 2290 us against greedy pass and search by smallest entries on
// 16-bit codes (3,220 scalar and 2,670 vector instructions a block; here 1,240 and 1,450, and a gather of half the bytes,
// which moves one cache line where that one moved two: 1.43 of the kernel's 1.9 ms are bare gathers).
#include "dtfm_internal.h"

#include <math.h>

#include <algorithm>
#include <type_traits>
#include <vector>

// x with lane `lane` set to value
__device__ int lane_write(int value, int lane, int x) __asm("llvm.amdgcn.writelane.i32");

namespace {

constexpr int LIST = 6;        // entries of a column that are told apart by their ranks
constexpr int BIDS = 5;        // as many free rows are matched by searches of their own, more by rounds of bids first
constexpr int WAVES = 4;       // wavefronts of a workgroup (launches of few blocks: one); they share nothing

__device__ __forceinline__ int first_bit(uint64_t m)   // scalar; -1: empty
{
    int c;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(c) : "s"(m));
    return c;
}
__device__ __forceinline__ int first_bit(uint32_t m)
{
    int c;
    asm("s_ff1_i32_b32 %0, %1" : "=s"(c) : "s"(m));
    return c;
}
__device__ __forceinline__ int lane_first_bit(uint32_t m)   // per lane; m = 0: -1
{
    int c;
    asm("v_ffbl_b32 %0, %1" : "=v"(c) : "v"(m));
    return c;
}
__device__ __forceinline__ int lane_first_bit(uint64_t m)
{
    uint32_t lo, hi;
    asm("v_ffbl_b32 %0, %1" : "=v"(lo) : "v"((uint32_t)m));   // ~0 for 0
    asm("v_ffbl_b32 %0, %1" : "=v"(hi) : "v"((uint32_t)(m >> 32)));
    return (int)min(lo, hi | 32u);
}
__device__ __forceinline__ bool any_bit(uint32_t m) { return m != 0u; }
__device__ __forceinline__ bool any_bit(uint64_t m)   // per lane, on 32-bit instructions: a 64-bit comparison takes longer than two
{
    uint32_t x;
    asm("v_or_b32 %0, %1, %2" : "=v"(x) : "v"((uint32_t)m), "v"((uint32_t)(m >> 32)));
    return x != 0u;
}
__device__ __forceinline__ bool in_lanes(uint64_t m)   // the lane's bit of a mask that is the same in all lanes
{
    return __builtin_amdgcn_inverse_ballot_w64(m);
}
__device__ __forceinline__ uint32_t wave_min(uint32_t k)
{
    k = min(k, (uint32_t)__builtin_amdgcn_update_dpp((int)k, (int)k, 0x111, 0xF, 0xF, false));   // row_shr:1
    k = min(k, (uint32_t)__builtin_amdgcn_update_dpp((int)k, (int)k, 0x112, 0xF, 0xF, false));
    k = min(k, (uint32_t)__builtin_amdgcn_update_dpp((int)k, (int)k, 0x114, 0xF, 0xF, false));
    k = min(k, (uint32_t)__builtin_amdgcn_update_dpp((int)k, (int)k, 0x118, 0xF, 0xF, false));
    const uint32_t m0 = (uint32_t)__builtin_amdgcn_readlane((int)k, 15), m1 = (uint32_t)__builtin_amdgcn_readlane((int)k, 31);
    const uint32_t m2 = (uint32_t)__builtin_amdgcn_readlane((int)k, 47), m3 = (uint32_t)__builtin_amdgcn_readlane((int)k, 63);
    return min(min(m0, m1), min(m2, m3));
}
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A lane's set of rows of a block.
template <int R>
using rowset = std::conditional_t<R <= 32, uint32_t, uint64_t>;

// Registers of a lane's column of R rows: row 8 k + i is byte k of the i-th, row 32 + 8 k + i of the (8 + i)-th.
template <int R>
constexpr int regs = R <= 32 ? 8 : 16;

// Rows whose byte is at most t (t from -1; bytes at most 127), as bits; those from R on have any value.
template <int R>
__device__ __forceinline__ rowset<R> within(const uint32_t (&E)[regs<R>], int t)
{
    const uint32_t top = (uint32_t)(0x80 + t) * 0x01010101u;   // a byte's difference keeps its bit 7 iff the byte is <= t
    uint32_t lo = 0u, hi = 0u;
#pragma unroll
    for (int i = 0; i < 8; i++) lo = (lo >> 1) | ((top - E[i]) & 0x80808080u);
    if constexpr (R > 32)
#pragma unroll
        for (int i = 0; i < 8; i++) hi = (hi >> 1) | ((top - E[8 + i]) & 0x80808080u);
    return (rowset<R>)((uint64_t)hi << 32 | lo);
}

// A matching of the block: free rows and columns as masks, lane b holds the column of row b and the row of column b.
struct matching {
    uint64_t freerows, freecols;
    int col_of, row_of;
};

// the path that ends in the free column c, back to the free row r0; from: the rows that reached the lane's column
template <typename M>
__device__ __forceinline__ void augment(matching &m, M from, int c, int r0)
{
    m.freecols &= ~(1ull << c);
    m.freerows &= ~(1ull << r0);
    int r;
    do {   // to a column reached a turn earlier
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)from, c);
        if constexpr (sizeof(M) == 4) {
            r = first_bit(lo);
        } else {
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(from >> 32), c);
            r = first_bit((uint64_t)hi << 32 | lo);
        }
        const int prev = __builtin_amdgcn_readlane(m.col_of, r);
        m.row_of = lane_write(r, c, m.row_of);
        m.col_of = lane_write(c, r, m.col_of);
        c = prev;
    } while (r != r0);
}

// Matches every free row within the masks; false: no perfect matching (the free rows left stay free).
template <typename M>
__device__ __forceinline__ bool complete(matching &m, M adj)
{
    while (m.freerows != 0ull) {
        const int r0 = first_bit(m.freerows);
        const M col = (M)1 << m.col_of;
        M t = adj & ((M)1 << r0), from = t;
        uint64_t cols = __ballot(any_bit(t)), seen = 0ull, hit = cols & m.freecols;
        while (hit == 0ull && cols != 0ull) {   // a turn reaches a new column or ends the search
            seen |= cols;
            const uint64_t rows = __ballot(any_bit((M)(col & (M)cols))) & ~m.freerows;
            t = adj & (M)rows;
            cols = __ballot(any_bit(t)) & ~seen;
            from = in_lanes(cols) ? t : from;
            hit = cols & m.freecols;
        }
        if (hit == 0ull) return false;
        augment(m, from, first_bit(hit), r0);
    }
    return true;
}

// takes the edges that the masks no longer hold out of the matching
template <typename M>
__device__ __forceinline__ void release(matching &m, M adj, uint64_t columns)
{
    const uint64_t lost = ~__ballot(any_bit((M)(adj & ((M)1 << m.row_of)))) & columns & ~m.freecols;
    const uint64_t rows = __ballot(any_bit((M)((M)lost & ((M)1 << m.col_of)))) & columns & ~m.freerows;
    m.freecols |= lost;
    m.freerows |= rows;
}

// Rounds in which every free column bids for a row it reaches, and the last bid in LDS wins it. The columns look upwards
// from their own number: bids for the lowest rows alone would meet.
template <int R>
__device__ __forceinline__ void bids(matching &m, int lane, rowset<R> adj, uint64_t rows, uint32_t *slot)
{
    using M = rowset<R>;
    const M up = (M)~0ull << (lane & (R <= 32 ? 31 : 63));
    slot[lane] = in_lanes(rows & ~m.freerows) ? (uint32_t)m.col_of : ~0u;
    lds_order();
#pragma unroll
    for (int round = 0; round < 4; round++) {
        const M open = adj & (M)m.freerows, above = open & up;
        const bool bid = any_bit(open) && in_lanes(m.freecols);
        const int r = lane_first_bit(any_bit(above) ? above : open);
        if (bid) slot[r] = (uint32_t)lane;
        lds_order();
        const bool won = bid && slot[r] == (uint32_t)lane;
        m.row_of = won ? r : m.row_of;
        m.freecols &= ~__ballot(won);
        m.freerows = rows & ~__ballot(slot[lane] != ~0u);
    }
    m.col_of = (int)slot[lane] & (R <= 32 ? 31 : 63);
}

// One wavefront after another takes the blocks of stage pair (wavefront mod pairs) of every `chunks`-th candidate.
// R: rows that are gathered (24, 32, 48 or 64), at least D_dp.
template <int R>
__global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(7)))
k_match_bits(dtfm_digits dg, const uint32_t *__restrict__ Wrank, const double *__restrict__ rank_val,
             const int32_t *__restrict__ perm, int N, int D_dp, int D_pp, double *__restrict__ ghat, int P, int inc_j, int inc_jp,
             int pairs, int chunks)
{
    __shared__ uint32_t slots[WAVES][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int id = (int)(blockIdx.x * (blockDim.x >> 6)) + wave;
    const int chunk = id / pairs;
    if (chunk >= chunks) return;
    int j1, j2;
    dtfm_match_pair(id - chunk * pairs, D_pp, inc_j, inc_jp, j1, j2);
    uint32_t *slot = slots[wave];
    const uint64_t all = D_dp >= 64 ? ~0ull : (1ull << D_dp) - 1ull;
    const bool active = lane < D_dp;
    using M = rowset<R>;
    const M mine = active ? (M)all : 0;
    const uint32_t last = (uint32_t)N - 1u;
    double first[2];   // the smallest weight of digits lane and lane + 64
    if (inc_j >= 0) {
        first[0] = dg.first[lane];
        first[1] = dg.first[64 + lane];
    }
    int guess = dg.usual;
    for (int p = chunk; p < P; p += chunks) {
        const int32_t *row = perm + (size_t)p * N, *Ca = row + j1 * D_dp;
        double *G = ghat + (size_t)p * D_pp * D_pp;
        const uint32_t coldev = active ? min((uint32_t)row[j2 * D_dp + lane], last) : 0u;
        if (inc_j >= 0) {   // the digit of the edge that the row had before the trial's swap
            const double v = G[j1 * D_pp + j2];
            guess = max(__popcll(__ballot(first[0] <= v)) + __popcll(__ballot(first[1] <= v)) - 1, 0);
        }
        const uint32_t rowdev = active ? min((uint32_t)Ca[lane], last) : 0u, rowat = rowdev * (uint32_t)N;
        uint32_t E[regs<R>];
        auto gather = [&](int level) {
            const auto W = __builtin_amdgcn_make_buffer_rsrc(dg.code + (size_t)level * N * N, 0, N * N, 0x00027000);
#pragma unroll
            for (int h = 0; 32 * h < R; h++) {   // at most 32 rows in flight
                uint32_t x[32];
#pragma unroll
                for (int b = 0; b < 32; b++)
                    x[b] = 32 * h + b < R ? __builtin_amdgcn_raw_buffer_load_b8(W, (int)coldev, __builtin_amdgcn_readlane((int)rowat, 32 * h + b), 0)
                                          : 0u;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 8; i++) E[8 * h + i] = (x[i] | x[8 + i] << 8) | (x[16 + i] | x[24 + i] << 8) << 16;
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        gather(0);
        matching m = {all, all, 0, 0};
        M low = 0, eq = mine;
        uint32_t result = ~0u;
        for (int level = 0; level < dg.levels; level++) {
            // a matching exists within digit hi, and none within digit lo
            int lo = -1, hi = dg.top[level], t = level == 0 ? guess : hi >> 1, step = 1;
            bool above = level != 0, below = level != 0;   // the bounds are close: halve what lies between
            M upto = low | eq, under = low;                // the masks within hi and lo
            bool fell = false;                             // the matching may hold edges above lo
            while (hi - lo > 1) {
                t = min(max(t, lo + 1), hi - 1);
                const M adj = low | (eq & within<R>(E, t));
                if (fell) release(m, adj, all);
                if (__popcll(m.freerows) > BIDS) bids<R>(m, lane, adj, all, slot);
                fell = complete(m, adj);
                if (fell) {
                    hi = t;
                    upto = adj;
                    above = true;
                } else {
                    lo = t;
                    under = adj;
                    below = true;
                }
                t = above && below ? (lo + hi) >> 1 : above ? t - step : t + step;
                step += step;
            }
            if (fell) release(m, under, all);
            // the entries of digit hi
            low = under;
            eq = upto & ~low;
            if (level == 0) guess = hi;
            if (level + 1 == dg.levels) {   // all of one rank
                const uint64_t who = __ballot(any_bit(eq));
                const int r = any_bit(eq) ? lane_first_bit(eq) : 0;
                const uint32_t d = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * r, (int)rowdev);
                const uint32_t k = any_bit(eq) ? Wrank[d * (uint32_t)N + coldev] : 0u;
                result = (uint32_t)__builtin_amdgcn_readlane((int)k, max(first_bit(who), 0));
                break;
            }
            if (__ballot((R <= 32 ? __popc((uint32_t)eq) : __popcll(eq)) > LIST) != 0ull) {
                gather(level + 1);
                continue;
            }
            uint32_t key[LIST];   // rank and row
#pragma unroll
            for (int q = 0; q < LIST; q++) {
                const bool has = any_bit(eq);
                const int r = has ? lane_first_bit(eq) : 0;
                const uint32_t d = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * r, (int)rowdev);
                key[q] = has ? Wrank[d * (uint32_t)N + coldev] << 6 | (uint32_t)r : ~0u;
                eq &= eq - 1;
            }
            uint32_t rank = 0u;
            M adj = low;
            while (m.freerows != 0ull) {
                const int r0 = first_bit(m.freerows);
                const M col = (M)1 << m.col_of;
                M from = 0;
                uint64_t rows = 1ull << r0, reached = rows, seen = 0ull, hit;
                do {   // a turn reaches a column, or admits an edge to one
                    const M t = adj & (M)rows;
                    const uint64_t cols = __ballot(any_bit(t)) & ~seen;
                    from = in_lanes(cols) ? t : from;
                    hit = cols & m.freecols;
                    seen |= cols;
                    rows = __ballot(any_bit((M)(col & (M)cols))) & ~m.freerows;
                    reached |= rows;
                    if (cols == 0ull) {
                        uint32_t k = ~0u;
#pragma unroll
                        for (int q = 0; q < LIST; q++) k = min(k, (((M)reached >> (key[q] & (R <= 32 ? 31u : 63u))) & 1) != 0 ? key[q] : ~0u);
                        k = in_lanes(seen) ? ~0u : k;
                        const uint32_t least = wave_min(k) >> 6;
                        if (least == ~0u >> 6) break;   // cannot happen: a matching exists within hi
                        rank = max(rank, least);
                        adj |= k >> 6 == least ? (M)1 << (k & (R <= 32 ? 31u : 63u)) : (M)0;
                        rows = reached;
                    }
                } while (hit == 0ull);
                if (hit == 0ull) {
                    rank = ~0u;
                    break;
                }
                augment(m, from, first_bit(hit), r0);
            }
            result = rank;
            break;
        }
        if (lane == 0) {
            const double v = result == ~0u ? INFINITY : rank_val[result];
            G[j1 * D_pp + j2] = v;
            G[j2 * D_pp + j1] = v;
        }
    }
}

// the digits of the ranks, and the smallest weight of every leading digit
__global__ void k_digits(const uint32_t *__restrict__ Wrank, size_t entries, int w1, int w2, int levels, uint8_t *__restrict__ code)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= entries) return;
    const uint32_t r = Wrank[i];
    code[i] = (uint8_t)(r / (uint32_t)w1);
    if (levels > 1) code[entries + i] = (uint8_t)(r % (uint32_t)w1 / (uint32_t)w2);
    if (levels > 2) code[2 * entries + i] = (uint8_t)(r % (uint32_t)w1 % (uint32_t)w2);
}
__global__ void k_digit_first(const double *__restrict__ rank_val, int ranks, int w1, double *__restrict__ first)
{
    const int d = threadIdx.x;
    if (d < 128) first[d] = (long long)d * w1 < ranks ? rank_val[d * w1] : INFINITY;
}

}  // namespace

// The digit that the searches begin at: the usual one of the blocks of random allocations (32 blocks or more); and whether it is
// that of a network whose links are all of their own.
static int dtfm_match_usual(dtfm_problem *pr)
{
    const size_t N = pr->N, n = pr->D_pp, rows = pr->npairs < 1 ? 0 : (32 + pr->npairs - 1) / pr->npairs;
    if (rows == 0) {
        DTFM_HIP(hipDeviceSynchronize());
        return DTFM_OK;
    }
    std::vector<int32_t> perm(rows * N);
    uint32_t x = 1u;
    for (size_t p = 0; p < rows; p++)
        for (size_t q = 0; q < N; q++) {   // a random device of those before gives way
            x = x * 1664525u + 1013904223u;
            const size_t at = (size_t)(((uint64_t)x * (uint64_t)(q + 1)) >> 32);
            perm[p * N + q] = perm[p * N + at];
            perm[p * N + at] = (int32_t)q;
        }
    std::vector<double> first(128), graph(rows * n * n), edges;
    char *mem = nullptr;
    DTFM_HIP(hipMalloc((void **)&mem, graph.size() * sizeof(double) + perm.size() * sizeof(int32_t)));
    double *ghat = reinterpret_cast<double *>(mem);
    int32_t *perm_dev = reinterpret_cast<int32_t *>(mem + graph.size() * sizeof(double));
    int rc = DTFM_OK;
    hipError_t e = hipMemcpy(perm_dev, perm.data(), perm.size() * sizeof(int32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) rc = dtfm_match_bits_enqueue(pr, perm_dev, rows, pr->npairs, ghat, -1, -1, (hipStream_t) nullptr);
    if (e == hipSuccess && rc == DTFM_OK) e = hipMemcpy(graph.data(), ghat, graph.size() * sizeof(double), hipMemcpyDeviceToHost);
    if (e == hipSuccess && rc == DTFM_OK) e = hipMemcpy(first.data(), pr->digits.first, 128 * sizeof(double), hipMemcpyDeviceToHost);
    (void)hipFree(mem);
    if (rc != DTFM_OK) return rc;
    DTFM_HIP(e);
    for (size_t p = 0; p < rows; p++)
        for (size_t a = 0; a < n; a++)
            for (size_t b = a + 1; b < n; b++) edges.push_back(graph[(p * n + a) * n + b]);
    std::nth_element(edges.begin(), edges.begin() + edges.size() / 2, edges.end());
    const double usual = edges[edges.size() / 2];
    dtfm_digits &dg = pr->digits;
    dg.usual = (int)std::max<ptrdiff_t>(std::upper_bound(first.begin(), first.end(), usual) - first.begin() - 1, 0);
    // D x D links of their own have a perfect matching about when no row and no column is left without one: at a share ln(2 D) / D
    // of the weights. Found 0.16 to 0.21 at 17 devices (regions, tied or not: 0.31 to 0.7), 0.08 to 0.11 at 48 (0.24 to 0.34).
    dg.own = (dg.usual + 0.5) / (dg.top[0] + 1) <= 1.4 * log(2.0 * pr->D_dp) / pr->D_dp;
    return DTFM_OK;
}

// W_rank and rank_val are there
int dtfm_match_prepare(dtfm_problem *pr)
{
    if (pr->D_dp <= 16) return DTFM_OK;
    const int ranks = pr->weights;
    const size_t entries = (size_t)pr->N * pr->N;
    const int w1 = (ranks + 126) / 127, w2 = (w1 + 126) / 127;   // ranks of a leading digit, of a pair of digits
    dtfm_digits &dg = pr->digits;
    dg.levels = w1 == 1 ? 1 : w2 == 1 ? 2 : 3;   // at most 2^20 ranks: a third digit tells all apart
    dg.top[0] = (ranks - 1) / w1;
    dg.top[1] = (w1 - 1) / w2;
    dg.top[2] = w2 - 1;
    void *mem = nullptr;
    DTFM_HIP(hipMalloc(&mem, 128 * sizeof(double) + dg.levels * entries));
    dg.first = static_cast<double *>(mem);
    dg.code = reinterpret_cast<uint8_t *>(dg.first + 128);
    hipLaunchKernelGGL(k_digits, dim3((unsigned)((entries + 255) / 256)), dim3(256), 0, (hipStream_t) nullptr, pr->W_rank, entries,
                       w1, w2, dg.levels, dg.code);
    DTFM_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_digit_first, dim3(1), dim3(128), 0, (hipStream_t) nullptr, pr->rank_val, ranks, w1, dg.first);
    DTFM_HIP(hipGetLastError());
    dg.usual = dg.top[0] / 4;
    return dtfm_match_usual(pr);
}

int dtfm_match_bits_enqueue(const dtfm_problem *pr, const int32_t *perm, size_t rows, int pairs, double *ghat, int inc_j, int inc_jp,
                            hipStream_t st)
{
    // 16,384 wavefronts, of which the chip holds 7,168 (28 a CU by their registers), each with as many candidates of one stage
    // pair as that takes
    const size_t share = ((size_t)2 * 256 * 32 + pairs - 1) / pairs, chunks = rows < share ? rows : share;
    const unsigned waves = (unsigned)(chunks * pairs), w = waves <= 2048u ? 1u : WAVES;
    auto kern = pr->D_dp <= 24 ? k_match_bits<24> : pr->D_dp <= 32 ? k_match_bits<32> : pr->D_dp <= 48 ? k_match_bits<48> : k_match_bits<64>;
    hipLaunchKernelGGL(kern, dim3((waves + w - 1) / w), dim3(64 * w), 0, st, pr->digits,
                       pr->W_rank, pr->rank_val, perm, pr->N, pr->D_dp, pr->D_pp, ghat, (int)rows, inc_j, inc_jp, pairs, (int)chunks);
    DTFM_HIP(hipGetLastError());
    return DTFM_OK;
}
