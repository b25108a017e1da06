// Eq. 4 for many stages by pruned subset recursion (the open-loop TSP over the coarsened graph, exact to the bit).
//
// Held-Karp fills tab[S][v] for all 2^n subsets (n = 16: 524,288 entries, 3.9 million relaxations a candidate). Nearly
// all of them belong to no path that comes near the optimum: with a lower bound on what the stages outside S still
// cost, some 50 to 200 entries per candidate are left (bounds and thresholds below; measured on coarsened graphs of
// region, cluster and independent networks at n = 14 and 16, where the dense recursion is the whole cost).
//   bound      node potentials pi turn an edge (i, j) into C_ij = g_ij + pi_i + pi_j. A path visits every inner stage
//              with degree 2, so the cheapest completion of a path over S that ends in v costs at least
//              MST_C(rest) + (cheapest edge into the rest is priced exactly, edge by edge) - 2 sum pi(rest) + the
//              smallest pi an end can have. Good potentials make this tight to some 1e-4 of the optimum; they come from
//              a few subgradient steps on the one-tree bound (Held & Karp 1970/71).
//   integers   g = floor(s min(Ghat, U)), U the cost of a path found by the nearest-neighbour rule and s = 2^24 / U;
//              potentials are integers too, so the bound itself is computed without rounding. A state is dropped iff
//              floor(s F) + bound > floor(s thr) + 1. The optimum T as the recursion defines it is a left-to-right
//              fp64 sum: s T >= (s F + rest)(1 - 17 * 2^-53), with s T <= 2^25 a difference far below the 1, so for
//              thr >= T no state on an optimal path is dropped, and its F is the value the full recursion gives it
//              (its best predecessor lies on an optimal path as well).
//   threshold  grows from just above the root bound until a path with T <= thr is found: every path of cost <= thr was
//              then kept, so T is the minimum. An attempt whose states die out proves T > thr; one that ends in
//              T' > thr gives the upper bound T' for the next.
// Sums along the path are fp64 in path order, exactly Held-Karp's; the result is the same number.
// Kernel times: 1024 allocations of 256 devices in 16 stages 0.16 ms (k_held_karp_blocked 2.2 ms), 4096 allocations of
// 1024 devices in 16 stages 0.32 ms (8.4 ms).
//
// One workgroup of four wavefronts takes four candidates (a launch of up to 1024: one, dtfm_tour_enqueue). The potentials of all
// four come from its first wavefront (16 lanes a candidate, a lane per stage: the chain of dependent minima bounds this
// part, and one wavefront's instructions serve four chains). Then every wavefront searches its own candidate: 16 lanes
// take a state, grow the spanning tree of its rest (one minimum over 16 lanes and one LDS row per edge), price the
// successors, one per lane, and put them into a hash table in LDS. A candidate with a layer of more than NARROW states is
// searched again by the whole workgroup on the joint tables, and so is the only candidate of a workgroup from the start.
// What does not fit there either, takes more than its share of the work (dtfm_tour_rule) or is not finite goes on a list
// for the dense recursion (k_held_karp_blocked).
//
// What the dense recursion gets at once: a launch takes it one round for every 256 candidates (one workgroup a CU) of 18,
// 32, 68, 130, 255 and 525 us at 11 to 16 stages, whatever the graph. A search takes 60 us where the graph has edges of
// many values, up to 200 us where it has a dozen, and ends in overfull tables on graphs of a few values (on graphs of
// region, cluster, independent and rounded networks of 1 to 64 devices a stage: 8 or more values at 16 stages: one
// candidate in thirty; 7: one in three; 4 and 5: three in four), where its time is lost. dtfm_tour_enqueue has the rule.
#include "dtfm_internal.h"

#include <math.h>

namespace {

constexpr int WAVES = 4;               // candidates (= wavefronts) per workgroup
// states per layer and wavefront; PER: candidates of the workgroup. With one of them four workgroups share a CU's LDS (tour_lds).
template <int PER>
constexpr int CAP = PER == 1 ? 224 : 256;
constexpr int SLOTS = 512;             // hash slots per wavefront
constexpr int LOG_SLOTS = 9;
constexpr int RSTR = 16;               // words between rows of the edge table
constexpr int NARROW = 40;             // layers wider than this go to the whole workgroup
constexpr int BATCH = 16 * 15;         // new states of one pass of a wavefront: 16 states, at most 15 successors each
// a pass is begun at no more than NARROW states (a wavefront alone) or WAVES * CAP (each wavefront of a workgroup)
static_assert(NARROW + BATCH < SLOTS && WAVES * (CAP<WAVES> + BATCH) < WAVES * SLOTS, "a search needs a free slot");
constexpr int STEPS = 18;              // subgradient steps
constexpr int LONE_STEPS = 16;         // the same where four step lengths go side by side
constexpr int REFINE_STEPS = 60;       // of a candidate whose layers outgrow the workgroup's tables
constexpr int UNIT_LOG = 24;           // the path U in integer units
constexpr int BIAS = 1 << 26;          // makes C_ij + BIAS positive: |pi| <= 2^24, 0 <= g <= 2^24
constexpr uint32_t EMPTY = 0xffffffffu;
constexpr size_t SPREAD = 256;         // up to so many candidates have a workgroup and a CU each, up to twice as many share it
constexpr double DOWN = 1.0 - 0x1p-50, UP = 1.0 + 0x1p-50;

// PER: candidates of the workgroup. With one of them 40 KiB: four workgroups a CU.
template <int PER>
struct tour_lds {
    double G[PER][16][16];
    double F[WAVES * CAP<PER>];
    unsigned long long hF[WAVES * SLOTS];
    alignas(16) uint32_t hkey[WAVES * SLOTS];         // ascend() writes its edge tables 16 bytes at a time: here and T
    uint32_t key[WAVES * CAP<PER>];         // set << 4 | last stage
    alignas(16) uint32_t T[PER][16][RSTR];            // (g_ij + pi_i) << 4
    int pi[PER][16];
    double scale[PER], U[PER], cap[PER], top[PER];
    double red[WAVES];
    double lo[PER], thr[PER], grow[PER];   // where a wavefront's own threshold loop stopped
    int L[PER], state[PER], values[PER];   // values: see edge_values
    int count;
    uint16_t slot[WAVES * CAP<PER>];
};
static_assert(sizeof(tour_lds<1>) <= 40960, "four workgroups a CU");
enum { SEARCH = 0, SETTLED = 1, DENSE = 2, WIDE = 3, SOLVED = 4 };
enum { FOUND, DIED, OVERFLOW_ };

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);   // folds into the consumer
}
// over the 16 lanes of a row, result in every lane (rotations by 8, 4, 2, 1)
__device__ __forceinline__ uint32_t row_min(uint32_t x)
{
    x = min(x, dpp<0x128>(x));
    x = min(x, dpp<0x124>(x));
    x = min(x, dpp<0x122>(x));
    return min(x, dpp<0x121>(x));
}
__device__ __forceinline__ int row_sum(int x)
{
    x += (int)dpp<0x128>((uint32_t)x);
    x += (int)dpp<0x124>((uint32_t)x);
    x += (int)dpp<0x122>((uint32_t)x);
    return x + (int)dpp<0x121>((uint32_t)x);
}
__device__ __forceinline__ double wave_min(double x)
{
    for (int o = 32; o >= 1; o >>= 1) x = fmin(x, __shfl_xor(x, o));
    return x;
}
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// potentials packed with their lane, order-preserving (|pi| <= 2^24)
__device__ __forceinline__ uint32_t pack_pi(int pi, int i) { return ((uint32_t)(pi + (1 << 25)) << 4) | (uint32_t)i; }
__device__ __forceinline__ int unpack_pi(uint32_t k) { return (int)(k >> 4) - (1 << 25); }

__device__ __forceinline__ int edge_units(double g, double U, double scale)
{
    return (int)(__dmul_rn(__dmul_rn(fmin(g, U), scale), DOWN));   // truncation: the values are >= 0
}

// Subgradient ascent on the one-tree bound from the potential `pi` of the lane's stage, by the 16 lanes of row `grp`
// (T: their table; cap: a bound above it settles the candidate). best, best_pi: the best bound and its potentials.
__device__ __forceinline__ void ascend(const int (&g)[16], uint32_t (*T)[RSTR], int grp, int i, int n, int steps, float lambda,
                                       float decay, bool fine, int cap, int pi, int &best, int &best_pi)
{
    const bool node = i < n;
    int before = 0;
    for (int it = 0; it < steps; it++) {
        {
            uint4 *row = reinterpret_cast<uint4 *>(&T[i][0]);
#pragma unroll
            for (int q = 0; q < 4; q++)
                row[q] = make_uint4((uint32_t)(g[4 * q] + pi) << 4, (uint32_t)(g[4 * q + 1] + pi) << 4,
                                    (uint32_t)(g[4 * q + 2] + pi) << 4, (uint32_t)(g[4 * q + 3] + pi) << 4);
        }
        wave_sync();
        // Prim from stage 0
        const uint32_t own = ((uint32_t)(pi + BIAS) << 4) | (uint32_t)i;
        uint32_t dead = node ? 0u : ~0u, k = ~0u, sum = 0u;
        int b = 0, par = 0;
        for (int t = 1; t < n; t++) {
            dead = i == b ? ~0u : dead;
            const uint32_t c = (T[b][i] + own) | dead;
            par = c < k ? b : par;
            k = min(k, c) | dead;
            const uint32_t m = row_min(k);
            b = (int)(m & 15u);
            sum += m >> 4;
        }
        // degrees: the children of lane i are the lanes whose parent is i
        uint64_t kids = __ballot(node && i != 0);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const uint64_t bit = __ballot((par >> q) & 1);
            kids &= ((i >> q) & 1) ? bit : ~bit;
        }
        int deg = __popc((uint32_t)(kids >> (16 * grp)) & 0xffffu) + (i != 0 ? 1 : 0);
        // the two ends hang on the smallest potentials
        const uint32_t mine = node ? pack_pi(pi, i) : ~0u;
        const uint32_t e1 = row_min(mine), e2 = row_min(mine == e1 ? ~0u : mine);
        deg += mine == e1 || mine == e2 ? 1 : 0;
        const int L = (int)(sum - (uint32_t)(n - 1) * (uint32_t)BIAS) + unpack_pi(e1) + unpack_pi(e2) - 2 * row_sum(node ? pi : 0);
        if (L > best) {
            best = L;
            best_pi = pi;
        }
        const int d = node ? deg - 2 : 0, dd = row_sum(d * d);
        if (__ballot(dd != 0 && best <= cap && fine) == 0ull) break;   // all four: a path, settled or not for this kernel
        const float step = dd != 0 ? lambda * (float)((1 << UNIT_LOG) - L) / (float)dd : 0.0f;
        lambda *= decay;
        pi += (int)rintf(fminf(fmaxf(step * (0.7f * (float)d + 0.3f * (float)before), -16777216.0f), 16777216.0f));
        pi = min(max(pi, -(1 << 24)), 1 << 24);
        before = d;
        wave_sync();
    }
}

__device__ __forceinline__ double lane_value(double x, int lane)   // lane: the same in all lanes
{
    const long long b = __double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)b, lane), hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// The number of different values among the edges of a graph (g(i, j): the edge), by one wavefront; beyond `limit` an
// estimate, from the share of the edges that limit + 1 values take. The lanes hold the edges from stage i to stage i + k,
// k up to n / 2; a turn counts one value and strikes out the edges that have it.
template <typename Edge>
__device__ __forceinline__ int edge_values(int lane, int n, int limit, Edge g)
{
    double own[2];
    uint64_t left[2];
#pragma unroll
    for (int q = 0; q < 2; q++) {
        const int i = lane & 15, k = 4 * q + (lane >> 4) + 1, j = i + k < n ? i + k : i + k - n;
        const bool edge = i < n && (2 * k < n || (2 * k == n && i < k));
        own[q] = edge ? g(i, j) : 0.0;
        left[q] = __ballot(edge);
    }
    int values = 0;
    for (; values <= limit && (left[0] | left[1]) != 0ull; values++) {
        const int q = left[0] != 0ull ? 0 : 1;
        const double v = lane_value(q == 0 ? own[0] : own[1], __ffsll((unsigned long long)left[q]) - 1);
        left[q] &= left[q] - 1ull;   // a NaN is not equal to itself
        left[0] &= ~__ballot(own[0] == v);
        left[1] &= ~__ballot(own[1] == v);
    }
    const int edges = n * (n - 1) / 2, rest = __popcll(left[0]) + __popcll(left[1]);
    return rest > 0 ? max(limit + 1, values * edges / (edges - rest)) : values;
}

// Upper bound, scale, potentials and root bound of candidate `grp` of the workgroup, by the 16 lanes of a row. The only candidate
// of a workgroup has all four rows: each goes its own way up, and the best is kept.
template <int PER>
__device__ __forceinline__ void tour_potentials(tour_lds<PER> &sm, int grp, int i, int n)
{
    const int cd = PER == 1 ? 0 : grp;
    const double (*G)[16] = sm.G[cd];
    const bool node = i < n;
    bool fine = true, equal = true;
    const double g01 = G[0][1];
    for (int j = 0; j < n; j++)
        if (node && j != i) {
            fine = fine && G[i][j] >= 0.0 && G[i][j] < INFINITY;
            equal = equal && G[i][j] == g01;
        }
    // nearest-neighbour path from every stage
    const uint32_t full = (1u << n) - 1u;
    double U = INFINITY;
    {
        uint32_t rest = full & ~(1u << (node ? i : 0));
        int u = node ? i : 0;
        double F = 0.0;
        for (int k = 1; k < n; k++) {
            int b = __ffs((int)rest) - 1;
            double best = G[u][b];
#pragma unroll
            for (int w = 1; w < 16; w++) {
                const double g = G[u][w];
                if (((rest >> w) & 1u) && g < best) {
                    best = g;
                    b = w;
                }
            }
            F = __dadd_rn(F, best);
            rest &= ~(1u << b);
            u = b;
        }
        if (node) U = F;
    }
    for (int o = 8; o >= 1; o >>= 1) U = fmin(U, __shfl_xor(U, o, 16));
    fine = fine && U > 1e-200 && U < 1e200;
    fine = ((__ballot(node && !fine) >> (16 * grp)) & 0xffffull) == 0ull;
    equal = fine && ((__ballot(node && !equal) >> (16 * grp)) & 0xffffull) == 0ull;   // every path has the same sum
    const double scale = fine ? __ddiv_rn((double)(1 << UNIT_LOG), U) : 0.0;
    int g[16];
#pragma unroll
    for (int j = 0; j < 16; j++) g[j] = fine && node && j < n ? edge_units(G[i][j], U, scale) : 0;
    // a bound above this settles a trial (see k_tour_search): in units, rounded so that the real bound is above cap
    const double cap_units = __dmul_rn(__dmul_rn(sm.cap[cd], scale), UP);
    const int cap = cap_units < 0x1p30 ? (cap_units > 0.0 ? (int)cap_units + 1 : 1) : INT32_MAX;
    int best = INT32_MIN, best_pi = 0;
    const bool go = fine && !equal && sm.state[cd] == SEARCH;
    if constexpr (PER == 1) {   // the hash tables are free for the edge tables
        uint32_t (*T)[RSTR] = reinterpret_cast<uint32_t (*)[RSTR]>(sm.hkey + grp * 16 * RSTR);
        const float lambda = grp == 0 ? 2.0f : grp == 1 ? 1.0f : grp == 2 ? 3.0f : 1.5f;
        const float decay = grp == 0 ? 0.80f : grp == 1 ? 0.87f : grp == 2 ? 0.73f : 0.79f;
        ascend(g, T, grp, i, n, LONE_STEPS, lambda, decay, go, cap, 0, best, best_pi);
        int top = max(best, __shfl_xor(best, 16));
        top = max(top, __shfl_xor(top, 32));
        const uint64_t who = __ballot(best == top);   // one row at least, whole
        if (grp != (__ffsll((unsigned long long)who) - 1) >> 4) return;
    } else {
        ascend(g, sm.T[cd], grp, i, n, STEPS, 2.0f, 0.82f, go, cap, 0, best, best_pi);
    }
    sm.pi[cd][i] = best_pi;
    if (i == 0) {
        sm.scale[cd] = scale;
        sm.U[cd] = U;
        sm.L[cd] = best;
        if (sm.state[cd] == SEARCH) sm.state[cd] = !fine ? DENSE : equal ? SOLVED : best > cap ? SETTLED : SEARCH;
    }
}

// Potentials of candidate `cd` again, from where they are, with more steps and four step lengths side by side, by the
// first wavefront (the hash tables are free for its edge tables).
template <int PER>
__device__ __forceinline__ void tour_refine(tour_lds<PER> &sm, int cd, int lane, int n)
{
    const int grp = lane >> 4, i = lane & 15;
    int g[16];
#pragma unroll
    for (int j = 0; j < 16; j++) g[j] = i < n && j < n ? edge_units(sm.G[cd][i][j], sm.U[cd], sm.scale[cd]) : 0;
    uint32_t (*T)[RSTR] = reinterpret_cast<uint32_t (*)[RSTR]>(sm.hkey + grp * 16 * RSTR);
    const float lambda = grp == 0 ? 2.0f : grp == 1 ? 1.2f : grp == 2 ? 0.7f : 0.4f;
    int best = sm.L[cd], best_pi = sm.pi[cd][i];
    ascend(g, T, grp, i, n, REFINE_STEPS, lambda, 0.93f, true, INT32_MAX, best_pi, best, best_pi);
    int top = best;
    top = max(top, __shfl_xor(top, 16));
    top = max(top, __shfl_xor(top, 32));
    const uint64_t who = __ballot(best == top);   // one row at least, whole
    if (grp == (__ffsll((unsigned long long)who) - 1) >> 4) {
        sm.pi[cd][i] = best_pi;
        if (i == 0) sm.L[cd] = best;
    }
}

// Cost of the best of 64 greedy paths of candidate `cd`: from every stage, by the nearest-neighbour rule on the edges
// with the potentials of their far ends at four weights added. The potentials make inner stages attractive that a plain
// nearest neighbour strands: nine candidates in ten get the optimum, so that one search at this threshold ends it.
template <int PER>
__device__ __forceinline__ double greedy_path(const tour_lds<PER> &sm, int cd, int lane, int n)
{
    const double (*G)[16] = sm.G[cd];
    const int start = (lane & 15) < n ? (lane & 15) : 0, r = lane >> 4;
    const int weight = r == 0 ? 16 : r == 1 ? 14 : r == 2 ? 12 : 8;   // sixteenths
    int far[16];
#pragma unroll
    for (int w = 0; w < 16; w++) far[w] = (sm.pi[cd][w] >> 4) * weight;
    uint32_t rest = ((1u << n) - 1u) & ~(1u << start);
    int u = start;
    double F = 0.0;
    for (int k = 1; k < n; k++) {
        int b = 0, best = INT32_MAX;
#pragma unroll
        for (int w = 0; w < 16; w++) {
            const int c = ((int)sm.T[cd][u][w] >> 4) + far[w];
            const bool take = ((rest >> w) & 1u) && c < best;
            best = take ? c : best;
            b = take ? w : b;
        }
        F = __dadd_rn(F, G[u][b]);
        rest &= ~(1u << b);
        u = b;
    }
    return wave_min(F);
}

// The edge table of candidate `cd` from its potentials, and the cost of the best path known, by one wavefront.
template <int PER>
__device__ __forceinline__ void tour_table(tour_lds<PER> &sm, int cd, int lane, int n)
{
    const double U = sm.U[cd], scale = sm.scale[cd];
    wave_sync();
    for (int e = lane; e < 256; e += 64) {
        const int a = e >> 4, b = e & 15;
        sm.T[cd][a][b] = (uint32_t)(edge_units(sm.G[cd][a][b], U, scale) + sm.pi[cd][a]) << 4;
    }
    wave_sync();
    const double path = greedy_path(sm, cd, lane, n);
    if (lane == 0) sm.top[cd] = fmin(path, sm.top[cd]);
    wave_sync();
}

// The successors of the states base .. base + 4 TEAM NJ - 1 of a layer of k stages, into the hash table. A row of 16
// lanes takes NJ states: their spanning trees are grown side by side (one tree alone leaves the wavefront waiting for
// its chain of LDS reads and minima).
template <int TEAM, int NJ, int PER>
__device__ __forceinline__ void expand(tour_lds<PER> &sm, int k, int n, int base, int cnt, int tid, uint32_t full, int pi,
                                       uint32_t own, double scale, double thr, int thr_units, const uint32_t *key,
                                       const double *F, unsigned long long *hF, uint32_t *hkey, uint16_t *slot,
                                       const double (*G)[16], const uint32_t (*E)[RSTR], int &made)
{
    constexpr int cap = TEAM * CAP<PER>, slots = TEAM * SLOTS;
    constexpr int shift = 32 - LOG_SLOTS - (TEAM == 4 ? 2 : 0);
    const int i = tid & 15, lane = tid & 63;
    uint32_t S[NJ], dead[NJ], m[NJ], sum[NJ];
    int u[NJ], b[NJ];
#pragma unroll
    for (int j = 0; j < NJ; j++) {
        const int e = base + (tid >> 4) + j * TEAM * 4;
        const uint32_t ky = e < cnt ? key[e] : full << 4;   // no state: nothing is left to visit
        S[j] = ky >> 4;
        u[j] = (int)(ky & 15u);
        const uint32_t rest = full & ~S[j];
        dead[j] = ((rest >> i) & 1u) ? 0u : ~0u;
        m[j] = ~0u;
        sum[j] = 0u;
        b[j] = rest != 0u ? __ffs((int)rest) - 1 : 0;
    }
    // spanning trees of the stages left (Prim)
    for (int t = n - k - 1; t > 0; t--) {
#pragma unroll
        for (int j = 0; j < NJ; j++) {
            const uint32_t c = E[b[j]][i] + own;
            dead[j] = i == b[j] ? ~0u : dead[j];
            m[j] = min(m[j], c) | dead[j];
        }
        uint32_t w[NJ];
#pragma unroll
        for (int j = 0; j < NJ; j++) w[j] = min(m[j], dpp<0x128>(m[j]));
#pragma unroll
        for (int j = 0; j < NJ; j++) w[j] = min(w[j], dpp<0x124>(w[j]));
#pragma unroll
        for (int j = 0; j < NJ; j++) w[j] = min(w[j], dpp<0x122>(w[j]));
#pragma unroll
        for (int j = 0; j < NJ; j++) w[j] = min(w[j], dpp<0x121>(w[j]));
#pragma unroll
        for (int j = 0; j < NJ; j++) {
            b[j] = (int)(w[j] & 15u);
            sum[j] += w[j] >> 4;
        }
    }
#pragma unroll
    for (int j = 0; j < NJ; j++) {
        if (NJ > 1 && base + j * TEAM * 4 >= cnt) break;
        const int e = base + (tid >> 4) + j * TEAM * 4;
        const bool in = ((full & ~S[j]) >> i) & 1u;
        const int tree = (int)(sum[j] - (uint32_t)(n - k - 1) * (uint32_t)BIAS);
        const uint32_t mine = in ? pack_pi(pi, i) : ~0u;
        const uint32_t e1 = row_min(mine), e2 = row_min(mine == e1 ? ~0u : mine);
        const int end = unpack_pi(mine == e1 ? e2 : e1), all = row_sum(in ? pi : 0);
        const double F2 = __dadd_rn(in ? F[e] : 0.0, G[u[j]][i]);
        bool keep = in && F2 <= thr;
        if (keep) {
            const int f = (int)__dmul_rn(__dmul_rn(F2, scale), DOWN);
            keep = (k == n - 1 ? f : f + tree + pi - 2 * all + end) <= thr_units;
        }
        bool fresh = false;
        const uint32_t want = ((S[j] | (1u << i)) << 4) | (uint32_t)i;
        uint32_t h = (want * 2654435761u) >> shift;
        if (keep) {
            // the table never fills (see BATCH)
            for (int probe = 0; probe < slots; probe++) {
                const uint32_t old = atomicCAS(&hkey[h], EMPTY, want);
                fresh = old == EMPTY;
                if (fresh || old == want) break;
                h = (h + 1u) & (uint32_t)(slots - 1);
            }
            atomicMin(&hF[h], (unsigned long long)__double_as_longlong(F2));
        }
        const uint64_t news = __ballot(fresh);
        const int nnew = __popcll(news);
        int first = made;
        if (TEAM > 1) {
            if (nnew > 0 && lane == 0) first = atomicAdd(&sm.count, nnew);
            first = __builtin_amdgcn_readfirstlane(first);
            if (nnew > 0) made = first + nnew;
        } else {
            made += nnew;
        }
        const int pos = first + __popcll(news & ((1ull << lane) - 1ull));
        if (fresh && pos < cap) slot[pos] = (uint16_t)h;
    }
}

// The states of a search, layer by layer, for the back-tracking: n layers of up to WAVES * CAP<PER>.
struct tour_record {
    double *F;
    uint32_t *key;
    int *count;
};

// All paths of candidate `cd` with cost <= thr, layer by layer. TEAM wavefronts work together (`tid`: thread of the
// team) on the tables of wavefront `cd` (TEAM = 1) or of the whole workgroup. FOUND: T = the smallest cost of a
// complete path kept, which is the optimum if T <= thr. work: the states that may still be priced. Graphs of at most n / 2
// values have layers of up to 560 states where the search succeeds (two cliques of eight stages) and outgrow any table
// where it does not, so they are given up at 40 n; the stage orders, whose full table is dearer, are not.
template <int TEAM, bool RECORD, int PER>
__device__ __forceinline__ int tour_search(tour_lds<PER> &sm, int cd, int tid, int n, double thr, double &T, int &work,
                                           const tour_record &rec)
{
    constexpr int slots = TEAM * SLOTS, NG = TEAM * 4;
    const int limit = TEAM == 1 ? NARROW : !RECORD && sm.values[cd] <= n / 2 ? 40 * n : TEAM * CAP<PER>;
    const int at = TEAM == 1 ? cd : 0;
    double *F = sm.F + at * CAP<PER>;
    unsigned long long *hF = sm.hF + at * SLOTS;
    uint32_t *hkey = sm.hkey + at * SLOTS, *key = sm.key + at * CAP<PER>;
    uint16_t *slot = sm.slot + at * CAP<PER>;
    const double (*G)[16] = sm.G[cd];
    const uint32_t (*E)[RSTR] = sm.T[cd];
    auto sync = [&]() {
        if (TEAM == 1) wave_sync();
        else __syncthreads();
    };
    const int i = tid & 15, lane = tid & 63;
    (void)lane;
    const uint32_t full = (1u << n) - 1u;
    const int pi = sm.pi[cd][i];
    const uint32_t own = ((uint32_t)(pi + BIAS) << 4) | (uint32_t)i;
    const double scale = sm.scale[cd];
    const int thr_units = (int)__dmul_rn(__dmul_rn(thr, scale), UP) + 1;   // thr <= U: at most 2^24 + 2
    for (int e = tid; e < slots; e += TEAM * 64) {
        hkey[e] = EMPTY;
        hF[e] = ~0ull;
    }
    if (tid < n) {
        key[tid] = (16u << tid) | (uint32_t)tid;
        F[tid] = 0.0;
    }
    if (TEAM > 1 && tid == 0) sm.count = 0;
    int cnt = n;
    sync();
    for (int k = 1; k < n; k++) {
        int made = 0;
        if (cnt <= NG) {
            expand<TEAM, 1>(sm, k, n, 0, cnt, tid, full, pi, own, scale, thr, thr_units, key, F, hF, hkey, slot, G, E, made);
        } else {
            for (int base = 0; base < cnt && made <= limit; base += 4 * NG)
                expand<TEAM, 4>(sm, k, n, base, cnt, tid, full, pi, own, scale, thr, thr_units, key, F, hF, hkey, slot, G, E, made);
        }
        sync();
        if (TEAM > 1) {
            made = sm.count;
            __syncthreads();
            if (tid == 0) sm.count = 0;
        }
        work -= cnt;
        if (made > limit || work < 0) return OVERFLOW_;
        if (made == 0) return DIED;
        for (int e = tid; e < made; e += TEAM * 64) {
            const int h = slot[e];
            key[e] = hkey[h];
            F[e] = __longlong_as_double((long long)hF[h]);
            if (RECORD) {
                rec.key[k * (WAVES * CAP<PER>) + e] = hkey[h];
                rec.F[k * (WAVES * CAP<PER>) + e] = __longlong_as_double((long long)hF[h]);
            }
            hkey[h] = EMPTY;
            hF[h] = ~0ull;
        }
        cnt = made;
        if (RECORD && tid == 0) rec.count[k] = made;
        sync();
    }
    double best = INFINITY;
    for (int e = tid; e < cnt; e += TEAM * 64) best = fmin(best, F[e]);
    best = wave_min(best);
    if (TEAM > 1) {
        if (lane == 0) sm.red[tid >> 6] = best;
        __syncthreads();
        for (int w = 0; w < TEAM; w++) best = fmin(best, sm.red[w]);
        __syncthreads();
    }
    T = best;
    return FOUND;
}

// Where the threshold loop of candidate `cd` starts when the workgroup runs all of it.
template <int PER>
__device__ __forceinline__ void first_threshold(tour_lds<PER> &sm, int cd)
{
    const double root = fmax((double)sm.L[cd], 0.0) / sm.scale[cd];
    sm.lo[cd] = root;
    sm.grow[cd] = 1.5e-3 * sm.top[cd];
    sm.thr[cd] = fmin(root + sm.grow[cd], fmin(sm.top[cd], sm.cap[cd]));
}

// The threshold loop. Returns SETTLED (the optimum is above cap), SEARCH with T the optimum, WIDE (a
// wavefront's layer outgrew NARROW: the workgroup goes on from the same threshold) or DENSE.
template <int TEAM, bool RECORD, int PER>
__device__ __forceinline__ int tour_solve(tour_lds<PER> &sm, int cd, int tid, int n, int &work, double &T, const tour_record &rec)
{
    const double cap = sm.cap[cd];
    double U = sm.top[cd], top = fmin(U, cap), root = fmax((double)sm.L[cd], 0.0) / sm.scale[cd];
    bool refined = false;
    double lo = root, over = INFINITY, grow = 1.5e-3 * U, thr = fmin(root + grow, top);
    if (TEAM > 1) {
        lo = sm.lo[cd];
        thr = sm.thr[cd];
        grow = sm.grow[cd];
    }
    for (int attempt = 0; attempt < 16; attempt++) {
        const int r = tour_search<TEAM, RECORD>(sm, cd, tid, n, thr, T, work, rec);
        if (r == FOUND) {
            if (T <= thr) return SEARCH;
            if (T >= over) return DENSE;
            thr = fmin(T, U);
            continue;
        }
        if (r == DIED) {
            if (thr >= cap) return SETTLED;
            if (thr >= U) return DENSE;   // cannot happen: U is the cost of a path
            lo = thr;
            grow *= 2.5;
            thr = fmin(root + grow, top);
            if (thr >= over) thr = 0.5 * (lo + over);
        } else if (TEAM == 1) {
            if ((tid & 63) == 0) {
                sm.lo[cd] = lo;
                sm.thr[cd] = thr;
                sm.grow[cd] = grow;
            }
            return WIDE;
        } else {
            if (!refined) {
                // Tables too small at this threshold: better potentials, unless the graph has few values, the bound no gap
                // left to close or the dense recursion takes less (up to 15 stages, where no order is asked for).
                if (work < 0 || (!RECORD && n < 16) || sm.values[cd] <= (RECORD ? n / 2 : 2 * n) ||
                    thr - root < 0x1p-18 * U)
                    return DENSE;
                refined = true;
                __syncthreads();
                if (tid < 64) {
                    tour_refine(sm, cd, tid, n);
                    tour_table(sm, cd, tid, n);
                }
                __syncthreads();
                U = sm.top[cd];
                root = fmax((double)sm.L[cd], 0.0) / sm.scale[cd];
                lo = fmax(lo, root);
                top = fmin(U, cap);
                grow = 1.5e-3 * U;
                thr = fmin(fmax(root + grow, lo), top);
                continue;
            }
            if (work < 0) return DENSE;
            over = thr;
            if (over - lo <= 1e-4 * U) return DENSE;
            thr = lo + 0.3 * (over - lo);
        }
    }
    return DENSE;
}

// rows: with `list`, list[0 .. count[0]), else all P. cur: costs of the current rows a trial is judged by (or null): a
// trial that is proven not to be strictly cheaper gets +inf, as in k_trial_shortcut. The rows left to the dense
// recursion go to dense[0 .. count[1]).
template <int PER>
__global__ void __launch_bounds__(64 * WAVES)
k_tour_search(const double *__restrict__ ghat, const double *__restrict__ datap, int n, double *__restrict__ cost, size_t P,
              const int32_t *__restrict__ list, int32_t *__restrict__ count, const double *__restrict__ cur,
              int trials_per_row, double *__restrict__ pp_out, int32_t *__restrict__ dense, dtfm_tour_rule rule)
{
    __shared__ tour_lds<PER> sm;
    const size_t todo = list != nullptr ? (size_t)count[0] : P;
    const int per = PER == 1 || todo <= SPREAD ? 1 : todo <= 2 * SPREAD ? 2 : WAVES;   // candidates of the workgroup
    // its candidates lie apart in the launch: neighbours are often trials of one row, and hard together
    const size_t groups = (todo + per - 1) / per;
    if (blockIdx.x >= groups) return;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const size_t idx = (size_t)blockIdx.x + (size_t)wave * groups;
    if (rule.split && (size_t)count[2] == todo) return;
    const bool have = wave < per && idx < todo;
    const size_t p = have ? (list != nullptr ? (size_t)list[idx] : idx) : 0;
    const bool few = [&]() {
        if (wave >= PER) return false;
        for (int e = lane; e < 256; e += 64) {
            const int a = e >> 4, b = e & 15;
            sm.G[wave][a][b] = have && a < n && b < n ? ghat[p * n * n + a * n + b] : 0.0;
        }
        if (lane == 0) {
            double cap = INFINITY;
            if (have && cur != nullptr) {
                // smallest PipelineP a rejected trial can have: fl(datap + cap) >= cur
                const double c = cur[p / (size_t)trials_per_row];
                cap = __dadd_rn(__dadd_rn(c, -datap[p]), __dmul_rn(c, 0x1p-51));
            }
            sm.cap[wave] = cap;
            sm.state[wave] = !have || cap <= 0.0 ? SETTLED : SEARCH;
        }
        wave_sync();
        const int values = edge_values(lane, n, max(rule.few, n / 2), [&](int i, int j) { return sm.G[wave][i][j]; });
        const bool f = values > 1 && values <= rule.few;
        if (lane == 0) {
            sm.values[wave] = values;
            if (sm.state[wave] == SEARCH && (f || !rule.worth(n, todo, (size_t)count[2]))) sm.state[wave] = DENSE;
        }
        return f;
    }();
    __syncthreads();
    bool any = false;
    for (int w = 0; w < PER; w++) any = any || sm.state[w] == SEARCH;
    if (any && wave == 0) tour_potentials(sm, lane >> 4, lane & 15, n);
    __syncthreads();
    double T = 0.0;
    int state = wave < PER ? sm.state[wave] : SETTLED;
    if (state == SEARCH) {
        if (lane == 0) sm.top[wave] = sm.U[wave];
        tour_table(sm, wave, lane, n);
        if (per == 1) {
            if (lane == 0) first_threshold(sm, 0);
            state = WIDE;
        } else if constexpr (PER > 1) {
            int work = INT32_MAX;
            state = tour_solve<1, false>(sm, wave, lane, n, work, T, tour_record());
            if (state == WIDE && n < 12) state = DENSE;   // 18 us there, 20 at the least here
        }
        if (lane == 0 && state == WIDE) sm.state[wave] = WIDE;
    }
    __syncthreads();
    int work = rule.work;
    for (int w = 0; w < PER; w++) {   // too wide for a quarter of the tables: all of them, one candidate at a time
        if (sm.state[w] != WIDE) continue;
        double Tw = 0.0;
        // Graphs of more than 2 n values or so end well: one in some hundred takes long, none of those seen were left to the dense
        // recursion, which would add its 525 us to a launch (1024 allocations of 1024 devices in regions: 1.46 and 1.97 ms).
        const bool bounded = sm.values[w] <= 2 * n;
        int budget = bounded ? work : INT32_MAX;
        const int s = budget < 0 ? DENSE : tour_solve<WAVES, false>(sm, w, tid, n, budget, Tw, tour_record());
        if (bounded) work = budget;
        if (w == wave) {
            state = s;
            T = Tw;
        }
        __syncthreads();
    }
    if (lane != 0 || !have) return;
    if (state == SOLVED) T = sm.U[wave];
    if (state == SEARCH || state == SOLVED) {
        cost[p] = __dadd_rn(datap[p], T);
        pp_out[p] = T;
    } else if (state == SETTLED) {
        cost[p] = INFINITY;
    } else if (!(rule.split && few)) {   // those are there already
        dense[atomicAdd(&count[1], 1)] = (int32_t)p;
    }
}

// Appends the rows whose graphs have 2 to rule.few values to dense and counts them in count[2], before the search: it
// takes no row if the dense recursion needs as many rounds without them. One wavefront per row.
__global__ void __launch_bounds__(64 * WAVES)
k_tour_split(const double *__restrict__ ghat, int n, size_t P, const int32_t *__restrict__ list, int32_t *__restrict__ count,
             int32_t *__restrict__ dense, dtfm_tour_rule rule)
{
    const int lane = threadIdx.x & 63;
    const size_t idx = (size_t)blockIdx.x * WAVES + (threadIdx.x >> 6), todo = list != nullptr ? (size_t)count[0] : P;
    if (idx >= todo) return;
    const size_t p = list != nullptr ? (size_t)list[idx] : idx;
    const int values = edge_values(lane, n, rule.few, [&](int i, int j) { return ghat[p * n * n + i * n + j]; });
    if (lane == 0 && values > 1 && values <= rule.few) {
        atomicAdd(&count[2], 1);
        dense[atomicAdd(&count[1], 1)] = (int32_t)p;
    }
}

// The stage order behind Eq. 4: the path ends in the lowest-numbered stage that attains the minimum, and the stage before
// v in a path over S is the lowest-numbered u with fl(tab[S - v][u] + Ghat[u][v]) = tab[S][v]. A search whose threshold is
// not below the optimum keeps every state of every optimal path with its exact value, so both choices can be read off its
// layers: a state of another path that met the equation would itself start an optimal path. One workgroup per candidate
// (a call has few of them: 32 orders of 16 stages take 3.0 ms by the full table in HBM, 0.09 to 0.14 ms this way); the rows
// left to the full table go to dense[0 .. count[1]).
__global__ void __launch_bounds__(64 * WAVES)
k_tour_path(const double *__restrict__ ghat, int n, size_t P, double *__restrict__ tab, int32_t *__restrict__ order,
            int32_t *__restrict__ count, int32_t *__restrict__ dense)
{
    __shared__ tour_lds<1> sm;
    const int tid = threadIdx.x, lane = tid & 63;
    double *slot = tab + (size_t)blockIdx.x * ((size_t)n << n);   // n * 2^n doubles hold the layers from n = 11 on
    const tour_record rec = {slot, reinterpret_cast<uint32_t *>(slot + n * WAVES * CAP<1>),
                             reinterpret_cast<int *>(slot + n * WAVES * CAP<1> + n * WAVES * CAP<1> / 2)};
    for (size_t p = blockIdx.x; p < P; p += gridDim.x) {
        __syncthreads();
        {
            const int a = tid >> 4, b = tid & 15;
            sm.G[0][a][b] = a < n && b < n ? ghat[p * n * n + a * n + b] : 0.0;
        }
        if (tid == 0) {
            sm.cap[0] = INFINITY;
            sm.state[0] = SEARCH;
        }
        __syncthreads();
        if (tid < 64) {
            sm.values[0] = edge_values(lane, n, n / 2, [&](int i, int j) { return sm.G[0][i][j]; });
            // the table of 12 stages takes 60 us, a search of such a graph up to 200
            if (n == 12 && sm.values[0] > 1 && sm.values[0] <= n / 2) sm.state[0] = DENSE;
            wave_sync();
            tour_potentials(sm, lane >> 4, lane & 15, n);
            wave_sync();
            if (sm.state[0] == SEARCH) {
                if (lane == 0) sm.top[0] = sm.U[0];
                tour_table(sm, 0, lane, n);
                if (lane == 0) first_threshold(sm, 0);
            }
        }
        if (tid < n) {
            rec.F[tid] = 0.0;
            rec.key[tid] = (16u << tid) | (uint32_t)tid;
            if (tid == 0) rec.count[0] = n;
        }
        __syncthreads();
        int state = sm.state[0];
        double T = 0.0;
        int work = min(max((n << n) >> 5, 1 << 12), 1 << 14);   // at most 0.7 ms
        if (state == SEARCH) state = tour_solve<WAVES, true>(sm, 0, tid, n, work, T, rec);
        __syncthreads();
        int32_t *ord = order + p * n;
        if (state == SOLVED) {   // equal edges: every state of a layer has the same value
            if (tid < n) ord[tid] = n - 1 - tid;
        } else if (state != SEARCH) {
            if (tid == 0) dense[atomicAdd(&count[1], 1)] = (int32_t)p;
        } else if (tid < 64) {
            uint32_t S = (1u << n) - 1u;   // stages of the path up to position k; its last one is sought
            int v = -1;
            double F = T;
            for (int k = n - 1; k >= 0; k--) {
                uint32_t best = ~0u;
                double val = 0.0;
                const int m = rec.count[k];
                for (int e = lane; e < m; e += 64) {
                    const uint32_t ky = rec.key[k * (WAVES * CAP<1>) + e];
                    const double f = rec.F[k * (WAVES * CAP<1>) + e];
                    const uint32_t u = ky & 15u;
                    if (ky >> 4 == S && u < best && (v < 0 ? f : __dadd_rn(f, sm.G[0][u][v])) == F) {
                        best = u;
                        val = f;
                    }
                }
                uint32_t low = best;
                for (int o = 32; o >= 1; o >>= 1) low = min(low, (uint32_t)__shfl_xor((int)low, o));
                const uint64_t who = __ballot(best == low);
                F = __shfl(val, __ffsll((unsigned long long)who) - 1);
                v = low < 16u ? (int)low : __ffs((int)S) - 1;   // found for every finite graph
                S &= ~(1u << v);
                if (lane == 0) ord[k] = v;
            }
        }
    }
}

}  // namespace

int dtfm_tour_path_enqueue(const dtfm_problem *pr, const dtfm_eval_bufs &b, double *tab, size_t slots, size_t rows,
                           int32_t *order, hipStream_t st)
{
    hipLaunchKernelGGL(k_tour_path, dim3((unsigned)slots), dim3(64 * WAVES), 0, st, b.ghat, pr->D_pp, rows, tab, order, b.count,
                       b.dense);
    DTFM_HIP(hipGetLastError());
    return DTFM_OK;
}

int dtfm_tour_enqueue(const dtfm_problem *pr, const dtfm_eval_bufs &b, size_t rows, double *cost, const int32_t *list,
                      const dtfm_trial_ref *ref, hipStream_t st)
{
    // for any number of rows up to `rows` (with a list it is known on the device only)
    const size_t packed = (rows + WAVES - 1) / WAVES, grid = rows < SPREAD ? rows : packed < SPREAD ? SPREAD : packed;
    const dtfm_tour_rule rule(pr, rows, b.hk_grid);
    const int n = pr->D_pp;
    if (rule.split) {
        hipLaunchKernelGGL(k_tour_split, dim3((unsigned)packed), dim3(64 * WAVES), 0, st, b.ghat, n, rows, list, b.count,
                           b.dense, rule);
        DTFM_HIP(hipGetLastError());
    }
    // Up to four workgroups a CU: each candidate has one of its own from the start, so that a hard one has four wavefronts and
    // waits for no other. Evaluations in regions, four candidates to a workgroup (one), 512 / 768 / 1024 rows: 16 stages of 16 287 /
    // 350 / 382 (238 / 286 / 304) us, 2 249 / 271 / 274 (206 / 211 / 217), 14 of 2 141 / 169 / 173 (115 / 125 / 131); the graphs of single
    // devices have no hard ones, 14 stages 74 / 77 / 80 (73 / 84 / 91).
    const bool lone = rows <= (pr->D_dp == 1 ? 512u : 1024u);
    hipLaunchKernelGGL(lone ? k_tour_search<1> : k_tour_search<WAVES>, dim3((unsigned)(lone ? rows : grid)),
                       dim3(64 * WAVES), 0, st, b.ghat, b.datap,
                       n, cost, rows, list, b.count, ref != nullptr ? ref->cur : (const double *)nullptr,
                       ref != nullptr ? ref->trials_per_row : 1, b.pp, b.dense, rule);
    DTFM_HIP(hipGetLastError());
    return DTFM_OK;
}
