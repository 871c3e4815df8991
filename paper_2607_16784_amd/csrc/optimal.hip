// optimal.hip -- the optimal placement of the placement-accuracy experiment
// (Sec. 6.4): the smallest mean drop (1/n) sum_p mu_p over every placement of
// n models onto G identical GPUs holding at most C models each, mu_p from
// Alg. 1's aggregation over the models sharing p's GPU.
//
// Design (gfx950): the mean drop of a placement is a sum of one cost per GPU,
// c(S) = sum of the drops of the models in S, so the optimum is a minimum
// over set partitions and a subset dynamic program finds it exactly:
//   f_k[m] = min over S, lowest(m) in S, S subset of m, |S| <= C, of
//            f_{k-1}[m \ S] + c(S),      f_0[0] = 0,
// the smallest total drop of the models in mask m on k GPUs (each partition
// of m is counted once: the block holding m's lowest model is split off
// last).  The optimum is min over k <= min(G, n) of f_k[all] / n.
//  * Layers are dense: an entry's place is its mask's rank among the kept
//    masks of its popcount (colexicographic over the positions
//    e = n - 1 - model, so that the kept masks are the first C(n - j, p)
//    ranks whatever j).  Indexed by the mask itself the few kept entries lay
//    spread over 2^n, and every read was a page of its own: 24 models on 8
//    GPUs of 3 took 0.61 ms that way.
//  * cost_kernel: one lane per candidate set S (|S| <= C, by combinatorial
//    rank), its members' drops in the aggregation's order and arithmetic;
//    the costs are also layer 1.
//  * layer_kernel: one launch per k = 2 .. G - 1 over the masks that can
//    hold k non-empty GPUs and leave a remainder the other GPUs can take.  A
//    group of lanes unranks its mask, and on the way tabulates per member
//    what it adds to the rank of a remainder and to the rank of a candidate
//    set in each role it can have (Members); a candidate's two addresses are
//    then sums of one table entry per member.  The group's lanes share the
//    candidates, and each mask records its chosen set (the first by size,
//    then by members, that attains the minimum).
//    A layer is a few million such reads out of the L2s: its chain of
//    launch, unranking and a few read batches bounds it, so a mask gets as
//    many lanes as keep the chip's lanes busy.
//  * finish_kernel: layer G's one mask (`all`), the minimum over k and a
//    backtrack through the recorded sets to one optimal placement (GPUs
//    numbered in order of their first model), in one wave.
#include <cmath>

#include "rm_common.h"

namespace rm {

constexpr int kOptBlock = 256, kCostBlock = 64;
// Lanes a layer launch aims at: two waves on every SIMD of the 256 CUs.
// Every lane of a mask unranks it, so more lanes add more work than they
// share: 24 models on 8 GPUs of 3 take 0.118 ms so, 0.16 ms with half as
// many, 0.131 ms with twice and 0.147 ms with four times as many (1.18 ms
// with every mask of a layer's popcounts, one lane each).  A layer of more masks
// than that has min_log2_lanes of them.
constexpr int64_t kLayerLanes = 256 * 4 * 2 * 64;

// Binomial coefficient C(x, y) for 0 <= y <= 4, 0 <= x <= 31 (closed forms
// with constant divisors; the products fit 32 bits).
__host__ __device__ inline int32_t binom_small(int32_t x, int32_t y)
{
    if (y < 0 || x < y) return 0;
    switch (y) {
    case 0: return 1;
    case 1: return x;
    case 2: return x * (x - 1) / 2;
    case 3: return x * (x - 1) * (x - 2) / 6;
    default: return x * (x - 1) * (x - 2) * (x - 3) / 24;
    }
}

// Index of the first set of each size in the cost table: sizes 1..C in turn.
__host__ __device__ inline int32_t size_base(int32_t n, int32_t s)
{
    int32_t b = 0;
    for (int32_t t = 1; t < s; ++t) b += binom_small(n, t);
    return b;
}

// Number of candidate sets of at most C of n models.
__host__ __device__ inline int32_t n_sets_upto(int32_t n, int32_t C)
{
    return size_base(n, C + 1);
}

// Masks on k GPUs that can still be completed: k <= popcount <= C k and
// the n - popcount models left fit the G - k other GPUs.
__host__ __device__ inline bool layer_holds(int32_t k, int32_t p, int32_t n, int32_t C, int32_t G)
{
    if (k == 0) return p == 0;
    return p >= k && p <= C * k && n - p <= C * (G - k);
}

// Sets split off before a mask of popcount p is left, at least: each holds
// the lowest model still there, so the mask lies above that many models.
__host__ __device__ inline int32_t sets_before(int32_t n, int32_t C, int32_t p)
{
    return (n - p + C - 1) / C;
}

// Binomial coefficients C(x, y), x <= 24, y <= 24, with three zero columns
// before y = 0 (y = -3 .. -1), and the colexicographic lists of pairs
// a < b and triples a < b < c of 0 .. 22, five bits a member from the low
// end.
constexpr int kOptN = RM_MAX_OPT_MODELS;
constexpr int kBinomRow = kOptN + 4;
constexpr int kPairs = (kOptN - 1) * (kOptN - 2) / 2;
constexpr int kTriples = (kOptN - 1) * (kOptN - 2) * (kOptN - 3) / 6;

struct OptTables {
    int32_t binom[(kOptN + 1) * kBinomRow];
    uint16_t pair[kPairs], triple[kTriples];
};

constexpr OptTables make_tables()
{
    OptTables t = {};
    for (int x = 0; x <= kOptN; ++x)
        for (int y = 0; y <= x; ++y)
            t.binom[x * kBinomRow + y + 3] =
                (y == 0 || y == x) ? 1
                                   : t.binom[(x - 1) * kBinomRow + y + 2] +
                                         t.binom[(x - 1) * kBinomRow + y + 3];
    int np = 0, nt = 0;
    for (int c = 0; c < kOptN - 1; ++c)
        for (int b = 0; b < c; ++b) {
            t.pair[np++] = (uint16_t)(b | (c << 5));
            for (int a = 0; a < b; ++a) t.triple[nt++] = (uint16_t)(a | (b << 5) | (c << 10));
        }
    return t;
}

__device__ const OptTables d_tables = make_tables();
static constexpr OptTables h_tables = make_tables();

// Entries of layer k below those of popcount p.
struct LayerPlan {
    int32_t start[kOptN + 2];   // start[p]; start[n + 1] = entries in all
};

static LayerPlan layer_plan(int32_t k, int32_t n, int32_t C, int32_t G)
{
    LayerPlan plan;
    int32_t at = 0;
    for (int32_t p = 0; p < kOptN + 2; ++p) {
        plan.start[p] = at;
        if (p <= n && layer_holds(k, p, n, C, G))
            at += h_tables.binom[(n - sets_before(n, C, p)) * kBinomRow + p + 3];
    }
    return plan;
}

struct OptArgs {
    int32_t N;                 // models in the library
    const double* delay;       // N x N
    const double* iso;
    const int32_t* q;
    int32_t n;                 // models to place
    const int32_t* models;     // their ids (positions 0..n-1)
    int32_t G, C;              // GPUs used at most (min(n_devices, n)), capacity
    int32_t drop_mode;
    double* cost;              // n_sets_upto(n, C)
    double* layers;            // G x 2^n: f_1 .. f_G
    uint32_t* choice;          // G x 2^n: the other members of the chosen set
    double* best_mean;
    int32_t* best_device;
    int32_t* status;
};

__device__ inline double drop_of_set(double T_agg, double T_iso, int32_t drop_mode)
{
    if (drop_mode == RM_DROP_ADJUSTED) return T_agg > 0.0 ? (T_agg - T_iso) / T_agg : 0.0;
    return T_iso > 0.0 ? (T_agg - T_iso) / T_iso : 0.0;
}

// c(S) for every candidate set: its members' drops summed in ascending
// position, each from T~_p = T_p + sum over the other members r (ascending)
// of gamma_pr * Delta_pr -- the aggregation's expressions in its order.
// Layer 1 holds the cost of the whole mask on one GPU, for the masks it
// keeps.
__global__ __launch_bounds__(kCostBlock) void cost_kernel(OptArgs a, int32_t n_sets,
                                                          LayerPlan first)
{
    const int32_t x = (int32_t)(blockIdx.x * kCostBlock + threadIdx.x);
    if (x >= n_sets) return;
    int32_t s = 1;
    while (s < a.C && x >= size_base(a.n, s + 1)) ++s;
    int32_t r = x - size_base(a.n, s);
    // unrank: largest c_i with C(c_i, i + 1) <= r, from the top element down.
    // Every loop below runs over all four members and skips those past s, so
    // that the members stay in registers and their reads go out together.
    int32_t c[4] = {0, 0, 0, 0};
    int32_t hi = a.n;
#pragma unroll
    for (int32_t i = 3; i >= 0; --i) {
        if (i >= s) continue;
        int32_t v = hi - 1;
        while (binom_small(v, i + 1) > r) --v;
        c[i] = v;
        r -= binom_small(v, i + 1);
        hi = v;
    }
    const int64_t N = a.N;
    bool ok = true;
    int32_t m[4], q[4];
    double T[4], dl[4][4];
#pragma unroll
    for (int32_t i = 0; i < 4; ++i) m[i] = a.models[c[i]];
#pragma unroll
    for (int32_t i = 0; i < 4; ++i) {
        ok = ok && (i >= s || (m[i] >= 0 && m[i] < a.N));
        if (!(m[i] >= 0 && m[i] < a.N)) m[i] = 0;
    }
#pragma unroll
    for (int32_t i = 0; i < 4; ++i) {
        T[i] = a.iso[m[i]];
        q[i] = a.q[m[i]];
#pragma unroll
        for (int32_t t = 0; t < 4; ++t)
            dl[i][t] = (i < s && t < s && t != i) ? a.delay[m[i] * N + m[t]] : 0.0;
    }
    double sum = 0.0;
    bool bad_delay = false;
#pragma unroll
    for (int32_t p = 0; p < 4; ++p) {
        if (p >= s) continue;
        double T_agg = T[p];
#pragma unroll
        for (int32_t t = 0; t < 4; ++t) {
            if (t == p || t >= s) continue;
            bad_delay = bad_delay || !(dl[p][t] >= 0.0 && dl[p][t] <= 1.7976931348623157e308);
            T_agg = T_agg + overlap_scale(q[p], q[t]) * dl[p][t];
        }
        sum = sum + drop_of_set(T_agg, T[p], a.drop_mode);
    }
    if (!ok) {
        sum = __builtin_nan("");
        bad_delay = false;
    }
    if (bad_delay && a.status) atomicOr(a.status, RM_ST_BAD_DELAY);
    a.cost[x] = sum;
    if (!layer_holds(1, s, a.n, a.C, a.G) || c[0] < sets_before(a.n, a.C, s)) return;
    // rank over the positions n - 1 - c, the highest model first
    int32_t at = first.start[s];
    uint32_t mask = 0;
#pragma unroll
    for (int32_t i = 0; i < 4; ++i) {
        if (i >= s) continue;
        at += binom_small(a.n - 1 - c[i], s - i);
        mask |= 1u << c[i];
    }
    // no placement through a cost that is not finite
    const bool finite = sum < __builtin_inf();
    a.layers[at] = finite ? sum : __builtin_inf();
    a.choice[at] = finite ? mask & (mask - 1) : 0u;
}

// What a member of a mask adds, by its ordinal o (position order: the
// highest model has ordinal 0, the lowest, u, ordinal p - 1) and its role in
// a candidate set.  With T_j[o] the sum of C(e_i, i + 1 - j) over the
// ordinals i in [o, p - 1) -- the members from o up, j of those above them
// taken away -- the remainder's rank is
//   R                                  without u alone (R: rank of the mask
//                                      minus u's own term),
//   r01[l], r01[l] + r12[h], r01[l] + r12[m] + r23[h]
//                                      without u and one, two, three others
//                                      (l < m < h the ordinals),
// with r01[o] = R - T_0[o] + T_1[o + 1], r12[o] = T_2[o + 1] - T_1[o],
// r23[o] = T_3[o + 1] - T_2[o]; the candidate's cost rank is its size's base
// plus u plus C(c, 2), C(c, 3), C(c, 4) of the others from the lowest model
// (highest ordinal) up.
// Tables that only larger capacities read are left out (C: the capacity).
template <int C>
struct Members {
    int32_t r01[kOptN], c2[kOptN];
    int32_t r12[C >= 3 ? kOptN : 1], c3[C >= 3 ? kOptN : 1];
    int32_t r23[C >= 4 ? kOptN : 1], c4[C >= 4 ? kOptN : 1];
};

// The binomials and the list of member pairs or triples that capacity C
// reads, in LDS.
template <int C>
struct LdsTables {
    int32_t binom[(kOptN + 1) * kBinomRow];
    uint16_t pair[C >= 3 ? kPairs : 1], triple[C >= 4 ? kTriples : 1];
};

template <int C>
__device__ inline void stage_tables(LdsTables<C>& tab)
{
    for (int32_t x = threadIdx.x; x < (kOptN + 1) * kBinomRow; x += blockDim.x)
        tab.binom[x] = d_tables.binom[x];
    if (C >= 3)
        for (int32_t x = threadIdx.x; x < kPairs; x += blockDim.x) tab.pair[x] = d_tables.pair[x];
    if (C >= 4)
        for (int32_t x = threadIdx.x; x < kTriples; x += blockDim.x)
            tab.triple[x] = d_tables.triple[x];
}

// The best candidate so far: its value, its place in the enumeration (size,
// then the others' offsets p - 2 - ordinal, five bits each, the lowest model
// first), which also names the set.
struct BestSet {
    double v;
    uint32_t order;
};

__device__ inline void keep_first_min(BestSet& b, double v, uint32_t order)
{
    if (v < b.v || (v == b.v && order < b.order)) {
        b.v = v;
        b.order = order;
    }
}

constexpr int kBatch = 4;   // candidates of a lane with their reads in flight together

// Unranks mask number r of popcount p on `bits` positions into the member
// tables (every lane of the group writes the same values) and finds the
// best split of the mask on layer k > 1, shared by the group's L lanes (lane
// t): f_{k-1}[m \ S] + c(S) over the sets S = {u} + others, |S| <= C, by
// size and then by members.  Returns the smallest value and the first set
// that attains it; `mask` the mask over the models.
template <int C>
__device__ inline BestSet best_split(const OptArgs& a, int32_t k, const LdsTables<C>& tab,
                                     const LayerPlan& prev, Members<C>& mb, int32_t bits,
                                     int32_t p, int32_t r, int32_t t, int32_t L, uint32_t& mask)
{
    const int32_t* binom = tab.binom;
    mask = 0;
    int32_t i = p, u = 0, R = 0;
    int32_t t0 = 0, t1 = 0, t2 = 0, t3 = 0;
    for (int32_t e = bits - 1; e >= 0 && i > 0; --e) {
        const int32_t* row = binom + e * kBinomRow + 3 + i;   // row[0] = C(e, i)
        const int32_t b0 = row[0], b1 = row[-1], b2 = C >= 3 ? row[-2] : 0,
                      b3 = C >= 4 ? row[-3] : 0;
        if (r < b0) continue;
        r -= b0;
        const int32_t c = a.n - 1 - e;
        mask |= 1u << c;
        if (i == p) {   // u, the lowest model
            u = c;
            R = r;
        } else {
            const int32_t o = i - 1;
            const int32_t* rc = binom + c * kBinomRow + 3;
            mb.r01[o] = R - (t0 + b0) + t1;
            mb.c2[o] = rc[2];
            if (C >= 3) {
                mb.r12[o] = t2 - (t1 + b1);
                mb.c3[o] = rc[3];
            }
            if (C >= 4) {
                mb.r23[o] = t3 - (t2 + b2);
                mb.c4[o] = rc[4];
            }
            t0 += b0;
            t1 += b1;
            t2 += b2;
            t3 += b3;
        }
        --i;
    }
    __builtin_amdgcn_wave_barrier();
    const double* f = a.layers + (int64_t)(k - 2) * ((int64_t)1 << a.n);
    const int32_t P = p - 1;   // members besides u
    BestSet best = {__builtin_inf(), 0u};
    if (layer_holds(k - 1, p - 1, a.n, C, a.G) && t == 0)
        keep_first_min(best, f[prev.start[p - 1] + R] + a.cost[u], 1u << 15);
    if (C >= 2 && p >= 2 && layer_holds(k - 1, p - 2, a.n, C, a.G)) {
        const double* f2 = f + prev.start[p - 2];
        const double* g2 = a.cost + size_base(a.n, 2) + u;
        for (int32_t o = t; o < P; o += L)
            keep_first_min(best, f2[mb.r01[o]] + g2[mb.c2[o]],
                           (2u << 15) | (uint32_t)(P - 1 - o));
    }
    if (C >= 3 && p >= 3 && layer_holds(k - 1, p - 3, a.n, C, a.G)) {
        const double* f3 = f + prev.start[p - 3];
        const double* g3 = a.cost + size_base(a.n, 3) + u;
        const int32_t total = P * (P - 1) / 2;
        for (int32_t x0 = t; x0 < total; x0 += kBatch * L) {
            double fv[kBatch], gv[kBatch];
            uint32_t od[kBatch];
#pragma unroll
            for (int32_t b = 0; b < kBatch; ++b) {
                const int32_t x = x0 + b * L;
                const uint32_t w = tab.pair[x < total ? x : x0];
                const int32_t l = (int32_t)(w & 31u), h = (int32_t)(w >> 5);
                fv[b] = f3[mb.r01[l] + mb.r12[h]];
                gv[b] = g3[mb.c2[h] + mb.c3[l]];
                od[b] = (3u << 15) | (uint32_t)((P - 1 - h) << 5) | (uint32_t)(P - 1 - l);
            }
#pragma unroll
            for (int32_t b = 0; b < kBatch; ++b) keep_first_min(best, fv[b] + gv[b], od[b]);
        }
    }
    if (C >= 4 && p >= 4 && layer_holds(k - 1, p - 4, a.n, C, a.G)) {
        const double* f4 = f + prev.start[p - 4];
        const double* g4 = a.cost + size_base(a.n, 4) + u;
        const int32_t total = P * (P - 1) * (P - 2) / 6;
        for (int32_t x0 = t; x0 < total; x0 += kBatch * L) {
            double fv[kBatch], gv[kBatch];
            uint32_t od[kBatch];
#pragma unroll
            for (int32_t b = 0; b < kBatch; ++b) {
                const int32_t x = x0 + b * L;
                const uint32_t w = tab.triple[x < total ? x : x0];
                const int32_t l = (int32_t)(w & 31u), m = (int32_t)((w >> 5) & 31u),
                              h = (int32_t)(w >> 10);
                fv[b] = f4[mb.r01[l] + mb.r12[m] + mb.r23[h]];
                gv[b] = g4[mb.c2[h] + mb.c3[m] + mb.c4[l]];
                od[b] = (4u << 15) | (uint32_t)((P - 1 - h) << 10) |
                        (uint32_t)((P - 1 - m) << 5) | (uint32_t)(P - 1 - l);
            }
#pragma unroll
            for (int32_t b = 0; b < kBatch; ++b) keep_first_min(best, fv[b] + gv[b], od[b]);
        }
    }
    for (int32_t o = L >> 1; o > 0; o >>= 1) {
        const double v = __shfl_xor(best.v, o, 64);
        const uint32_t od = (uint32_t)__shfl_xor((int)best.order, o, 64);
        keep_first_min(best, v, od);
    }
    return best;
}

// The members of a chosen set besides the mask's lowest model: offset x in
// the order's fields names the x-th lowest of the others.
__device__ inline uint32_t chosen_members(uint32_t mask, uint32_t order)
{
    const uint32_t size = order >> 15;
    uint32_t t = 0;
    for (uint32_t s = 2; s <= size; ++s) {
        uint32_t x = (order >> (5 * (s - 2))) & 31u, w = mask & (mask - 1);
        while (x--) w &= w - 1;
        t |= w & (0u - w);
    }
    return t;
}

// Group g of 2^log2_lanes lanes takes entry g of layer k.
template <int C>
__global__ __launch_bounds__(kOptBlock) void layer_kernel(OptArgs a, int32_t k, int32_t log2_lanes,
                                                          LayerPlan plan, LayerPlan prev)
{
    extern __shared__ int32_t lds[];
    Members<C>* members = reinterpret_cast<Members<C>*>(lds);   // one per group of lanes
    __shared__ LdsTables<C> tab;
    stage_tables(tab);
    __syncthreads();
    const int32_t L = 1 << log2_lanes;
    const int32_t group = (int32_t)((blockIdx.x * kOptBlock + threadIdx.x) >> log2_lanes);
    const int32_t t = (int32_t)threadIdx.x & (L - 1);
    int32_t p = 0;
    while (p <= a.n && group >= plan.start[p + 1]) ++p;
    if (p > a.n) return;   // the group's lanes leave together
    uint32_t mask;
    const BestSet best = best_split(a, k, tab, prev, members[threadIdx.x >> log2_lanes],
                                    a.n - sets_before(a.n, C, p), p, group - plan.start[p], t, L,
                                    mask);
    if (t == 0) {
        const int64_t at = (int64_t)(k - 1) * ((int64_t)1 << a.n) + group;
        a.layers[at] = best.v;
        a.choice[at] = chosen_members(mask, best.order);
    }
}

// One wave: layer G's mask (`all`, split over the 64 lanes; layer 1 comes
// from the costs), the optimum over k and one placement attaining it.
template <int C>
__global__ __launch_bounds__(64) void finish_kernel(OptArgs a, LayerPlan prev)
{
    __shared__ Members<C> members;
    __shared__ LdsTables<C> tab;
    const int32_t n = a.n, lane = threadIdx.x;
    bool mine = true;
    for (int32_t p = lane; p < n; p += 64) mine = mine && a.models[p] >= 0 && a.models[p] < a.N;
    if (__ballot(!mine)) {
        if (lane == 0) {
            if (a.status) atomicOr(a.status, RM_ST_BAD_MODEL_ID);
            *a.best_mean = __builtin_nan("");
        }
        for (int32_t p = lane; p < n; p += 64) a.best_device[p] = -1;
        return;
    }
    if (n == 0) {
        if (lane == 0) *a.best_mean = 0.0;
        return;
    }
    stage_tables(tab);
    __syncthreads();
    const int64_t full = (int64_t)1 << n;
    const uint32_t all = (uint32_t)(full - 1);
    // place of the entry of mask m (popcount p) in layer k
    auto place_of = [&](int32_t k, uint32_t m, int32_t p) {
        int32_t x = 0;
        if (lane < p && layer_holds(k, lane, n, C, a.G))   // popcounts below p
            x = tab.binom[(n - sets_before(n, C, lane)) * kBinomRow + lane + 3];
        if (lane < n && ((m >> lane) & 1u)) {   // model `lane`: members above it rank below
            const int32_t above = __builtin_popcount(m >> lane) - 1;
            x += tab.binom[(n - 1 - lane) * kBinomRow + above + 1 + 3];
        }
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        return (int64_t)(k - 1) * full + x;
    };
    BestSet last = {__builtin_inf(), 0u};
    uint32_t mask = all;
    if (a.G > 1) last = best_split(a, a.G, tab, prev, members, n, n, 0, lane, 64, mask);
    double best = __builtin_inf();
    int32_t kb = 0;
    for (int32_t k = 1; k <= a.G; ++k) {
        if (!layer_holds(k, n, n, C, a.G)) continue;
        const double v = (k == a.G && k > 1) ? last.v : a.layers[place_of(k, all, n)];
        if (v < best) {
            best = v;
            kb = k;
        }
    }
    if (lane == 0) *a.best_mean = best / (double)n;
    // lane p: GPU of model p
    int32_t device = -1, block = 0;
    uint32_t m = all;
    for (int32_t k = kb; k >= 1 && m; --k, ++block) {
        const uint32_t t = (k == a.G && k > 1)
                               ? chosen_members(all, last.order)
                               : a.choice[place_of(k, m, __builtin_popcount(m))];
        const uint32_t S = (m & (0u - m)) | t;
        if (lane < n && ((S >> lane) & 1u)) device = block;
        m ^= S;
    }
    if (lane < n) a.best_device[lane] = device;
}

// Lanes of a mask, at least: so many that a workgroup's member tables and lists
// stay within 64 KB of LDS, which every launch may take and which leaves two or
// three workgroups a CU (two lanes a mask at capacity 3, four at capacity 4).
// Twice and four times as many lanes: 24 models on 9 GPUs of 3 0.221, 0.249, 0.267
// ms; on 12 of 3 0.57, 0.62, 0.68; on 6 of 4 0.292, 0.302, 0.339; on 12 of 4 5.27,
// 5.22, 6.30; 20 on 8 of 4 0.310, 0.282, 0.306 (one lane a mask of all popcounts:
// 4.57, 14.9, 3.62, 82.9, 2.34 ms).
template <int C>
constexpr int32_t min_log2_lanes()
{
    int32_t l = 0;
    while ((kOptBlock >> l) * sizeof(Members<C>) + sizeof(LdsTables<C>) > 65536) ++l;
    return l;
}

// Layers 2 .. G - 1 and the finish, for capacity C.
template <int C>
static hipError_t launch_layers(const OptArgs& a, LayerPlan prev, hipStream_t s)
{
    for (int32_t k = 2; k < a.G; ++k) {
        const LayerPlan plan = layer_plan(k, a.n, C, a.G);
        const int32_t masks = plan.start[a.n + 1];
        if (masks > 0) {
            int32_t log2_lanes = min_log2_lanes<C>();
            while (log2_lanes < 6 && ((int64_t)masks << log2_lanes) < kLayerLanes) ++log2_lanes;
            const int64_t lanes = (int64_t)masks << log2_lanes;
            hipLaunchKernelGGL(layer_kernel<C>,
                               dim3((unsigned)((lanes + kOptBlock - 1) / kOptBlock)),
                               dim3(kOptBlock), (kOptBlock >> log2_lanes) * sizeof(Members<C>), s,
                               a, k, log2_lanes, plan, prev);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        prev = plan;
    }
    hipLaunchKernelGGL(finish_kernel<C>, dim3(1), dim3(64), 0, s, a, prev);
    return hipGetLastError();
}

size_t place_optimal_cost_entries(int32_t n, int32_t C)
{
    return (size_t)n_sets_upto(n, C);
}

hipError_t launch_place_optimal(int32_t n_models, const double* delay, const double* iso,
                                const int32_t* q, int32_t n, const int32_t* models,
                                int32_t G, int32_t C, int32_t drop_mode, double* cost,
                                double* layers, uint32_t* choice, double* best_mean,
                                int32_t* best_device, int32_t* status, hipStream_t s)
{
    OptArgs a;
    a.N = n_models;
    a.delay = delay;
    a.iso = iso;
    a.q = q;
    a.n = n;
    a.models = models;
    a.G = G;
    a.C = C;
    a.drop_mode = drop_mode;
    a.cost = cost;
    a.layers = layers;
    a.choice = choice;
    a.best_mean = best_mean;
    a.best_device = best_device;
    a.status = status;
    const LayerPlan first = layer_plan(1, n, C, G);
    if (n > 0) {
        const int32_t sets = n_sets_upto(n, C);
        hipLaunchKernelGGL(cost_kernel, dim3((unsigned)((sets + kCostBlock - 1) / kCostBlock)),
                           dim3(kCostBlock), 0, s, a, sets, first);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    switch (C) {   // capacities up to RM_MAX_OPT_CAPACITY
    case 1: return launch_layers<1>(a, first, s);
    case 2: return launch_layers<2>(a, first, s);
    case 3: return launch_layers<3>(a, first, s);
    default: return launch_layers<4>(a, first, s);
    }
}

}  // namespace rm
