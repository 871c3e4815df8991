// sim.hip -- the adjusted-occupancy simulation of Sec. 3.2: two models'
// kernel sequences run side by side; while the two running kernels
// interfere (Eq. 2) each keeps only the blocks that fit beside the other
// under equal partitioning ("Adjusted occupancy"), runs at o~/o of its
// isolated speed, and the first to finish hands over to the next kernel of
// its model with the other continuing from what it has left ("Two-phase
// execution", Eq. 4).  Each stretch of wall time e adds e minus the work it
// completed to the model's delay; the simulation ends when either model runs
// out of kernels.
//
// Readings (the same in the CPU oracle):
//  * equal partitioning: each of the two kernels may hold at most half of
//    every SM resource (capacity / 2, rounded down); what the partner leaves
//    of its half stays available.  b~_k = min(beta_k, left_warps / W_b,
//    left_regs / (R T), left_smem / M, left_slots), no limit from a zero
//    demand;
//  * priority-based (for Delta_ij, model j's kernel first) and
//    first-come-first-served (the kernel that was running before the other
//    started first; kernels that start together share equally): the first
//    kernel keeps all its blocks at its isolated speed, the other keeps what
//    fits beside that whole footprint and makes no progress (o/o~ = inf,
//    o~/o = 0) while not one block fits;
//  * o/o~ = beta / b~ and o~/o = b~ / beta, each one correctly rounded fp64
//    quotient (beta: the blocks Eq. 2 counts on the busiest SM);
//  * when either kernel cannot keep one block beside the other, the two
//    alternate on the SM: o/o~ = 2, o~/o = 1/2 for both;
//  * delays accumulate in time order, every operation rounded as written
//    (no contraction), so the result equals the sequential definition bit
//    for bit.
//
// Design (gfx950): the simulation is sequential in time, so a run -- one
// (pair, alignment) from start to end -- is a chain of events.  Two
// neighbouring lanes run it, each one model's side: a lane holds its model's
// running kernel, the work left on it and its delay, and reads what it needs
// of the partner's (what the partner's kernel leaves of each SM resource, its
// wall time to completion) with DPP lane swaps, most of them operands of the
// instructions that use them.  One lane for both sides took 165 to 180 VALU
// instructions an event and wave: every event in some lane either side moves
// on to its next kernel, so both moves were issued each time.  256 x 2000
// FIRST is 32,896 runs: with two lanes each they fill every SIMD with one
// wave (514 waves before).
//  * Block counts: prepare writes 1/x of each per-block demand x and what
//    the kernel leaves of each resource, as floats, so an event's three
//    floor quotients are three products, their minimum with beta and the
//    slots one integer minimum (the floats are positive, so their bits order
//    as they do) and one conversion (exact, see SimRecord).
//  * The quotients beta / b~ and b~ / beta of every block count come from an
//    LDS table (16 bytes per entry), filled once per
//    workgroup with correctly rounded quotients.  Kernels that do not interfere
//    need no test of Eq. (2): what the partner leaves then holds all beta
//    blocks, and beta / beta = 1.
//  * Each lane streams its model's 32-byte records from memory in order, the
//    next one in flight while the current event is simulated.
// Devices and tables beyond the usual form's range (sim_general) run the
// same events with integer division constants and reciprocals, and so do many
// runs under PRIORITY, one lane each (simulate_victim).
#include <algorithm>
#include <type_traits>

#include "rm_common.h"

namespace rm {

// Workgroup of many runs (few runs: one wave, see launch_runs).
constexpr int kSimBlock = 256;

// The partner lane's value (lanes 2r and 2r + 1 hold the two sides of a run).
__device__ inline uint32_t other(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppXor1, 0xF, 0xF, true);
}

__device__ inline double other(double v)
{
    return dpp_take<kDppXor1>(v);
}

__device__ inline uint32_t bits_of(float v)
{
    return __builtin_bit_cast(uint32_t, v);
}

__device__ inline float float_of(uint32_t b)
{
    return __builtin_bit_cast(float, b);
}

// A SimRecord is read as two vectors of four words: {d, d, bytes, inv_w} and
// {inv_r, inv_m, left_r, left_m} (or the general form's words).  A side holds
// its next record in such registers, and when it moves on it takes every word
// out of them (taken) before it loads the record after next over them: left
// to itself the compiler loads into other registers and copies them over at
// once, which waits for the load in the same event.
typedef uint32_t Words __attribute__((ext_vector_type(4)));

// A copy of a word into another register, made where it stands.
__device__ inline uint32_t taken(uint32_t v)
{
    uint32_t r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

__device__ inline double duration_of(Words lo)
{
    return __builtin_bit_cast(double, ((uint64_t)taken(lo.y) << 32) | taken(lo.x));
}

// Table of the quotients of an adjusted occupancy, at LDS address 0 (the
// kernels have no static LDS): row beta holds {beta / b, b / beta} for b = 1
// .. beta, before them at index 0 the entry of two kernels that cannot share
// the SM in space and alternate, {2, 1/2}, and at index -1 that of a kernel
// that waits for a partner's whole footprint, {inf, 0}.  Row 0 (a kernel with
// no resident block, which never interferes) is {1, 1} throughout.
typedef double Quotients __attribute__((ext_vector_type(2)));   // o/o~ and o~/o
typedef __attribute__((address_space(3))) Quotients* LdsQuotients;
typedef __attribute__((address_space(3))) double* LdsDouble;

__host__ __device__ constexpr uint32_t quotient_row_bytes(uint32_t max_beta)
{
    return (max_beta + 2u) * (uint32_t)sizeof(Quotients);
}

__host__ __device__ constexpr uint32_t quotient_bytes(uint32_t max_beta)
{
    return (max_beta + 1u) * quotient_row_bytes(max_beta);
}

// The reciprocals 1 / n go to LDS first (in row 0, filled last); a quotient
// is then a product and one correction step, the correctly rounded quotient
// for integers up to 255 (checked exhaustively).
__device__ inline void build_quotients(int32_t max_beta)
{
    const auto at = [](int32_t x) { return (LdsQuotients)(size_t)(16u * (uint32_t)x); };
    const int32_t row = max_beta + 2, n = row * (max_beta + 1);
    for (int32_t x = threadIdx.x; x < row; x += blockDim.x) {
        Quotients y;
        y.x = y.y = 1.0 / (double)(x ? x : 1);
        *at(x) = y;
    }
    __syncthreads();
    for (int32_t x = row + (int32_t)threadIdx.x; x < n; x += blockDim.x) {
        const int32_t beta = x / row, b = x - beta * row - 1;
        const double yb = at(b > 0 ? b : 1)->x, ybeta = at(beta)->x;
        Quotients e;
        e.x = b > 0 ? div_by_recip((double)beta, (double)b, yb) : 2.0;
        e.y = b > 0 ? div_by_recip((double)b, (double)beta, ybeta) : 0.5;
        if (b < 0) {
            e.x = __builtin_inf();
            e.y = 0.0;
        }
        *at(x) = e;
    }
    __syncthreads();
    for (int32_t x = threadIdx.x; x < row; x += blockDim.x) {
        Quotients one;
        one.x = one.y = 1.0;
        *at(x) = one;
    }
    __syncthreads();
}

// How a lane's kernel runs beside its partner's: the two together, or one of
// them first (it has priority or was running before).
constexpr int kTogether = 0, kOwnFirst = 1, kOtherFirst = 2;

// A model's records in order, through a buffer descriptor: 32-bit offsets,
// and reads past the table's end give 0 (a side requests up to two records
// past its model's last, which are never used).
struct BufferStream {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t next, end;   // offsets of the record to load, and of it when the model is done

    __device__ BufferStream(const SweepArgs& g, int32_t first, int32_t q, int32_t k)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<SimRecord*>(g.sim), 0,
                                                 (int)((uint32_t)g.n_kernels * 32u), 0x00027000)),
          next(32u * (uint32_t)(first + k)), end(32u * (uint32_t)(first + q + 2))
    {
    }
    __device__ void step() { next += 32u; }
    __device__ bool done() const { return next == end; }   // after the step past the last kernel
    __device__ Words lo() const { return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)next, 0, 0); }
    __device__ Words hi() const
    {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)next + 16, 0, 0);
    }
};

// The same by pointers, for tables of any size; the last record is read
// again instead of those past it.
struct PointerStream {
    const Words* base;
    int32_t k, q;   // the record to load

    __device__ PointerStream(const SweepArgs& g, int32_t first, int32_t q_, int32_t k_)
        : base(reinterpret_cast<const Words*>(g.sim + first)), k(k_), q(q_)
    {
    }
    __device__ void step() { ++k; }
    __device__ bool done() const { return k == q + 2; }
    __device__ const Words* at() const { return base + 2 * (int64_t)(k < q ? k : q - 1); }
    __device__ Words lo() const { return at()[0]; }
    __device__ Words hi() const { return at()[1]; }
};

// The running kernel of one side in the usual form: blocks() counts the blocks
// it keeps beside what its partner leaves (at least 1 for a kernel with no
// resident block, which never interferes), entry() gives the quotients of that
// count, of 0 (the two alternate) or of kWaits.
constexpr uint32_t kWaits = ~0u;   // index -1
struct ReadyKernel {
    static constexpr bool kTable = true;          // reads the table of quotients
    static constexpr uint32_t kMany = 100;        // above the most blocks of a kernel
    using Stream = BufferStream;
    float inv_w, inv_r, inv_m;
    uint32_t beta;                                // the float's bits
    uint32_t left_w, left_r, left_m, left_b;      // floats' bits, for the partner
    uint32_t row;                                 // LDS address of its row of quotients

    static __device__ void build(int32_t max_beta) { build_quotients(max_beta); }

    // What its own blocks need and what it leaves, of a record.
    __device__ void set_own(Words lo, Words hi, uint32_t row_bytes)
    {
        const uint32_t bytes = lo.z;   // (converted, so copied)
        inv_w = float_of(taken(lo.w));
        inv_r = float_of(taken(hi.x));
        inv_m = float_of(taken(hi.y));
        beta = bits_of((float)(bytes >> 24));
        row = __umul24(bytes & 0xffu, row_bytes);
    }
    static __device__ Words left_hi(const Stream& s) { return s.hi(); }

    template <int POLICY>
    __device__ void set_left(const SweepArgs&, Words lo, Words hi)
    {
        const uint32_t bytes = lo.z;
        left_r = taken(hi.z);
        left_m = taken(hi.w);
        left_w = bits_of((float)((bytes >> 8) & 0xffu));
        left_b = bits_of((float)((bytes >> 16) & 0xffu));
    }

    // Equal partitioning: at least the upper half of each capacity is left.
    static __device__ void at_least_half(const SweepArgs& g, uint32_t& lw, uint32_t& lr,
                                         uint32_t& lm, uint32_t& lb)
    {
        lw = max(lw, bits_of((float)(2u * (g.cap_w - g.cap_w / 2u) + 1u)));
        lr = max(lr, bits_of((float)(g.cap_r - g.cap_r / 2u) + 0.5f));
        lm = max(lm, bits_of((float)(g.cap_m - g.cap_m / 2u) + 0.5f));
        lb = max(lb, bits_of((float)(g.cap_b - g.cap_b / 2u)));
    }

    __device__ uint32_t blocks(uint32_t lw, uint32_t lr, uint32_t lm, uint32_t lb) const
    {
        const uint32_t fit = min(min(bits_of(float_of(lw) * inv_w), bits_of(float_of(lr) * inv_r)),
                                 bits_of(float_of(lm) * inv_m));
        return (uint32_t)float_of(min(min(beta, lb), fit));
    }

    __device__ uint32_t all_blocks() const { return (uint32_t)float_of(beta); }

    __device__ Quotients entry(uint32_t b) const
    {
        return *(LdsQuotients)(size_t)(row + (b << 4) + 16u);
    }
};

// floor(left / x) for left below 2^23 through x's division constant (exact,
// see div_constant); `none` when x = 0.
__device__ inline uint32_t fit(uint32_t left, uint32_t x, uint32_t mag, uint32_t sh, uint32_t none)
{
    const uint32_t q = (uint32_t)(((uint64_t)left * mag) >> sh);
    return x ? q : none;
}

// The running kernel of one side in the general form.  The reciprocals 1 / n of
// the block counts (at most 255) are at LDS address 0.
constexpr size_t kReciprocalLds = 256 * sizeof(double);
struct ShapeKernel {
    static constexpr bool kTable = false;
    static constexpr uint32_t kMany = 256;
    using Stream = PointerStream;
    uint32_t beta, wb, rt, m;         // no demand of a kernel with no resident block
    uint32_t left_w, left_r, left_m, left_b;
    uint32_t mag_wb, mag_rt, mag_m;   // division constants of the three demands
    uint32_t shifts;

    static __device__ void build(int32_t)
    {
        static_assert(kSimBlock * sizeof(double) == kReciprocalLds, "one entry per lane");
        *(LdsDouble)(size_t)(8u * threadIdx.x) = 1.0 / (double)(threadIdx.x ? threadIdx.x : 1u);
        __syncthreads();
    }
    static __device__ double reciprocal(uint32_t n) { return *(LdsDouble)(size_t)(8u * n); }

    static __device__ uint64_t shape_of(Words lo) { return ((uint64_t)lo.w << 32) | lo.z; }

    __device__ void set_own(Words lo, Words hi, uint32_t)
    {
        const uint64_t sh = shape_of(lo);   // (taken apart, so copied)
        beta = (uint32_t)sh & 0xffu;
        wb = beta ? (uint32_t)(sh >> 8) & 0xffu : 0u;
        rt = beta ? (uint32_t)(sh >> 16) & 0xffffffu : 0u;
        m = beta ? (uint32_t)(sh >> 40) : 0u;
        mag_wb = taken(hi.x);
        mag_rt = taken(hi.y);
        mag_m = taken(hi.z);
        shifts = taken(hi.w);
    }
    // (what it leaves follows from the first vector)
    static __device__ Words left_hi(const Stream&) { return Words{0, 0, 0, 0}; }

    template <int POLICY>
    __device__ void set_left(const SweepArgs& g, Words lo, Words)
    {
        const uint64_t sh = shape_of(lo);
        const uint32_t n = (uint32_t)sh & 0xffu;
        // a kernel with resident blocks holds at most the capacities
        left_w = (uint32_t)g.cap_w - n * ((uint32_t)(sh >> 8) & 0xffu);
        left_r = (uint32_t)g.cap_r - n * ((uint32_t)(sh >> 16) & 0xffffffu);
        left_m = (uint32_t)g.cap_m - n * (uint32_t)(sh >> 40);
        left_b = (uint32_t)g.cap_b - n;
        if (POLICY == RM_POLICY_EQUAL) at_least_half(g, left_w, left_r, left_m, left_b);
    }

    static __device__ void at_least_half(const SweepArgs& g, uint32_t& lw, uint32_t& lr,
                                         uint32_t& lm, uint32_t& lb)
    {
        lw = max(lw, (uint32_t)(g.cap_w - g.cap_w / 2));
        lr = max(lr, (uint32_t)(g.cap_r - g.cap_r / 2));
        lm = max(lm, (uint32_t)(g.cap_m - g.cap_m / 2));
        lb = max(lb, (uint32_t)(g.cap_b - g.cap_b / 2));
    }

    __device__ uint32_t blocks(uint32_t lw, uint32_t lr, uint32_t lm, uint32_t lb) const
    {
        uint32_t b = min(all_blocks(), lb);
        b = min(b, fit(lw, wb, mag_wb, shifts & 0xffu, b));
        b = min(b, fit(lr, rt, mag_rt, (shifts >> 8) & 0xffu, b));
        return min(b, fit(lm, m, mag_m, (shifts >> 16) & 0xffu, b));
    }

    __device__ uint32_t all_blocks() const { return max(beta, 1u); }

    __device__ Quotients entry(uint32_t b) const
    {
        const uint32_t n = min(b, 255u);
        Quotients e;
        e.x = div_by_recip((double)beta, (double)n, reciprocal(n));
        e.y = div_by_recip((double)n, (double)beta, reciprocal(beta));
        if (b == 0u) {
            e.x = 2.0;
            e.y = 0.5;
        }
        if (b == kWaits) {
            e.x = __builtin_inf();
            e.y = 0.0;
        }
        if (beta == 0u) e.x = e.y = 1.0;
        return e;
    }
};

// Both, of a whole record.
template <int POLICY, typename KERNEL>
__device__ inline void set_kernel(KERNEL& k, const SweepArgs& g, Words lo, Words hi,
                                  uint32_t row_bytes)
{
    k.set_own(lo, hi, row_bytes);
    k.template set_left<POLICY>(g, lo, hi);
}

// The quotients of this side's kernel beside the partner lane's.  Two kernels
// that do not interfere (Eq. 2) need no test: what the partner leaves then holds
// all beta blocks, and beta / beta = 1.
template <int POLICY, typename KERNEL>
__device__ inline Quotients quotients(const SweepArgs& g, const KERNEL& own, int order)
{
    uint32_t lw = other(own.left_w), lr = other(own.left_r), lm = other(own.left_m),
             lb = other(own.left_b);
    if (POLICY == RM_POLICY_FCFS && order == kTogether) KERNEL::at_least_half(g, lw, lr, lm, lb);
    uint32_t b = own.blocks(lw, lr, lm, lb);
    // together: alternating when either keeps no block (the factor makes the
    // partner's count a limit only when it is 0)
    const uint32_t limit = (uint32_t)__umul24(other(b), KERNEL::kMany);
    const uint32_t both = min(b, limit);
    if (POLICY == RM_POLICY_EQUAL) {
        b = both;
    } else {
        const uint32_t alone = b ? b : kWaits;
        const uint32_t all = own.all_blocks();   // (here: read in a branch it costs 10%)
        b = order == kOtherFirst ? alone : order == kOwnFirst ? all : both;
    }
    return own.entry(b);
}

// min(x, y) of two times in one instruction; a NaN loses against a number,
// as with fmin (the library minimum first quiets signalling NaNs, which
// products never are).
__device__ inline double min_time(double x, double y)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}

// One side of a run: its model's records from `first`, of which kernels
// k .. q - 1 are still to run, kernel k with r isolated work left.  Both
// lanes of a run call this together; they return their model's delay when
// either model has run out of kernels.  `order` says which running kernel
// came first (FCFS; fixed under PRIORITY).
//
// One event: whether this side's kernel completes; the work left and the
// delay move on (a kernel that completes leaves r to its successor).
template <int POLICY, typename KERNEL>
__device__ inline bool event(const SweepArgs& g, const KERNEL& own, double& r, double& delay,
                             int& order)
{
    const Quotients e = quotients<POLICY>(g, own, order);
    const double t = r * e.x;          // wall time until this side's kernel completes
    const double to = other(t);
    // the stretch ends when the first kernel completes; the minimum and
    // !(a > b) treat the two models alike even for a NaN time (from a NaN
    // duration), which completes both, so every event advances
    const double len = min_time(t, to);
    const bool done = !(t > to);
    const double w = len * e.y;        // work this side completes
    delay = delay + (len - (done ? r : w));
    r = r - w;
    if (POLICY == RM_POLICY_FCFS)   // the kernel that did not complete came first
        order = done ? (!(to > t) ? kTogether : kOtherFirst) : kOwnFirst;
    return done;
}

// Both lanes of every run of which one lane is in the mask.
__device__ inline uint64_t whole_runs(uint64_t m)
{
    constexpr uint64_t kEven = 0x5555555555555555ull;
    return m | ((m & kEven) << 1) | ((m >> 1) & kEven);
}

template <int POLICY, typename KERNEL>
__device__ inline double simulate(const SweepArgs& g, int32_t first, int32_t q, int32_t k,
                                  double r, int order)
{
    const uint32_t row_bytes = quotient_row_bytes((uint32_t)g.max_beta);
    typename KERNEL::Stream stream(g, first, q, k);
    KERNEL own;
    set_kernel<POLICY>(own, g, stream.lo(), stream.hi(), row_bytes);
    stream.step();
    Words lo = stream.lo(), hi = stream.hi();   // the next kernel's record
    stream.step();
    double delay = 0.0;
    for (;;) {
        if (event<POLICY>(g, own, r, delay, order)) {
            r = duration_of(lo);
            set_kernel<POLICY>(own, g, lo, hi, row_bytes);
            __builtin_amdgcn_sched_barrier(0);   // the record has been read: load over it
            lo = stream.lo();
            hi = stream.hi();
            stream.step();
        }
        const uint64_t over = __ballot(stream.done());
        if (over && __builtin_amdgcn_inverse_ballot_w64(whole_runs(over))) break;
    }
    return delay;
}

// The same for few runs, where nothing but the wave itself hides a load: the
// records of a side are requested kAhead kernels ahead.  A request stays in
// flight for kAhead events (the event loop is unrolled by kAhead, each event
// with registers of its own for it) and is then written to the lane's ring
// of kAhead records in LDS; the next kernel's record is read from the ring
// into registers one event before it can be needed.  The request is issued
// by every lane in every event, so that its place among the others in flight
// is known: a lane whose kernel did not complete requests an offset past the
// table, which reads no memory, and writes to a spare slot of its ring.  A
// record requested when kernel k starts, k + 1 + kAhead, is in the ring from
// the kAhead-th event on, and needed after kAhead of this side's kernels have
// completed at the earliest; its slot is that of record k + 1, read before.
constexpr int kAhead = 4;
constexpr uint32_t kRingSlot = 64 * 16;                           // one vector per lane
constexpr uint32_t kRingBytes = (kAhead + 1) * 2 * kRingSlot;     // of one wave; the last slot is spare
typedef __attribute__((address_space(3))) Words* LdsWords;

template <int POLICY>
__device__ inline double simulate_ahead(const SweepArgs& g, int32_t first, int32_t q, int32_t k,
                                        double r, int order)
{
    const uint32_t row_bytes = quotient_row_bytes((uint32_t)g.max_beta);
    const uint32_t ring = quotient_bytes((uint32_t)g.max_beta) + 16u * (threadIdx.x & 63u);
    const uint32_t spare = ring + kAhead * 2u * kRingSlot;
    // slot of the record at table offset x (32 bytes a record)
    const auto slot_of = [&](uint32_t x) {
        static_assert(kAhead == 4 && kRingSlot == 1024, "shift");
        return ring + ((x & (32u * (kAhead - 1))) << 6);
    };
    const auto put = [](uint32_t at, Words lo, Words hi) {
        *(LdsWords)(size_t)at = lo;
        *(LdsWords)(size_t)(at + kRingSlot) = hi;
    };
    BufferStream stream(g, first, q, k);
    ReadyKernel own;
    set_kernel<POLICY>(own, g, stream.lo(), stream.hi(), row_bytes);
    stream.step();
    Words lo = stream.lo(), hi = stream.hi();   // the next kernel's record
    stream.step();
#pragma unroll
    for (int x = 0; x < kAhead; ++x) {   // records k + 2 .. k + 1 + kAhead
        put(slot_of(stream.next), stream.lo(), stream.hi());
        stream.step();
    }
    const uint32_t end = stream.end + 32u * kAhead;
    Words flo[kAhead], fhi[kAhead];   // requests in flight
    uint32_t to[kAhead];              // and their slots
#pragma unroll
    for (int x = 0; x < kAhead; ++x) {
        flo[x] = fhi[x] = Words{0, 0, 0, 0};
        to[x] = spare;
    }
    // the records read so far have landed (s_waitcnt vmcnt(0)): otherwise the
    // compiler, which sees them join the loop's own, waits for requests in
    // flight in every round
    __builtin_amdgcn_s_waitcnt(0x0F70);
    // The loop runs until every run of the wave is over, without leaving it
    // in between, so that every path through it issues the same requests; a
    // run that is over has its delay kept and goes on, on records that follow
    // its models' or on none.
    double delay = 0.0, result = 0.0;
    uint64_t running = __ballot(true);
    do {
#pragma unroll
        for (int x = 0; x < kAhead; ++x) {
            const bool done = event<POLICY>(g, own, r, delay, order);
            put(to[x], flo[x], fhi[x]);   // after the event's own, awaited LDS read
            const uint32_t slot = slot_of(stream.next);
            uint32_t from = 0xffffff00u;
            to[x] = spare;
            if (done) {
                r = duration_of(lo);
                set_kernel<POLICY>(own, g, lo, hi, row_bytes);
                __builtin_amdgcn_sched_barrier(0);   // the record has been read: read over it
                lo = *(LdsWords)(size_t)slot;
                hi = *(LdsWords)(size_t)(slot + kRingSlot);
                from = stream.next;
                to[x] = slot;
                stream.step();
            }
            flo[x] = __builtin_amdgcn_raw_buffer_load_b128(stream.rsrc, (int)from, 0, 0);
            fhi[x] = __builtin_amdgcn_raw_buffer_load_b128(stream.rsrc, (int)from + 16, 0, 0);
            uint64_t over = __ballot(stream.next == end) & running;
            if (over) {
                over = whole_runs(over);
                if (__builtin_amdgcn_inverse_ballot_w64(over)) result = delay;
                running &= ~over;
            }
        }
    } while (running);
    return result;
}

// PRIORITY with many runs (sim_one_lane): one lane a run.  Model j's kernels keep
// all their blocks and their isolated speed, and only model i's delay is wanted,
// so the second lane of a run would carry little: an event is what simulate()
// does for the one side, and a step along j's isolated timeline.  The launch is
// bound by the accesses of the lanes' record reads (address unit 80% busy, VALU
// 30%): a wave's lanes share 16 models (run_pair), and in the general form a
// kernel of model j is read with one access -- the float form's second access
// costs more than its cheaper block counts save, but for sampled starts: 1000 x
// 60 FIRST 291 us with two lanes a run, 257 us with one, 198 us in the general
// form; 128 x 60 OFFSETS(64) 333, 296, 238 us; 128 x 50..500 sampled(64) 944, 851,
// 1053 us.
template <typename KERNEL>
__device__ inline double simulate_victim(const SweepArgs& g, int32_t first_i, int32_t q_i,
                                         int32_t k_i, double r, int32_t first_j, int32_t q_j,
                                         int32_t k_j, double r_j)
{
    constexpr int kPolicy = RM_POLICY_PRIORITY;
    const uint32_t row_bytes = quotient_row_bytes((uint32_t)g.max_beta);
    typename KERNEL::Stream si(g, first_i, q_i, k_i), sj(g, first_j, q_j, k_j);
    KERNEL own, first;
    own.set_own(si.lo(), si.hi(), row_bytes);
    first.template set_left<kPolicy>(g, sj.lo(), KERNEL::left_hi(sj));
    si.step();
    sj.step();
    Words lo = si.lo(), hi = si.hi();        // the next kernels' records
    Words lo_j = sj.lo(), hi_j = KERNEL::left_hi(sj);
    si.step();
    sj.step();
    double delay = 0.0;
    do {
        const uint32_t b = own.blocks(first.left_w, first.left_r, first.left_m, first.left_b);
        const Quotients e = own.entry(b ? b : kWaits);
        const double t = r * e.x;   // wall time until i's kernel completes; j's: r_j
        const double len = min_time(t, r_j);
        const bool done = !(t > r_j), done_j = !(r_j > t);
        const double w = len * e.y;
        delay = delay + (len - (done ? r : w));
        r = r - w;
        r_j = r_j - len;
        if (done) {
            r = duration_of(lo);
            own.set_own(lo, hi, row_bytes);
            __builtin_amdgcn_sched_barrier(0);   // the record has been read: load over it
            lo = si.lo();
            hi = si.hi();
            si.step();
        }
        if (done_j) {
            r_j = duration_of(lo_j);
            first.template set_left<kPolicy>(g, lo_j, hi_j);
            __builtin_amdgcn_sched_barrier(0);
            lo_j = sj.lo();
            hi_j = KERNEL::left_hi(sj);
            sj.step();
        }
    } while (!(si.done() || sj.done()));
    return delay;
}

// How a launch runs: two lanes a run, two lanes a run with records requested
// further ahead (few runs), or one lane a run (PRIORITY, many runs).
constexpr int kTwoLanes = 0, kTwoAhead = 1, kOneLane = 2;

// A run from kernel k_i of model i and kernel k_j of model j, both not begun, or
// (BEGUN) with r_i isolated work left on model i's; the delay of this lane's side
// (`odd`: model j's).  `order` is model i's.  PRIORITY: model j's kernels keep
// their blocks.
template <int POLICY, typename KERNEL, int MODE, bool BEGUN = false>
__device__ inline double run(const SweepArgs& g, bool odd, const ModelInfo& mi, int32_t k_i,
                             const ModelInfo& mj, int32_t k_j, int order, double r_i = 0.0)
{
    if constexpr (MODE == kOneLane) {
        if (!BEGUN) r_i = g.sim[mi.first + k_i].d;
        return simulate_victim<KERNEL>(g, mi.first, mi.q, k_i, r_i, mj.first, mj.q, k_j,
                                       g.sim[mj.first + k_j].d);
    } else {
        if (POLICY == RM_POLICY_PRIORITY) order = kOtherFirst;
        if (odd && order != kTogether) order = order == kOwnFirst ? kOtherFirst : kOwnFirst;
        const int32_t first = odd ? mj.first : mi.first, q = odd ? mj.q : mi.q, k = odd ? k_j : k_i;
        double r = g.sim[first + k].d;
        if (BEGUN && !odd) r = r_i;
        if constexpr (MODE == kTwoAhead)
            return simulate_ahead<POLICY>(g, first, q, k, r, order);
        else
            return simulate<POLICY, KERNEL>(g, first, q, k, r, order);
    }
}

// Pair x of a launch's pairs: all ordered pairs, or the unordered ones where a run
// gives both directions (under PRIORITY the rule depends on the roles: Delta_ij
// comes from the run in which model j's kernels keep their blocks).  With one lane
// a run a wave takes a tile of 8 x 8 ordered pairs, so that it reads the records of
// 16 models instead of 65; false for a pair of a tile past the last model.
template <bool ORDERED, int MODE>
__device__ inline bool run_pair(int32_t N, int64_t x, int32_t& i, int32_t& j)
{
    if (MODE == kOneLane) {
        const int64_t tiles = (N + 7) / 8, t = x >> 6, row = t / tiles;
        const int32_t l = (int32_t)(x & 63);
        i = (int32_t)row * 8 + (l >> 3);
        j = (int32_t)(t - row * tiles) * 8 + (l & 7);
        return i < N && j < N;
    }
    if (ORDERED) {
        i = (int32_t)(x / N);
        j = (int32_t)(x - (int64_t)i * N);
    } else {
        row_pair_at(N, x, i, j);
    }
    return true;
}

static int64_t run_pairs(int64_t N, bool ordered, int mode)
{
    const int64_t tiles = (N + 7) / 8;
    return mode == kOneLane ? tiles * tiles * 64 : ordered ? N * N : N * (N + 1) / 2;
}

// body(x, odd) for the runs x of this lane and its side of them; two lanes of a
// run are neighbours.  A launch of few runs (kTwoAhead) has lanes for each.
template <int MODE, typename Body>
__device__ inline void for_runs(int64_t n_runs, Body body)
{
    const int64_t lane = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t lanes = (int64_t)gridDim.x * blockDim.x;
    if (MODE == kTwoAhead) {
        if (lane >> 1 < n_runs) body(lane >> 1, (bool)(threadIdx.x & 1));
    } else if (MODE == kTwoLanes) {
        for (int64_t x = lane >> 1; x < n_runs; x += lanes >> 1)
            body(x, (bool)(threadIdx.x & 1));
    } else {
        for (int64_t x = lane; x < n_runs; x += lanes) body(x, false);
    }
}

// ---------------------------------------------------------------------------
// FIRST: one run per pair of run_pair.
// ---------------------------------------------------------------------------
template <int POLICY, typename KERNEL, int MODE>
__global__ __launch_bounds__(MODE == kTwoAhead ? 64 : kSimBlock) void sim_first_kernel(SweepArgs g, int64_t n_runs)
{
    KERNEL::build(g.max_beta);
    for_runs<MODE>(n_runs, [&](int64_t x, bool odd) {
        int32_t i, j;
        if (!run_pair<POLICY == RM_POLICY_PRIORITY, MODE>(g.n_models, x, i, j)) return;
        const ModelInfo mi = g.info[i], mj = g.info[j];
        double D = 0.0;
        if (mi.q > 0 && mj.q > 0)
            D = run<POLICY, KERNEL, MODE>(g, odd, mi, 0, mj, 0, kTogether);
        // a self pair's two sides agree; under PRIORITY the odd side kept its blocks
        if (odd && (POLICY == RM_POLICY_PRIORITY || i == j)) return;
        const int32_t a = odd ? j : i, b = odd ? i : j;   // this side's model, the partner's
        const int64_t ab = (int64_t)a * g.n_models + b;
        g.delay[ab] = D;
        if (g.slowdown)
            g.slowdown[ab] = slowdown_of(D, odd ? mj.q : mi.q, odd ? mi.q : mj.q, odd ? mj.T : mi.T);
        if (g.per_alignment) g.per_alignment[ab] = D;
    });
}

// ---------------------------------------------------------------------------
// OFFSETS: one run per (ordered pair, offset r); model j joins
// tau_r = T_i * r / K after model i.  Run x = r * N^2 + pair, so the runs of
// a wave share r and have windows of similar length.  Model i runs alone
// until tau: its kernel running at tau keeps P_i[k+1] - tau of work.
// ---------------------------------------------------------------------------
template <int POLICY, typename KERNEL, int MODE>
__global__ __launch_bounds__(MODE == kTwoAhead ? 64 : kSimBlock) void sim_offsets_kernel(SweepArgs g, int64_t n_runs,
                                                                int64_t n_pairs)
{
    KERNEL::build(g.max_beta);
    const int32_t K = g.num_offsets;
    for_runs<MODE>(n_runs, [&](int64_t x, bool odd) {
        const int32_t r = (int32_t)(x / n_pairs);
        int32_t i, j;
        if (!run_pair<true, MODE>(g.n_models, x - (int64_t)r * n_pairs, i, j)) return;
        const int64_t p = (int64_t)i * g.n_models + j;
        const ModelInfo mi = g.info[i], mj = g.info[j];
        double D = 0.0;
        if (mi.q > 0 && mj.q > 0) {
            const double tau = mi.T * (double)r / (double)K;
            int32_t k = 0;
            double ri = g.sim[mi.first].d;
            bool i_first = false;
            if (tau > 0.0) {
                // kernels of i whose isolated interval ends by tau: P_i[k+1] <= tau
                const Record* Pi = g.rec + mi.first;   // Pi[k].end = P_i[k+1]
                int32_t lo = 0, hi = mi.q;
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (Pi[mid].end <= tau)
                        lo = mid + 1;
                    else
                        hi = mid;
                }
                k = lo;
                ri = k < mi.q ? Pi[k].end - tau : 0.0;
                // kernel k started at P_i[k], before j's first kernel unless at tau
                const double start_k = k > 0 ? Pi[k - 1].end : 0.0;
                i_first = k < mi.q && start_k < tau;
            }
            if (k < mi.q)
                D = run<POLICY, KERNEL, MODE, true>(g, odd, mi, k, mj, 0,
                                                    i_first ? kOwnFirst : kTogether, ri);
        }
        if (odd) return;
        g.align_scratch[p * K + r] = D;
        if (g.per_alignment) g.per_alignment[p * K + r] = D;
    });
}

// Whether two kernels interfere (Eq. 2): their packed footprints, the device
// bias added, reach a guard bit.
__device__ inline bool interfere(const SweepArgs& g, int64_t u, int64_t v)
{
    return ((g.rec[u].fp + g.rec[v].fp + g.bias) & g.guard) != 0;
}

// ---------------------------------------------------------------------------
// CONFLICT_STARTS: one workgroup per ordered pair; its lane pairs run start
// pairs (s_i, s_j) whose kernels interfere and write the per-alignment
// scratch ([first_i + s_i][first_j + s_j], NaN outside C_ij) that the
// reduction kernel of the temporal sweep reads.
// ---------------------------------------------------------------------------
template <int POLICY, typename KERNEL>
__global__ __launch_bounds__(kSimBlock) void sim_starts_kernel(SweepArgs g, int64_t n_pairs)
{
    KERNEL::build(g.max_beta);
    const bool odd = threadIdx.x & 1;
    const int64_t N = g.n_models;
    const int64_t nk = g.n_kernels;
    for (int64_t p = blockIdx.x; p < n_pairs; p += gridDim.x) {
        const int32_t i = (int32_t)(p / N), j = (int32_t)(p % N);
        const ModelInfo mi = g.info[i], mj = g.info[j];
        const int64_t total = (int64_t)mi.q * mj.q;
        // the reduction flags and skips pairs beyond its capacity
        if ((int64_t)mi.q + mj.q > g.pair_cap || total > g.starts_cap) continue;
        for (int64_t c = threadIdx.x >> 1; c < total; c += kSimBlock / 2) {
            const int32_t si = (int32_t)(c / mj.q), sj = (int32_t)(c - (int64_t)si * mj.q);
            double v = __builtin_nan("");
            if (interfere(g, (int64_t)mi.first + si, (int64_t)mj.first + sj)) {
                v = run<POLICY, KERNEL, kTwoLanes>(g, odd, mi, si, mj, sj, kTogether);
            }
            if (!odd) g.starts[((int64_t)mi.first + si) * nk + mj.first + sj] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// SAMPLED_STARTS: one run per (pair of run_pair, draw r); draw x of the
// unordered pair {a <= b} starts model a at kernel floor(hi32(x) q_a / 2^32)
// and model b at floor(lo32(x) q_b / 2^32).  A draw whose start kernels do
// not interfere (Eq. 2) is outside C_ij and yields NaN.  Run x = r * pairs +
// pair, so the runs of a wave share r.  The per-draw delays go to
// align_scratch ([ordered pair][r]) for the reduction kernel.
// ---------------------------------------------------------------------------
template <int POLICY, typename KERNEL, int MODE>
__global__ __launch_bounds__(MODE == kTwoAhead ? 64 : kSimBlock) void sim_sampled_kernel(SweepArgs g, int64_t n_runs,
                                                                int64_t n_pairs)
{
    KERNEL::build(g.max_beta);
    const int64_t N = g.n_models;
    const int32_t K = g.num_offsets;
    for_runs<MODE>(n_runs, [&](int64_t x, bool odd) {
        const int32_t r = (int32_t)(x / n_pairs);
        int32_t i, j;
        if (!run_pair<POLICY == RM_POLICY_PRIORITY, MODE>(g.n_models, x - (int64_t)r * n_pairs, i, j))
            return;
        const ModelInfo mi = g.info[i], mj = g.info[j];
        double D = __builtin_nan("");
        if (mi.q > 0 && mj.q > 0) {
            const int64_t lo = i < j ? i : j, hi = i < j ? j : i;
            const uint64_t w = g.draws[(row_start(N, lo) + (hi - lo)) * K + r];
            const uint32_t wi = i <= j ? (uint32_t)(w >> 32) : (uint32_t)w;
            const uint32_t wj = i <= j ? (uint32_t)w : (uint32_t)(w >> 32);
            const int32_t si = sampled_start(wi, mi.q), sj = sampled_start(wj, mj.q);
            if (interfere(g, (int64_t)mi.first + si, (int64_t)mj.first + sj)) {
                D = run<POLICY, KERNEL, MODE>(g, odd, mi, si, mj, sj, kTogether);
            }
        }
        if (odd && (POLICY == RM_POLICY_PRIORITY || i == j)) return;
        const int64_t a = odd ? j : i, b = odd ? i : j;
        g.align_scratch[(a * N + b) * K + r] = D;
    });
}

// ---------------------------------------------------------------------------
// launchers: one kernel per scheduler policy, record form and way of reading
// ahead, so that a kernel holds one event loop (the policies together in one
// kernel took about 60% more registers and halved the waves a SIMD holds)
// ---------------------------------------------------------------------------

// Runs so few that all their waves are on the chip at once, five to a CU by
// the LDS of a 32-block device: then what a run waits for bounds the launch,
// records are requested further ahead and every wave is a workgroup of its
// own, so that the waves spread evenly.  256 x 2000 FIRST, 1028 waves: 0.775
// ms against 0.88 ms without reading ahead (1.08 ms in workgroups of four
// waves).  With more runs other waves fill the waits, and four waves share
// one table of quotients: edge OFFSETS(64), 32,768 waves, 2.61 ms against
// 2.81 ms with a table per wave.
constexpr int64_t kAheadWaves = 5 * 256;
constexpr size_t kAheadLds = 32 * 1024;
constexpr int64_t kSimLanes = int64_t(1) << 31;   // of one dispatch, at most

static size_t ahead_lds(const SweepArgs& a)
{
    return (size_t)quotient_bytes((uint32_t)a.max_beta) + kRingBytes;
}

template <typename KERNEL, int MODE>
struct RunKind {
    using Kernel = KERNEL;
    static constexpr int kMode = MODE;
};

template <typename Launch>
static hipError_t pick_policy(const SweepArgs& a, Launch launch)
{
    switch (a.policy) {
    case RM_POLICY_PRIORITY: return launch(std::integral_constant<int, RM_POLICY_PRIORITY>{});
    case RM_POLICY_FCFS: return launch(std::integral_constant<int, RM_POLICY_FCFS>{});
    default: return launch(std::integral_constant<int, RM_POLICY_EQUAL>{});
    }
}

// launch(policy, kind of run, workgroups, lanes of one, LDS bytes, runs, pairs) for
// K runs of each pair (FLOAT_ONE_LANE: also in the usual form on one lane each).  A
// dispatch holds fewer than 2^32 work-items; the workgroups
// of a larger one loop over the runs.
template <bool FLOAT_ONE_LANE, typename Launch>
static hipError_t launch_runs(const SweepArgs& a, bool ordered, int64_t K, Launch launch)
{
    return pick_policy(a, [&](auto policy) {
        const auto with = [&](auto kind, int block, size_t lds) {
            constexpr int kMode = decltype(kind)::kMode;
            const int64_t n_pairs = run_pairs(a.n_models, ordered, kMode), n_runs = n_pairs * K;
            const int64_t lanes = kMode == kOneLane ? n_runs : 2 * n_runs;
            const int64_t blocks = std::min((lanes + block - 1) / block, kSimLanes / block);
            return launch(policy, kind, dim3((unsigned)blocks), dim3((unsigned)block), lds, n_runs,
                          n_pairs);
        };
        const int64_t n_runs = run_pairs(a.n_models, ordered, kTwoLanes) * K;
        const size_t table = quotient_bytes((uint32_t)a.max_beta);
        if constexpr (decltype(policy)::value == RM_POLICY_PRIORITY) {
            if constexpr (FLOAT_ONE_LANE)
                if (a.sim_one_lane && !a.sim_general)
                    return with(RunKind<ReadyKernel, kOneLane>{}, kSimBlock, table);
            if (a.sim_one_lane)
                return with(RunKind<ShapeKernel, kOneLane>{}, kSimBlock, kReciprocalLds);
        }
        if (a.sim_general)
            return with(RunKind<ShapeKernel, kTwoLanes>{}, kSimBlock, kReciprocalLds);
        if (2 * n_runs <= kAheadWaves * 64 && ahead_lds(a) <= kAheadLds)
            return with(RunKind<ReadyKernel, kTwoAhead>{}, 64, ahead_lds(a));
        return with(RunKind<ReadyKernel, kTwoLanes>{}, kSimBlock, table);
    });
}

hipError_t launch_sim_first(const SweepArgs& a, hipStream_t s)
{
    return launch_runs<false>(a, a.policy == RM_POLICY_PRIORITY, 1, [&](auto policy, auto kind, dim3 blocks, dim3 block,
            size_t lds, int64_t n_runs, int64_t) {
        using K = decltype(kind);
        hipLaunchKernelGGL(
            (sim_first_kernel<decltype(policy)::value, typename K::Kernel, K::kMode>), blocks, block,
            lds, s, a, n_runs);
        return hipGetLastError();
    });
}

hipError_t launch_sim_offsets(const SweepArgs& a, hipStream_t s)
{
    return launch_runs<false>(a, true, a.num_offsets, [&](auto policy, auto kind, dim3 blocks, dim3 block,
            size_t lds, int64_t n_runs, int64_t n_pairs) {
        using K = decltype(kind);
        hipLaunchKernelGGL(
            (sim_offsets_kernel<decltype(policy)::value, typename K::Kernel, K::kMode>), blocks, block,
            lds, s, a, n_runs, n_pairs);
        return hipGetLastError();
    });
}

hipError_t launch_sim_sampled(const SweepArgs& a, hipStream_t s)
{
    return launch_runs<true>(a, a.policy == RM_POLICY_PRIORITY, a.num_offsets, [&](auto policy, auto kind, dim3 blocks, dim3 block,
            size_t lds, int64_t n_runs, int64_t n_pairs) {
        using K = decltype(kind);
        hipLaunchKernelGGL(
            (sim_sampled_kernel<decltype(policy)::value, typename K::Kernel, K::kMode>), blocks, block,
            lds, s, a, n_runs, n_pairs);
        return hipGetLastError();
    });
}

hipError_t launch_sim_starts(const SweepArgs& a, hipStream_t s)
{
    const int64_t N = a.n_models;
    const int64_t n_pairs = N * N;
    const int64_t cap = int64_t(1) << 20;
    const unsigned blocks = (unsigned)(n_pairs < cap ? n_pairs : cap);
    return pick_policy(a, [&](auto policy) {
        constexpr int kPolicy = decltype(policy)::value;
        if (a.sim_general)
            hipLaunchKernelGGL((sim_starts_kernel<kPolicy, ShapeKernel>), dim3(blocks),
                               dim3(kSimBlock), kReciprocalLds, s, a, n_pairs);
        else
            hipLaunchKernelGGL((sim_starts_kernel<kPolicy, ReadyKernel>), dim3(blocks),
                               dim3(kSimBlock), quotient_bytes((uint32_t)a.max_beta), s, a,
                               n_pairs);
        return hipGetLastError();
    });
}

// The kernels of this file keep their tables and the ring at LDS address 0 and
// after it (see lds_from_zero).
template <int POLICY, typename KERNEL, int MODE>
static void add_kernels(const void** list, int& n)
{
    list[n++] = reinterpret_cast<const void*>(sim_first_kernel<POLICY, KERNEL, MODE>);
    list[n++] = reinterpret_cast<const void*>(sim_offsets_kernel<POLICY, KERNEL, MODE>);
    list[n++] = reinterpret_cast<const void*>(sim_sampled_kernel<POLICY, KERNEL, MODE>);
}

template <int POLICY>
static void add_policy(const void** list, int& n)
{
    add_kernels<POLICY, ReadyKernel, kTwoLanes>(list, n);
    add_kernels<POLICY, ReadyKernel, kTwoAhead>(list, n);
    add_kernels<POLICY, ShapeKernel, kTwoLanes>(list, n);
    list[n++] = reinterpret_cast<const void*>(sim_starts_kernel<POLICY, ReadyKernel>);
    list[n++] = reinterpret_cast<const void*>(sim_starts_kernel<POLICY, ShapeKernel>);
}

hipError_t sim_lds_from_zero(bool* ok)
{
    static std::atomic<int> state{0};
    const void* list[3 * 11 + 4];
    int n = 0;
    add_policy<RM_POLICY_EQUAL>(list, n);
    add_policy<RM_POLICY_PRIORITY>(list, n);
    add_policy<RM_POLICY_FCFS>(list, n);
    add_kernels<RM_POLICY_PRIORITY, ShapeKernel, kOneLane>(list, n);
    list[n++] = reinterpret_cast<const void*>(
        sim_sampled_kernel<RM_POLICY_PRIORITY, ReadyKernel, kOneLane>);
    return lds_from_zero(list, n, state, ok);
}

}  // namespace rm
