// prefix.hip -- per-model preparation for the pair sweep: the isolated
// timeline P[0] = 0, P[k+1] = P[k] + d_k (kernel order; the model's isolated
// time is T_m = P[q_m], Sec. 3.2 "Performance drop") and every kernel's
// occupancy footprint (Sec. 3.1 Eq. 1, Sec. 3.2 Eq. 2), written together as
// the 16-byte records the sweep stages.
//
// The sum is taken strictly in sequence so every boundary is the same fp64
// value the CPU oracle produces and boundary ties resolve identically: a
// chain of dependent adds, at least 2 ns each, which bounds this kernel.  One workgroup
// of six waves per model; a chunk's durations are staged into LDS by all of
// them, then its sub-chunks go through a pipeline with one barrier a step:
//  * wave 0 runs the chain over sub-chunk s.  The 16 lanes of a row hold a
//    block of 16 consecutive durations in one register, and v_fmac_f64 with
//    a row_newbcast operand adds lane k's duration (times 1, so the sum rounds
//    once, as an addition does) with no read or move between two adds; the
//    blocks ahead are in flight.  Only the running sum at the start of every
//    span of two blocks is kept.
//  * waves 2-5 compute the footprints of sub-chunk s.
//  * wave 1 finishes sub-chunk s - 1: 16 lanes redo one span's 32 adds each
//    from its starting sum -- the same additions in the same order, so the
//    same values -- and the wave writes whole 16-byte records.
// 256 models of 2000 kernels: 21.4 us with one lane reading the durations out
// of LDS value by value and the redo after the whole chain, 16.4 us now (1.9 us
// until the durations are staged, 2 us a sub-chunk, 5 us of launch).
#include "rm_common.h"

namespace rm {

constexpr int kPrepareThreads = 384;
constexpr int kBlk = 16;                    // values per block of the add chain
constexpr int kSubBlks = 32;                // blocks per sub-chunk
constexpr int kSub = kSubBlks * kBlk;
constexpr int kSpanBlks = 2;                // blocks per redo span
constexpr int kSpan = kSpanBlks * kBlk;
constexpr int kSubSpans = kSubBlks / kSpanBlks;
constexpr int kPrepareChunk = 2048;
constexpr int kStageRegs = (kPrepareChunk + kPrepareThreads - 1) / kPrepareThreads;
constexpr int kFootLanes = kPrepareThreads - 128;   // waves 2-5
constexpr int kFootRegs = kSub / kFootLanes;
static_assert(kPrepareChunk % kSub == 0 && kSub % kFootLanes == 0, "whole sub-chunks");

// LDS slot of value t of a chunk: one spare slot after every 16 values, so
// the lanes that redo consecutive spans read different banks.
__device__ inline int slot_of(int t)
{
    return t + (t >> 4);
}
constexpr int kBufSlots = kPrepareChunk + kPrepareChunk / kBlk;

// sum + x[0] + ... + x[15], one after the other, x[k] held by lane k of each
// 16-lane row.  (The wait states cover x written by an instruction just
// before: a DPP operand is read past the forwarding paths.)
__device__ inline double add_block(double sum, double x)
{
    const double one = 1.0;
#define RM_ADD(K)                                                                          \
    "v_fmac_f64_dpp %0, %1, %2 row_newbcast:" #K " row_mask:0xf bank_mask:0xf\n\t"
    asm("s_nop 1\n\t" RM_ADD(0) RM_ADD(1) RM_ADD(2) RM_ADD(3) RM_ADD(4) RM_ADD(5) RM_ADD(6)
            RM_ADD(7) RM_ADD(8) RM_ADD(9) RM_ADD(10) RM_ADD(11) RM_ADD(12) RM_ADD(13) RM_ADD(14)
                RM_ADD(15)
        : "+v"(sum)
        : "v"(x), "v"(one));
#undef RM_ADD
    return sum;
}

// The chain over a sub-chunk's values in buf (zero past the end), from `run`;
// start[kStartLane l + e] receives the running sum before redo span e, once
// per lane l, so that no lane is masked off for it (lane 0's are used).  Blocks
// go through eight at a time, the next eight read meanwhile: 2.6 ns an add
// without the stores, 3.05 ns with one per block, 3.65 ns with one per block
// by a single lane (one wave alone).
constexpr int kStartLane = kSubSpans + 1;
__device__ inline double add_chain(const double* buf, double* start, int len, int lane, double run)
{
    constexpr int kGroup = 8;
    static_assert(kSubBlks % kGroup == 0, "whole groups");
    const int nb = (len + kBlk - 1) / kBlk, l = lane & (kBlk - 1);
    start += kStartLane * lane;
    double x[kGroup];
#pragma unroll
    for (int u = 0; u < kGroup; ++u) x[u] = buf[(kBlk + 1) * u + l];
#pragma unroll 1
    for (int b = 0; b < nb; b += kGroup) {
        double y[kGroup];
        const int ahead = b + kGroup < kSubBlks ? b + kGroup : b;
#pragma unroll
        for (int u = 0; u < kGroup; ++u) y[u] = buf[(kBlk + 1) * (ahead + u) + l];
        __builtin_amdgcn_sched_barrier(0);   // these reads go out before the adds
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {   // blocks past the end add zeros
            if (u % kSpanBlks == 0) start[(b + u) / kSpanBlks] = run;
            run = add_block(run, x[u]);
        }
#pragma unroll
        for (int u = 0; u < kGroup; ++u) x[u] = y[u];
    }
    return run;
}

// What a kernel of footprint `used` leaves of an SM capacity for its partner.
__device__ inline uint32_t left_of(uint32_t cap, uint32_t used, bool half)
{
    const uint32_t held = half && used > cap / 2u ? cap / 2u : used;
    return cap - held;
}

__device__ inline SimRecord sim_record(const Desc& d, SimForm form, double dur, uint32_t beta,
                                       uint32_t wb, uint64_t rt, uint64_t m)
{
    SimRecord r;
    r.d = dur;
    if (form.general) {
        const uint64_t shape = pack_shape(beta, wb, rt, m);
        r.shape.shape_lo = (uint32_t)shape;
        r.shape.shape_hi = (uint32_t)(shape >> 32);
        // division constants of the (clamped) packed demands
        uint32_t s0, s1, s2;
        div_constant(wb & 0xffu, r.shape.mag_wb, s0);
        div_constant((uint32_t)(shape >> 16) & 0xffffffu, r.shape.mag_rt, s1);
        div_constant((uint32_t)(shape >> 40), r.shape.mag_m, s2);
        r.shape.shifts = s0 | (s1 << 8) | (s2 << 16);
        return r;
    }
    // a kernel with resident blocks demands at most the capacities
    const float inf = __builtin_inff();
    const uint32_t rt32 = beta ? (uint32_t)rt : 0u, m32 = beta ? (uint32_t)m : 0u;
    const uint32_t lw = left_of((uint32_t)d.W, beta * wb, form.half);
    const uint32_t lr = left_of((uint32_t)d.regs, beta * rt32, form.half);
    const uint32_t lm = left_of((uint32_t)d.smem, beta * m32, form.half);
    const uint32_t lb = left_of((uint32_t)d.max_blocks, beta, form.half);
    r.ready.bytes = beta | ((2u * lw + 1u) << 8) | (lb << 16) | ((beta ? beta : 1u) << 24);
    r.ready.inv_w = beta ? 1.0f / (float)(2u * wb) : inf;
    r.ready.inv_r = rt32 ? 1.0f / (float)rt32 : inf;
    r.ready.inv_m = m32 ? 1.0f / (float)m32 : inf;
    r.ready.left_r = (float)lr + 0.5f;
    r.ready.left_m = (float)lm + 0.5f;
    return r;
}

__global__ __launch_bounds__(kPrepareThreads) void prepare_kernel(
    Desc d, Packing pk, int32_t n_models, const int64_t* __restrict__ offsets,
    int64_t n_kernels, const int32_t* __restrict__ grid, const int32_t* __restrict__ threads,
    const int32_t* __restrict__ regs, const int32_t* __restrict__ smem,
    const double* __restrict__ dur, Record* __restrict__ records, SimRecord* __restrict__ sim,
    SimForm form, int64_t* __restrict__ model_first, int32_t* __restrict__ kernel_count,
    double* __restrict__ iso_time, ModelInfo* __restrict__ info, int32_t* status)
{
    __shared__ double buf[kBufSlots];
    __shared__ uint64_t fps[kPrepareChunk];
    __shared__ double start[2][kStartLane * 64];   // by sub-chunk parity
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (wave == 0) __builtin_amdgcn_s_setprio(3);   // the chain shares its SIMD
    for (int32_t m = blockIdx.x; m < n_models; m += gridDim.x) {
        int64_t first = offsets[m], last = offsets[m + 1];
        int32_t st = 0;
        if (first < 0 || last > n_kernels || last < first) {
            st |= RM_ST_BAD_OFFSETS;
            first = last = 0;
        }
        const int64_t q = last - first;
        if (q == 0 && tid == 0) st |= RM_ST_EMPTY_MODEL;
        const auto length = [&](int64_t c) {
            return (int)((q - c) < kPrepareChunk ? (q - c) : kPrepareChunk);
        };
        // a chunk's durations, every load in flight; past the end the last one
        double next[kStageRegs];
        const auto request = [&](int64_t c) {
            const int len = length(c);
#pragma unroll
            for (int u = 0; u < kStageRegs; ++u) {
                const int t = tid + kPrepareThreads * u;
                next[u] = dur[first + c + (t < len ? t : len - 1)];
            }
        };
        double run = 0.0;   // meaningful in wave 0 only
        if (q > 0) request(0);
        for (int64_t c = 0; c < q; c += kPrepareChunk) {
            const int len = length(c);
#pragma unroll
            for (int u = 0; u < kStageRegs; ++u) {
                const int t = tid + kPrepareThreads * u;
                if (t < len && (!(next[u] > 0.0) || !isfinite(next[u]))) st |= RM_ST_BAD_DURATION;
                if (t < kPrepareChunk) buf[slot_of(t)] = t < len ? next[u] : 0.0;
            }
            if (c + kPrepareChunk < q) request(c + kPrepareChunk);
            // launch shapes of waves 2-5's kernels of a sub-chunk
            int32_t G[kFootRegs], T[kFootRegs], R[kFootRegs], M[kFootRegs];
            const auto shapes = [&](int t0) {
#pragma unroll
                for (int u = 0; u < kFootRegs; ++u) {
                    const int t = t0 + (tid - 128) + kFootLanes * u;
                    const int64_t x = first + c + (t < len ? t : len - 1);
                    G[u] = grid[x];
                    T[u] = threads[x];
                    R[u] = regs[x];
                    M[u] = smem[x];
                }
            };
            if (wave >= 2) shapes(0);
            __syncthreads();
            // steps of the pipeline: sub-chunks [0, len) and one step more
#pragma unroll 1
            for (int t0 = 0, par = 0; t0 < len + kSub; t0 += kSub, par ^= 1) {
                if (wave == 0) {
                    if (t0 < len)
                        run = add_chain(buf + slot_of(t0), start[par],
                                        len - t0 < kSub ? len - t0 : kSub, lane, run);
                } else if (wave == 1) {
                    const int f0 = t0 - kSub;   // the sub-chunk to finish
                    if (f0 >= 0 && f0 < len) {
                        if (lane < kSubSpans) {
                            double r = start[par ^ 1][lane];
                            double* v = buf + slot_of(f0 + lane * kSpan);
#pragma unroll 1
                            for (int w = 0; w < kSpanBlks; ++w, v += kBlk + 1) {
#pragma unroll
                                for (int u = 0; u < kBlk; ++u) {
                                    r = r + v[u];
                                    v[u] = r;
                                }
                            }
                        }
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int u = 0; u < kSub / 64; ++u) {
                            const int t = f0 + lane + 64 * u;
                            Record r;
                            r.end = buf[slot_of(t)];
                            r.fp = fps[t];
                            if (t < len) records[first + c + t] = r;
                        }
                    }
                } else if (t0 < len) {
                    KernelOcc o[kFootRegs];
#pragma unroll
                    for (int u = 0; u < kFootRegs; ++u) {
                        const int t = t0 + (tid - 128) + kFootLanes * u;
                        o[u] = kernel_occupancy(d, pk, G[u], T[u], R[u], M[u]);
                        if (t < len) st |= o[u].status;
                        fps[t] = o[u].fp;
                        if (sim && t < len) {
                            const uint32_t wb = ((uint32_t)(T[u] > 0 ? T[u] : 1) +
                                                 (uint32_t)d.warp - 1u) / (uint32_t)d.warp;
                            const uint64_t rt = (uint64_t)(R[u] > 0 ? R[u] : 0) *
                                                (uint64_t)(T[u] > 0 ? T[u] : 0);
                            const uint64_t mm = (uint64_t)(M[u] > 0 ? M[u] : 0);
                            const int64_t x = first + c + t;
                            sim[x] = sim_record(d, form, dur[x], o[u].beta, wb, rt, mm);
                        }
                    }
                    if (t0 + kSub < len) shapes(t0 + kSub);
                }
                __syncthreads();
            }
        }
        if (tid == 0) {
            model_first[m] = first;
            kernel_count[m] = (int32_t)q;
            iso_time[m] = run;
            ModelInfo mi;
            mi.T = run;
            mi.first = (int32_t)first;
            mi.q = (int32_t)q;
            info[m] = mi;
        }
        report_status(status, st);
    }
}

hipError_t launch_prepare(const Desc& d, const Packing& pk, int32_t n_models,
                          const int64_t* offsets, int64_t n_kernels, const int32_t* grid,
                          const int32_t* threads, const int32_t* regs, const int32_t* smem,
                          const double* duration, Record* records, SimRecord* sim, SimForm form,
                          int64_t* model_first, int32_t* kernel_count, double* iso_time,
                          ModelInfo* info, int32_t* status, hipStream_t s)
{
    const unsigned blocks = (unsigned)(n_models < 65536 ? n_models : 65536);
    hipLaunchKernelGGL(prepare_kernel, dim3(blocks), dim3(kPrepareThreads), 0, s, d, pk,
                       n_models, offsets, n_kernels, grid, threads, regs, smem, duration,
                       records, sim, form, model_first, kernel_count, iso_time, info, status);
    return hipGetLastError();
}

}  // namespace rm
