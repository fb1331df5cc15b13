// Collectives of one clock step on P virtual ranks in HBM:
//   - the staleness decision of Algorithm 1 (fused into both kernels below),
//   - allgatherv-style assembly into the last-received vector,
//   - the partial allreduce with stale substitution and the min-clock rule.
//
// Both kernels read the versions of the previous step from one half of a
// double buffer and write the new versions to the other half, so the
// workgroups that copy or reduce data (which all evaluate the decision for
// the ranks they touch) never race with the workgroup that records it.
#include <algorithm>
#include <type_traits>

#include "ecc_common.h"

namespace ecc {

// Assembly: workgroup 0 records the step; workgroup 1 + k copies tile k if
// its rank's block is taken at this step.  Copies use 16-byte accesses when
// source and destination have the same alignment modulo 16 bytes.
__global__ __launch_bounds__(kAssembleThreads) void k_assemble(
    int32_t P, int32_t S, int64_t t, const uint8_t *__restrict__ arrived,
    const int32_t *__restrict__ ver_in, int32_t *__restrict__ ver_out,
    int32_t *__restrict__ age_state, uint8_t *__restrict__ eff_state,
    unsigned long long *__restrict__ forced, uint8_t *__restrict__ eff_user,
    int32_t *__restrict__ age_user, const Tile *__restrict__ tiles,
    const int64_t *__restrict__ displs, const double *const *__restrict__ send_ptrs,
    const double *__restrict__ send_base, double *__restrict__ recv,
    const int32_t *__restrict__ done) {
    if (done && *done) return;
    if (blockIdx.x == 0) {
        record_step(P, S, t, arrived, ver_in, ver_out, age_state, eff_state, forced, eff_user,
                    age_user, nullptr);
        return;
    }
    const Tile tile = tiles[blockIdx.x - 1];
    const int32_t p = tile.rank;
    if (!stale_select(ver_in[p], arrived[p], t, S)) return;
    const int64_t d0 = displs[p];
    const double *src = (send_ptrs ? send_ptrs[p] : send_base + d0) + tile.off;
    double *dst = recv + d0 + tile.off;
    const int32_t len = tile.len;
    const int tid = threadIdx.x;
    if ((((uintptr_t)src ^ (uintptr_t)dst) & 15) == 0) {
        const int32_t h = (((uintptr_t)dst & 15) != 0 && len > 0) ? 1 : 0;
        if (tid == 0 && h) dst[0] = src[0];
        const int32_t body = len - h;
        const int32_t npair = body >> 1;
        const double2 *s2 = reinterpret_cast<const double2 *>(src + h);
        double2 *d2 = reinterpret_cast<double2 *>(dst + h);
        static_assert(kAssembleTile / 2 / kAssembleThreads == 4, "four pairs per thread");
        // reads are clamped into range so that all four are in flight together
        if (npair > 0) {
            const int32_t last = npair - 1;
            const int32_t k0 = tid, k1 = tid + kAssembleThreads, k2 = tid + 2 * kAssembleThreads,
                          k3 = tid + 3 * kAssembleThreads;
            const double2 v0 = s2[min(k0, last)], v1 = s2[min(k1, last)],
                          v2 = s2[min(k2, last)], v3 = s2[min(k3, last)];
            if (k0 < npair) d2[k0] = v0;
            if (k1 < npair) d2[k1] = v1;
            if (k2 < npair) d2[k2] = v2;
            if (k3 < npair) d2[k3] = v3;
        }
        if (tid == 0 && (body & 1)) dst[len - 1] = src[len - 1];
    } else {
        static_assert(kAssembleTile / kAssembleThreads == 8, "eight elements per thread");
        if (len > 0) {
            const int32_t last = len - 1;
            double v[8];
            // fully unrolled with clamped reads: the array lives in registers
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[min(tid + u * kAssembleThreads, last)];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int32_t k = tid + u * kAssembleThreads;
                if (k < len) dst[k] = v[u];
            }
        }
    }
}

// Partial allreduce: workgroup 0 records the step; every other workgroup owns
// NTH * VP * W consecutive elements and, for p = 0..P-1 in order, takes the
// fresh contribution of eff ranks (writing it to the rank's slot) or the slot
// of the others, summing in rank order.  A contribution that its producer
// wrote into the slot itself (fresh[p] == slots[p]) is read there and not
// written back.  Memory-bound: 8 m (P + taken + 1) bytes, one add per element
// read.
//
// Each workgroup stages its ranks' source and slot addresses in LDS once, so
// that the loads of U ranks go out together with no pointer chase between
// them, and W = 2 moves 16 bytes per lane at any 8-byte alignment (gfx950
// takes such accesses unaligned).  The last pair of an odd vector is moved
// back by one element: two lanes then handle the same element with the same
// values.
//
// Loads and stores retire through one in-order counter, so the first load
// awaited after a batch's slot stores waits for those stores.  SPLIT takes
// the stores out of the chain: the grid's first workgroups only sum (eff
// ranks are read from fresh, which the slots will equal), further workgroups
// copy fresh to slot, 4 vectors per thread, and no workgroup reads what
// another writes.  HELD: fresh and slots are the same array, so nothing is
// copied.
struct ReduceArgs {
    int32_t P, S;
    int64_t t;
    const uint8_t *arrived;
    const int32_t *ver_in;
    int32_t *ver_out;
    int32_t *age_state;
    uint8_t *eff_state;
    unsigned long long *forced;
    uint8_t *eff_user;
    int32_t *result_clock;
    int64_t m;
    const double *const *fresh;
    double *const *slots;
    double *result;
    int64_t n_sum;  // workgroups that sum (SPLIT: followed by those that copy)
};

constexpr int kReduceCopies = 4;   // SPLIT: vectors one thread of a copying workgroup moves
constexpr int kReduceStage = 256;  // ranks staged in LDS at a time

template <int NTH, int W, int VP, int U, bool SPLIT, bool HELD = false>
__global__ __launch_bounds__(NTH) void k_allreduce(ReduceArgs a) {
    using T = typename WordVec<W>::t;
    __shared__ uint64_t s_src[kReduceStage], s_dst[kReduceStage];
    const int tid = threadIdx.x;
    const int64_t m = a.m;
    if (blockIdx.x == 0) {
        record_step(a.P, a.S, a.t, a.arrived, a.ver_in, a.ver_out, a.age_state, a.eff_state,
                    a.forced, a.eff_user, nullptr, a.result_clock);
        return;
    }
    if constexpr (SPLIT) {
        if ((int64_t)blockIdx.x > a.n_sum) {
            constexpr int64_t chunk = (int64_t)NTH * W * kReduceCopies;
            const uint32_t chunks = (uint32_t)((m + chunk - 1) / chunk);
            const uint32_t b = (uint32_t)(blockIdx.x - 1 - a.n_sum);
            const int32_t p = (int32_t)(b / chunks);
            if (!stale_select(a.ver_in[p], a.arrived[p], a.t, a.S)) return;
            const double *src = a.fresh[p];
            double *dst = a.slots[p];
            if (src == dst) return;
            const int64_t e0 = (int64_t)(b % chunks) * chunk + (int64_t)tid * W;
            T v[kReduceCopies];
#pragma unroll
            for (int j = 0; j < kReduceCopies; ++j)
                v[j] = *(GlobalPtr<const T>)(src + min(e0 + (int64_t)j * NTH * W, m - W));
#pragma unroll
            for (int j = 0; j < kReduceCopies; ++j) {
                const int64_t e = e0 + (int64_t)j * NTH * W;
                if (e < m) *(GlobalPtr<T>)(dst + min(e, m - W)) = v[j];
            }
            return;
        }
    }
    const int64_t base = (int64_t)(blockIdx.x - 1) * (NTH * VP * W);
    int64_t at[VP];
    bool in[VP];
    T acc[VP];
#pragma unroll
    for (int j = 0; j < VP; ++j) {
        const int64_t e = base + ((int64_t)j * NTH + tid) * W;
        in[j] = e < m;
        at[j] = min(e, m - W);  // lanes past the end read the last vector
        acc[j] = T(0.0);
    }
    for (int32_t c0 = 0; c0 < a.P; c0 += kReduceStage) {
        const int32_t nc = min(kReduceStage, a.P - c0);
        if (c0) __syncthreads();
        for (int32_t k = tid; k < nc; k += NTH) {
            const int32_t p = c0 + k;
            const bool e = stale_select(a.ver_in[p], a.arrived[p], a.t, a.S);
            const double *f = a.fresh[p];
            double *s = a.slots[p];
            s_src[k] = (uint64_t)(e ? f : s);
            s_dst[k] = (!SPLIT && !HELD && e && f != s) ? (uint64_t)s : 0;
        }
        __syncthreads();
        // one batch of up to U ranks: every load, then the stores and the sums
        auto batch = [&](int32_t k0, auto whole) {
            T v[U][VP];
            uint64_t src[U], dst[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t k = whole ? k0 + u : min(k0 + u, nc - 1);
                src[u] = s_src[k];
                if constexpr (!SPLIT && !HELD) dst[u] = s_dst[k];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                src[u] = wave_uniform(src[u]);
                if constexpr (!SPLIT && !HELD) dst[u] = wave_uniform(dst[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (whole || k0 + u < nc) {
#pragma unroll
                    for (int j = 0; j < VP; ++j)
                        v[u][j] = HELD ? __builtin_nontemporal_load(
                                             (GlobalPtr<const T>)((const double *)src[u] + at[j]))
                                       : *(GlobalPtr<const T>)((const double *)src[u] + at[j]);
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (whole || k0 + u < nc) {
                    if constexpr (!SPLIT && !HELD) {
                        if (dst[u]) {
#pragma unroll
                            for (int j = 0; j < VP; ++j)
                                if (in[j]) *(GlobalPtr<T>)((double *)dst[u] + at[j]) = v[u][j];
                        }
                    }
#pragma unroll
                    for (int j = 0; j < VP; ++j)
                        acc[j] = (u == 0 && c0 + k0 == 0) ? v[u][j] : acc[j] + v[u][j];
                }
        };
        int32_t k = 0;
        for (; k + U <= nc; k += U) batch(k, std::true_type{});
        if (k < nc) batch(k, std::false_type{});
    }
#pragma unroll
    for (int j = 0; j < VP; ++j)
        if (in[j]) *(GlobalPtr<T>)(a.result + at[j]) = acc[j];
}

// The same for the longest vectors of many ranks: 1,024 threads own 16,384
// elements (8 pairs per thread), and one rank's loads are in flight at a
// time, its addresses and decision read per rank.  At this size the memory
// sets the pace, and it runs best when all workgroups stream the same rank's
// vector together.  256 x 4M, on one box (the table below is another's):
// 2,806 us; 2,837 with the addresses staged in LDS, 2,832 with the next rank
// loaded before this one's sums, 2,860 to 3,240 in narrower chunks.
constexpr int kWideThreads = 1024;
constexpr int kWidePairs = 8;

__global__ __launch_bounds__(kWideThreads) void k_allreduce_wide(
    int32_t P, int32_t S, int64_t t, const uint8_t *__restrict__ arrived,
    const int32_t *__restrict__ ver_in, int32_t *__restrict__ ver_out,
    int32_t *__restrict__ age_state, uint8_t *__restrict__ eff_state,
    unsigned long long *__restrict__ forced, uint8_t *__restrict__ eff_user,
    int32_t *__restrict__ result_clock, int64_t m, const double *const *__restrict__ fresh,
    double *const *__restrict__ slots, double *__restrict__ result) {
    using T = typename WordVec<2>::t;
    if (blockIdx.x == 0) {
        record_step(P, S, t, arrived, ver_in, ver_out, age_state, eff_state, forced, eff_user,
                    nullptr, result_clock);
        return;
    }
    const int64_t base = (int64_t)(blockIdx.x - 1) * (kWideThreads * kWidePairs * 2);
    int64_t at[kWidePairs];
    bool in[kWidePairs];
    T acc[kWidePairs];
#pragma unroll
    for (int j = 0; j < kWidePairs; ++j) {
        const int64_t e = base + 2 * ((int64_t)threadIdx.x + (int64_t)j * kWideThreads);
        in[j] = e < m;
        at[j] = min(e, m - 2);
        acc[j] = T(0.0);
    }
    for (int32_t p = 0; p < P; ++p) {
        const bool e = stale_select(ver_in[p], arrived[p], t, S);
        const double *fp = fresh[p];
        double *sp = slots[p];
        const bool wr = e && fp != sp;
        const double *src = e ? fp : sp;
        T v[kWidePairs];
#pragma unroll
        for (int j = 0; j < kWidePairs; ++j)
            v[j] = *(GlobalPtr<const T>)(src + at[j]);
        if (wr) {
#pragma unroll
            for (int j = 0; j < kWidePairs; ++j)
                if (in[j]) *(GlobalPtr<T>)(sp + at[j]) = v[j];
        }
#pragma unroll
        for (int j = 0; j < kWidePairs; ++j) acc[j] = (p == 0) ? v[j] : acc[j] + v[j];
    }
#pragma unroll
    for (int j = 0; j < kWidePairs; ++j)
        if (in[j]) *(GlobalPtr<T>)(result + at[j]) = acc[j];
}

// The shape of the launch by the vectors' length.  Wide chunks (8 pairs per
// thread, few ranks in flight) stream each rank's vector in long runs, and pay
// from 16 ranks on as long as the device holds all of their workgroups at
// once, one per CU: from kReduceFill of them to kReduceCus for the first, to
// kReduceCus for the second, and the largest beyond (an 8,192-element chunk
// of 2.5M makes 306, and the 50 second ones cost a fifth).  Shorter vectors
// take chunks of one pair per thread with more ranks in flight instead, and
// the shortest the split form.  Measured on MI355X, us per call, 70 % of the
// ranks arriving and no bound on staleness; "before" is a 1,024-thread
// workgroup of 16,384 elements, one rank in flight, at every length:
//                  pairs  4,096  8,192  wide   before
//   256 x 4,194,304 2,920  2,878  2,822  2,669  2,709
//   256 x 2,500,000 1,756  1,811  2,077  1,717  1,765
//   256 x 1,700,001 1,455  1,255  1,087  1,647  2,149
//   256 x 1,200,000   849    999    795  1,324  1,424
//   256 x   830,000   586    522    699  1,254  1,333
//    16 x 2,500,000   107    113    132    112    116
//    16 x 1,200,000    43     54     50     80     84
//   48 x 150,001     20 pairs, 23 split, 41 at 4,096, 215 before
//   2 x 8,000,001    44 at 256 x 2 pairs x 4 ranks, 45 pairs, 53 before
//   24 x 30,011      4.5 split (the launch itself), 109 before
//   256 x 40,000     31 split or pairs, 660 before
// Where fresh and slots are one array (HELD) a producer has written the slots
// and none is copied.  Non-temporal loads of one pair per thread, eight ranks
// in flight, then pay between the size of the Infinity Cache, which holds what
// was just written, and four times that, where the widest chunk catches up.
// With a producer that writes four fifths of the slots before each call, us
// of both: 24 x 3,520,000 (645 MiB) 271 against 303 in the shapes above and
// 306 before; 32 x 3,520,000 (860 MiB) 359, 387, 390; 64 x 1,700,001 (830
// MiB) 303, 329, 412; but 64 x 4,194,304 (2 GiB) 911, 863, 868; 128 x
// 4,194,304 1,783, 1,669, 1,684; 128 x 150,001 (147 MiB) 57, 47, 277.
// (The factorisation asks for this shape at every length, for what its loads
// leave in the caches: allreduce_streamed.)
constexpr int64_t kReduceCus = 256;
constexpr int64_t kReduceFill = 200;        // workgroups that fill them well enough
constexpr int32_t kReduceManyRanks = 16;    // wide chunks pay from here on
constexpr int64_t kReduceSplitMax = 65536;  // elements: the split form up to here
constexpr int64_t kReduceTinyMax = 4096;    // elements: single elements, 32 ranks in flight
constexpr int32_t kReduceSplitRanks = 1024;
constexpr int64_t kReduceHeldMin = int64_t(1) << 25;  // elements of all ranks: 256 MiB
constexpr int64_t kReduceHeldMax = int64_t(1) << 27;  // 1 GiB
// A launch holds fewer than 2^32 threads; from here on 16 elements each.
constexpr int64_t kReduceFewMax = int64_t(1) << 33;

// The shapes a launch can take; kReduceShapes is indexed by them.
enum ReduceForm {
    kReduceSplitOne,   // split, single elements
    kReduceSplitPair,  // split, pairs
    kReduceOne,        // single elements: vectors shorter than a pair
    kReducePair,
    kReduceFew,        // long vectors of few ranks
    kReduceMiddle,
    kReduceLonger,
    kReduceWide,       // k_allreduce_wide
    kReduceHeld,
    kReduceForms
};
struct ReduceShape {
    int32_t threads, width, vecs;  // elements per access, accesses per thread and rank
    bool split;
};
constexpr ReduceShape kReduceShapes[kReduceForms] = {
    {64, 1, 1, true},  {128, 2, 1, true},  {64, 1, 1, false},
    {128, 2, 1, false}, {256, 2, 2, false}, {256, 2, 8, false},
    {512, 2, 8, false}, {kWideThreads, 2, kWidePairs, false}, {256, 2, 1, false}};

// Elements of each rank's vector a workgroup owns.
constexpr int64_t reduce_chunk(ReduceForm f) {
    return (int64_t)kReduceShapes[f].threads * kReduceShapes[f].width * kReduceShapes[f].vecs;
}

// held: fresh and slots are one array.  A vector shorter than a pair takes a
// shape of single elements whatever its ranks: the lanes of a wider one would
// read and write the element before it.
static ReduceForm reduce_form(int32_t P, int64_t m, bool held) {
    if (m <= kReduceSplitMax && P <= kReduceSplitRanks)
        return m <= kReduceTinyMax ? kReduceSplitOne : kReduceSplitPair;
    if (m < 2) return kReduceOne;
    if (P >= kReduceManyRanks) {
        if (held && m > kReduceHeldMin / P && m <= (kReduceHeldMax - 1) / P) return kReduceHeld;
        if (m > kReduceCus * reduce_chunk(kReduceLonger)) return kReduceWide;
        if (m > kReduceCus * reduce_chunk(kReduceMiddle)) return kReduceLonger;
        if (m >= kReduceFill * reduce_chunk(kReduceMiddle)) return kReduceMiddle;
    } else if (m >= (1 << 19)) {
        return m < kReduceFewMax ? kReduceFew : kReduceWide;
    }
    return kReducePair;
}

// Workgroups of a launch: one that records, those that sum and, split, those
// that copy.
static int64_t reduce_sums(ReduceForm f, int64_t m) {
    const int64_t chunk = reduce_chunk(f);
    return m / chunk + (m % chunk != 0);
}
static int64_t reduce_grid(ReduceForm f, int32_t P, int64_t m) {
    const ReduceShape &s = kReduceShapes[f];
    const int64_t copy = (int64_t)s.threads * s.width * kReduceCopies;
    return 1 + reduce_sums(f, m) + (s.split ? P * ((m + copy - 1) / copy) : 0);
}

template <ReduceForm F, int U, bool HELD = false>
static void launch_reduce(const ReduceArgs &a, unsigned grid, hipStream_t stream) {
    constexpr ReduceShape s = kReduceShapes[F];
    hipLaunchKernelGGL((k_allreduce<s.threads, s.width, s.vecs, U, s.split, HELD>), dim3(grid),
                       dim3(s.threads), 0, stream, a);
}

static ecc_status_t launch_reduce_any(ReduceForm f, ReduceArgs &a, hipStream_t stream) {
    // every lane's access lies in [0, m): at = min(e, m - width) in the kernels
    if (a.m > 0 && a.m < kReduceShapes[f].width) {
        set_error("allreduce: %lld elements in accesses of %d", (long long)a.m,
                  kReduceShapes[f].width);
        return ECC_ERR_STATE;
    }
    const unsigned grid = (unsigned)reduce_grid(f, a.P, a.m);
    a.n_sum = reduce_sums(f, a.m);
    switch (f) {
        case kReduceSplitOne: launch_reduce<kReduceSplitOne, 32>(a, grid, stream); break;
        case kReduceSplitPair: launch_reduce<kReduceSplitPair, 16>(a, grid, stream); break;
        case kReduceOne: launch_reduce<kReduceOne, 8>(a, grid, stream); break;
        case kReducePair: launch_reduce<kReducePair, 8>(a, grid, stream); break;
        case kReduceFew: launch_reduce<kReduceFew, 4>(a, grid, stream); break;
        case kReduceMiddle: launch_reduce<kReduceMiddle, 2>(a, grid, stream); break;
        case kReduceLonger: launch_reduce<kReduceLonger, 1>(a, grid, stream); break;
        case kReduceHeld: launch_reduce<kReduceHeld, 8, true>(a, grid, stream); break;
        default:
            hipLaunchKernelGGL(k_allreduce_wide, dim3(grid), dim3(kWideThreads), 0, stream, a.P,
                               a.S, a.t, a.arrived, a.ver_in, a.ver_out, a.age_state, a.eff_state,
                               a.forced, a.eff_user, a.result_clock, a.m, a.fresh, a.slots,
                               a.result);
    }
    ECC_LAUNCH_CHECK();
    return ECC_OK;
}

static ecc_status_t allreduce(ecc_plan_t plan, int64_t m, const double *const *d_fresh,
                              double *const *d_slots, double *d_result, const uint8_t *d_arrived,
                              uint8_t *d_eff_out, int32_t *d_result_clock, bool streamed) {
    ecc_status_t st = check_plan(plan);
    if (st != ECC_OK) return st;
    ECC_ARG(m >= 0, "m must be >= 0");
    ECC_ARG(d_fresh && d_slots, "d_fresh and d_slots must be device arrays of P pointers");
    ECC_ARG(d_arrived != nullptr, "d_arrived is NULL");
    ECC_ARG(d_result != nullptr || m == 0, "d_result is NULL");
    const int64_t t = plan->clock;
    ReduceArgs a{};
    a.P = plan->P;
    a.S = plan->S;
    a.t = t;
    a.arrived = d_arrived;
    a.ver_in = plan->d_version + (t & 1) * plan->P;
    a.ver_out = plan->d_version + ((t + 1) & 1) * plan->P;
    a.age_state = plan->d_age;
    a.eff_state = plan->d_eff;
    a.forced = plan->d_forced;
    a.eff_user = d_eff_out;
    a.result_clock = d_result_clock;
    a.m = m;
    a.fresh = d_fresh;
    a.slots = d_slots;
    a.result = d_result;
    ReduceForm form = reduce_form(a.P, m, d_fresh == (const double *const *)d_slots);
    // whatever the length: the shapes below 2^32 threads that are not split
    if (streamed && a.P >= kReduceManyRanks && m >= 2 && m < int64_t(1) << 32 &&
        !kReduceShapes[form].split)
        form = kReduceHeld;
    if (reduce_grid(form, a.P, m) > 0x7fffffff) {
        set_error("m too large");
        return ECC_ERR_RANGE;
    }
    {
        TimedLaunch timed(plan, ECC_TIMING_ALLREDUCE);
        st = launch_reduce_any(form, a, plan->stream);
    }
    if (st != ECC_OK) return st;
    plan->clock = t + 1;
    return ECC_OK;
}

ecc_status_t allreduce_streamed(ecc_plan_t plan, int64_t m, double *const *d_slots,
                                double *d_result, const uint8_t *d_arrived, uint8_t *d_eff_out) {
    return allreduce(plan, m, d_slots, d_slots, d_result, d_arrived, d_eff_out, nullptr, true);
}

ecc_status_t launch_assemble(ecc_plan_t plan, const double *const *d_send,
                             const double *d_send_base, double *d_recv,
                             const uint8_t *d_arrived, uint8_t *d_eff_out, int32_t *d_age_out,
                             const int32_t *d_done) {
    const int64_t t = plan->clock;
    const int32_t *ver_in = plan->d_version + (t & 1) * plan->P;
    int32_t *ver_out = plan->d_version + ((t + 1) & 1) * plan->P;
    const int64_t grid = 1 + plan->n_tiles;
    if (grid > 0x7fffffff) {
        set_error("too many assembly tiles");
        return ECC_ERR_RANGE;
    }
    TimedLaunch timed(plan, ECC_TIMING_ASSEMBLE);
    hipLaunchKernelGGL(k_assemble, dim3((unsigned)grid), dim3(kAssembleThreads), 0, plan->stream,
                       plan->P, plan->S, t, d_arrived, ver_in, ver_out, plan->d_age, plan->d_eff,
                       plan->d_forced, d_eff_out, d_age_out, plan->d_tiles, plan->d_displs,
                       d_send, d_send_base, d_recv, d_done);
    ECC_LAUNCH_CHECK();
    plan->clock = t + 1;
    return ECC_OK;
}

}  // namespace ecc

using namespace ecc;

extern "C" {

ecc_status_t ecc_allgatherv_assemble(ecc_plan_t plan, const double *const *d_send,
                                     double *d_recv, const uint8_t *d_arrived,
                                     uint8_t *d_eff_out, int32_t *d_age_out) {
    clear_error();
    ecc_status_t st = check_plan(plan);
    if (st != ECC_OK) return st;
    if (!plan->has_layout) {
        set_error("plan was created without counts/displs");
        return ECC_ERR_STATE;
    }
    ECC_ARG(d_send != nullptr, "d_send is NULL");
    ECC_ARG(d_arrived != nullptr, "d_arrived is NULL");
    ECC_ARG(d_recv != nullptr || plan->extent == 0, "d_recv is NULL");
    return launch_assemble(plan, d_send, nullptr, d_recv, d_arrived, d_eff_out, d_age_out,
                           nullptr);
}

ecc_status_t ecc_allgatherv_assemble_packed(ecc_plan_t plan, const double *d_send_base,
                                            double *d_recv, const uint8_t *d_arrived,
                                            uint8_t *d_eff_out, int32_t *d_age_out) {
    clear_error();
    ecc_status_t st = check_plan(plan);
    if (st != ECC_OK) return st;
    if (!plan->has_layout) {
        set_error("plan was created without counts/displs");
        return ECC_ERR_STATE;
    }
    ECC_ARG(d_send_base != nullptr || plan->extent == 0, "d_send_base is NULL");
    ECC_ARG(d_arrived != nullptr, "d_arrived is NULL");
    ECC_ARG(d_recv != nullptr || plan->extent == 0, "d_recv is NULL");
    ECC_ARG(d_send_base != d_recv || plan->extent == 0, "d_send_base must not alias d_recv");
    return launch_assemble(plan, nullptr, d_send_base, d_recv, d_arrived, d_eff_out, d_age_out,
                           nullptr);
}

ecc_status_t ecc_allreduce_shape(int32_t P, int64_t m, int32_t held, int64_t *workgroups,
                                 int32_t *threads, int32_t *width) {
    clear_error();
    ECC_ARG(P >= 1 && m >= 0, "P must be >= 1 and m >= 0");
    ECC_ARG(workgroups && threads && width, "NULL output");
    const ReduceForm f = reduce_form(P, m, held != 0);
    *workgroups = reduce_grid(f, P, m);
    *threads = kReduceShapes[f].threads;
    *width = kReduceShapes[f].width;
    return ECC_OK;
}

ecc_status_t ecc_allreduce_partial(ecc_plan_t plan, int64_t m, const double *const *d_fresh,
                                   double *const *d_slots, double *d_result,
                                   const uint8_t *d_arrived, uint8_t *d_eff_out,
                                   int32_t *d_result_clock) {
    clear_error();
    return allreduce(plan, m, d_fresh, d_slots, d_result, d_arrived, d_eff_out, d_result_clock,
                     false);
}

}  // extern "C"
