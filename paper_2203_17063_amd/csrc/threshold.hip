// Eventually consistent Broadcast and Reduce with a threshold (Section III-B,
// with the threshold/status parameters of Section III), and the partial
// allreduce that drops the contributions that did not arrive.
//
// Binomial spanning tree (BST) over P processes numbered relative to the
// root: the children of q are q + 2^i for every i above q's highest set bit
// with q + 2^i < P, so stage s involves min(2^s, P) processes.
//  - Broadcast delivers the first ceil(theta * m) elements of the root's
//    vector to every other process: on one GPU the tree's forwarding
//    reduces to prefix copies (every receiver gets the root's data); each
//    tile of the prefix is read once and written P - 1 times.
//  - Reduce sums either the first ceil(theta * m) elements of every process
//    or the full vectors of the processes of the first stages of the tree
//    (at least ceil(theta * P) of them).  The order is the tree's: a parent
//    adds its children's partial sums leaves first, which is, stage by stage
//    from the last one, q += partial(q + 2^s) for every q < 2^s.  A thread
//    carries one element of every involved process in registers; beyond 32
//    processes it sums them in the same tree as a pairwise sum (below).
//  - The dropping allreduce sums, in rank order from +0.0, the contributions
//    of the ranks that arrived in this step.
// All sums are fp64 without contraction, in the order stated, so results
// are bitwise reproducible.
#include <algorithm>
#include <cmath>

#include "ecc_common.h"

namespace ecc {

constexpr int kThrThreads = 256;
constexpr int kThrMaxStages = 5;  // Reduce: at most 32 processes in registers
constexpr int kThrMaxStagesBig = 12;  // Reduce beyond 32 processes: up to 4096

// Broadcast: a workgroup loads a tile of the prefix (PAIRS pairs per thread)
// from the root's vector into registers once and stores it into `per`
// processes' buffers (blockIdx.y picks which).  Write-bound: 8 k P bytes.
// The last pair of an odd prefix is moved back by one element (two lanes
// then store the same value).
template <int PAIRS>
__global__ __launch_bounds__(kThrThreads) void k_bcast_prefix(int32_t P, int32_t root, int64_t k,
                                                              int32_t per,
                                                              const double *__restrict__ src,
                                                              double *const *__restrict__ dst) {
    using T = typename WordVec<2>::t;
    const int32_t p0 = (int32_t)blockIdx.y * per;
    const int32_t p1 = (int32_t)min((int64_t)P, (int64_t)p0 + per);
    if (k == 1) {
        if (threadIdx.x == 0)
            for (int32_t p = p0; p < p1; ++p)
                if (p != root) dst[p][0] = src[0];
        return;
    }
    const int64_t t0 = (int64_t)blockIdx.x * (2 * PAIRS * kThrThreads);
    T v[PAIRS];
    int64_t at[PAIRS];
    bool in[PAIRS];
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) {
        const int64_t e = t0 + 2 * ((int64_t)threadIdx.x + (int64_t)u * kThrThreads);
        in[u] = e < k;
        at[u] = min(e, k - 2);
        v[u] = *(GlobalPtr<const T>)(src + at[u]);
    }
    const bool whole = t0 + 2 * PAIRS * kThrThreads <= k;
    for (int32_t p = p0; p < p1; ++p) {
        if (p == root) continue;
        double *d = dst[p];
        if (whole) {
#pragma unroll
            for (int u = 0; u < PAIRS; ++u) *(GlobalPtr<T>)(d + at[u]) = v[u];
        } else {
#pragma unroll
            for (int u = 0; u < PAIRS; ++u)
                if (in[u]) *(GlobalPtr<T>)(d + at[u]) = v[u];
        }
    }
}

// The same in 4,096-element tiles written to every process, for prefixes
// whose copies leave the Infinity Cache but which make few such tiles: rows
// that are not 16-byte aligned are stored by 8 bytes there, and the row end is
// tested per pair.
constexpr int kBcastPairs = 8;
constexpr int kBcastTile = 2 * kBcastPairs * kThrThreads;

__global__ __launch_bounds__(kThrThreads) void k_bcast_middle(int32_t P, int32_t root, int64_t k,
                                                              const double *__restrict__ src,
                                                              double *const *__restrict__ dst) {
    const int64_t t0 = (int64_t)blockIdx.x * kBcastTile;
    const bool src16 = ((uintptr_t)src & 15) == 0;
    double2 v[kBcastPairs];
#pragma unroll
    for (int u = 0; u < kBcastPairs; ++u) {
        const int64_t e = t0 + 2 * ((int64_t)threadIdx.x + (int64_t)u * kThrThreads);
        if (e + 1 < k) {
            if (src16) v[u] = *reinterpret_cast<const double2 *>(src + e);
            else v[u] = make_double2(src[e], src[e + 1]);
        } else {
            v[u] = make_double2(e < k ? src[e] : 0.0, 0.0);
        }
    }
    for (int32_t p = 0; p < P; ++p) {
        if (p == root) continue;
        double *__restrict__ d = dst[p];
        const bool d16 = ((uintptr_t)d & 15) == 0;
#pragma unroll
        for (int u = 0; u < kBcastPairs; ++u) {
            const int64_t e = t0 + 2 * ((int64_t)threadIdx.x + (int64_t)u * kThrThreads);
            if (e + 1 < k) {
                if (d16) *reinterpret_cast<double2 *>(d + e) = v[u];
                else {
                    d[e] = v[u].x;
                    d[e + 1] = v[u].y;
                }
            } else if (e < k) {
                d[e] = v[u].x;
            }
        }
    }
}

// Long prefixes take 4,096-element tiles written to every process; short ones
// 512-element tiles, their processes split over enough workgroups (at least
// kBcastRows processes each) to fill the device; and between kBcastMiddle and
// kBcastLong, where the copies exceed kBcastCached, k_bcast_middle. Measured
// on MI355X, us in 512-element tiles / k_bcast_middle / 4,096-element tiles:
//   16 x   300,000   7.4 /  12.4 /   9.0    200 x   300,000   92 / 114 /  95
//   32 x 1,000,001  38.0 /  38.2 /  38.2    200 x   500,001  195 / 163 / 159
//   64 x 1,000,001   116 /    99 /   112    200 x   524,288  171 / 126 / 146
//   48 x 1,900,001   170 /   147 /   146    200 x 1,000,001  411 / 318 / 349
//   64 x 2,300,001   301 /   257 /   244     16 x 3,500,000 84.9 / 86.2 / 85.9
// 48 x 22,509: 4.1 us in 512-element tiles, 28 in 4,096-element ones; 32 x
// 4.2M: 172-194 us (5.5-6.2 TB/s; what the kernel before it left to be
// written back counts here).
constexpr int64_t kBcastMiddle = 400000;          // elements
constexpr int64_t kBcastLong = int64_t(1) << 21;  // elements: 512 workgroups of long tiles
constexpr int64_t kBcastCached = int64_t(1) << 25;  // elements of all copies: 256 MiB
constexpr int32_t kBcastRows = 4;
constexpr int64_t kBcastFill = 1024;

// Reduce over relative ranks 0 .. n-1 (n <= 2^S) of the first k elements.
// Every contribution is read once: non-temporal loads (measured on MI355X,
// 32 processes x 4.2M elements: 190 us against 261 us with ordinary loads
// and a grid capped at 8 workgroups per CU), and one workgroup per 256
// elements.
template <int S>
__global__ __launch_bounds__(kThrThreads) void k_reduce_bst(int32_t P, int32_t root, int32_t n,
                                                            int64_t k,
                                                            const double *const *__restrict__ src,
                                                            double *__restrict__ result) {
    static_assert(S >= 0 && S <= kThrMaxStages, "the register fold holds at most 32 processes");
    constexpr int N = 1 << S;
    const int64_t stride = (int64_t)gridDim.x * kThrThreads;
    for (int64_t j = (int64_t)blockIdx.x * kThrThreads + threadIdx.x; j < k; j += stride) {
        double part[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if (q < n) {
                const int32_t p = (q + root) % P;
                part[q] = __builtin_nontemporal_load(src[p] + j);
            }
        }
#pragma unroll
        for (int s = S - 1; s >= 0; --s) {
#pragma unroll
            for (int q = 0; q < (1 << s); ++q)
                if (q + (1 << s) < n) part[q] = part[q] + part[q + (1 << s)];
        }
        result[j] = part[0];
    }
}

// More than 32 processes (measured on MI355X, 64 x 32 MB: 362 against 369
// us with all 64 in registers, 169 VGPRs; 32 x 64 MB: 377 against 360 us,
// so the register fold stays up to 32).  Stage by stage from the last,
// q += partial(q + 2^s) builds a binary tree whose leaves, read left to
// right, are the relative ranks in the bit-reversed order of D =
// ceil(log2 n) bits: the two children of a node combined at stage s are
// its halves, the lower rank on the left and added first.  A rank at or beyond n is absent; as
// absence grows with the rank, a node whose left child is absent has an
// absent right child too, and a node with an absent right child is its
// left child.  So the reduction is a pairwise sum over that order, and a
// thread computes it for its element with a stack of one node per level:
// the 8 leaves of each group of 8 consecutive positions are loaded
// together and added into one node, which is merged into the stack as a
// binary counter over the group index.
constexpr int kBrev3[8] = {0, 4, 2, 6, 1, 5, 3, 7};

template <int D>
__global__ __launch_bounds__(kThrThreads) void k_reduce_bst_big(
    int32_t P, int32_t root, int32_t n, int64_t k, const double *const *__restrict__ src,
    double *__restrict__ result) {
    constexpr int H = D - 3;  // levels above a group of 8 leaves
    static_assert(H >= 1 && D <= kThrMaxStagesBig, "between 9 and 4,096 processes");
    const int64_t stride = (int64_t)gridDim.x * kThrThreads;
    for (int64_t j = (int64_t)blockIdx.x * kThrThreads + threadIdx.x; j < k; j += stride) {
        double st[H];
        bool sv[H];
#pragma unroll
        for (int l = 0; l < H; ++l) {
            st[l] = 0.0;
            sv[l] = false;
        }
        double node = 0.0;
        for (int32_t b = 0; b < (1 << H); ++b) {
            // leaf u of group b sits at position 8 b + u: relative rank
            // bitrev3(u) 2^H + bitrev_H(b)
            const int32_t hb = (int32_t)(__brev((uint32_t)b) >> (32 - H));
            double v[8];
            bool e[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int32_t q = (kBrev3[u] << H) | hb;
                e[u] = q < n;
                int32_t p = (e[u] ? q : 0) + root;  // (an absent leaf names no process)
                if (p >= P) p -= P;
                v[u] = e[u] ? __builtin_nontemporal_load(src[p] + j) : 0.0;
            }
            // the group's node: pairs, then quads, then the eight
#pragma unroll
            for (int w = 1; w < 8; w *= 2) {
#pragma unroll
                for (int u = 0; u < 8; u += 2 * w)
                    if (e[u + w]) v[u] = v[u] + v[u + w];
            }
            node = v[0];
            bool nv = e[0];
            // merge as a binary counter: level l holds the left sibling while
            // bit l of b is 1
            bool carry = true;
#pragma unroll
            for (int l = 0; l < H; ++l) {
                if (carry) {
                    if ((b >> l) & 1) {
                        if (sv[l] && nv) node = st[l] + node;
                        else if (sv[l]) node = st[l];
                        nv = sv[l];
                    } else {
                        st[l] = node;
                        sv[l] = nv;
                        carry = false;
                    }
                }
            }
        }
        // the last group (b = 2^H - 1) carried through every level: the root
        result[j] = node;
    }
}

// Dropping partial allreduce: result = +0.0 + the contributions of the ranks
// that arrived, in rank order.  Read-bound: 8 m (arrived + 1) bytes.  Each
// workgroup lists the arrived ranks' addresses in LDS (kDropStage ranks at a
// time, in rank order), so that the loads of U ranks go out together without
// a test or a pointer chase between them; each contribution is read once by
// one lane per element of a grid without a loop, non-temporally where the
// contributions of all ranks exceed the Infinity Cache (us per call alone / in
// a pass with a Broadcast and a Reduce, ordinary and non-temporal loads: 16 x
// 2M, 244 MiB, 32.6 / 81.1 and 38.6 / 83.7; 12 x 2M 26.4 / 60.4 and 31.6 /
// 65.9; 16 x 3M, 366 MiB, 50.1 / 136.6 and 55.5 / 120.1).
// Measured on MI355X, 26 of 32 ranks x 8.4M: 332 us (5.5 TB/s), against 451
// us for k_allreduce_drop_few; pairs per lane 337 to 371 us; 38 of 48 x
// 30,011: 5.0 against 12.7 us.
constexpr int kDropStage = 256;

constexpr int kDropU = 16;  // ranks whose loads are in flight together
constexpr int64_t kDropLaunch = int64_t(1) << 31;  // elements of one launch

template <bool NT>
__device__ __forceinline__ double drop_load(uint64_t src, int64_t at) {
    const GlobalPtr<const double> p = (GlobalPtr<const double>)((const double *)src + at);
    return NT ? __builtin_nontemporal_load(p) : *p;
}

template <bool NT>
__global__ __launch_bounds__(kThrThreads) void k_allreduce_drop(int32_t P, int64_t e0,
                                                        int64_t m,
                                                        const double *const *__restrict__ fresh,
                                                        const uint8_t *__restrict__ arrived,
                                                        double *__restrict__ result,
                                                        int32_t *__restrict__ count) {
    __shared__ uint64_t s_src[kDropStage];
    __shared__ int32_t s_wave[kDropStage / 64];
    const int tid = threadIdx.x;
    const int64_t e = e0 + (int64_t)blockIdx.x * kThrThreads + tid;
    const int64_t at = max<int64_t>(0, min(e, m - 1));
    double acc = 0.0;
    int32_t total = 0;
    for (int64_t c0 = 0; c0 < P; c0 += kDropStage) {
        if (c0) __syncthreads();
        // the 64-rank groups of this stage, one wave at a time each
        for (int32_t g = tid >> 6; g < kDropStage / 64; g += kThrThreads / 64) {
            const int64_t p = c0 + g * 64 + (tid & 63);
            const uint64_t on = __ballot(p < P && arrived[p] != 0);
            if ((tid & 63) == 0) s_wave[g] = __popcll(on);
        }
        __syncthreads();
        for (int32_t g = tid >> 6; g < kDropStage / 64; g += kThrThreads / 64) {
            const int64_t p = c0 + g * 64 + (tid & 63);
            const bool here = p < P && arrived[p] != 0;
            const uint64_t on = __ballot(here);
            int32_t at0 = 0;
            for (int32_t h = 0; h < g; ++h) at0 += s_wave[h];
            if (here && m > 0)
                s_src[at0 + __popcll(on & ((1ull << (tid & 63)) - 1))] = (uint64_t)fresh[p];
        }
        int32_t nc = 0;
#pragma unroll
        for (int h = 0; h < kDropStage / 64; ++h) nc += s_wave[h];
        total += nc;
        __syncthreads();
        if (m == 0) continue;
        int32_t k = 0;
        for (; k + kDropU <= nc; k += kDropU) {
            uint64_t src[kDropU];
            double v[kDropU];
#pragma unroll
            for (int u = 0; u < kDropU; ++u) src[u] = wave_uniform(s_src[k + u]);
#pragma unroll
            for (int u = 0; u < kDropU; ++u)
                v[u] = drop_load<NT>(src[u], at);
#pragma unroll
            for (int u = 0; u < kDropU; ++u) acc = acc + v[u];
        }
        if (k < nc) {
            uint64_t src[kDropU];
            double v[kDropU];
#pragma unroll
            for (int u = 0; u < kDropU; ++u) src[u] = wave_uniform(s_src[min(k + u, nc - 1)]);
#pragma unroll
            for (int u = 0; u < kDropU; ++u)
                if (k + u < nc) v[u] = drop_load<NT>(src[u], at);
#pragma unroll
            for (int u = 0; u < kDropU; ++u)
                if (k + u < nc) acc = acc + v[u];
        }
    }
    if (e < m) result[e] = acc;
    if (count && blockIdx.x == 0 && tid == 0) *count = total;
}

constexpr int64_t kDropCached = int64_t(1) << 25;  // elements of all ranks: 256 MiB
bool drop_cached(int32_t P, int64_t m) { return m <= kDropCached / P; }

// The same for few ranks, whose list costs a workgroup more than its 256
// elements' sums: at most kDropFewGrid workgroups walk the vector, a test
// before each rank's load, eight loads in flight.  Measured on MI355X, us per
// call alone / in a pass with a Broadcast and a Reduce of the same vectors,
// with the walk, and with the list: 1 of 2 x 6,000,001 18.0 / 44.5 and 52.9 /
// 77.2; 3 of 5 x 3M 19.5 / 44.0 and 32.3 / 55.6; 5 of 8 x 3M 26.3 / 63.0 and
// 36.0 / 70.3, x 8M 92 / 195 and 88 / 180; 6 of 9 x 4,000,001 41 / 116 and 51 /
// 101; 7 of 10 x 700,001 11.1 / 28.0 and 10.3 / 26.6.
constexpr int kDropFewU = 8;
constexpr int64_t kDropFewGrid = 2048;  // eight workgroups per CU
constexpr int32_t kDropFewRanks = 7;    // the walk at every length
constexpr int32_t kDropFewRanksHot = 9;  // and while the contributions fit the cache

bool drop_few(int32_t P, int64_t m) {
    return P <= kDropFewRanks || (P <= kDropFewRanksHot && drop_cached(P, m));
}

__global__ __launch_bounds__(kThrThreads) void k_allreduce_drop_few(
    int32_t P, int64_t m, const double *const *__restrict__ fresh,
    const uint8_t *__restrict__ arrived, double *__restrict__ result,
    int32_t *__restrict__ count) {
    if (count && blockIdx.x == 0 && threadIdx.x == 0) {
        int32_t c = 0;
        for (int32_t p = 0; p < P; ++p) c += arrived[p] != 0;
        *count = c;
    }
    const int64_t stride = (int64_t)gridDim.x * kThrThreads;
    for (int64_t j = (int64_t)blockIdx.x * kThrThreads + threadIdx.x; j < m; j += stride) {
        double acc = 0.0;
        for (int32_t p0 = 0; p0 < P; p0 += kDropFewU) {
            bool on[kDropFewU];
            double v[kDropFewU];
#pragma unroll
            for (int u = 0; u < kDropFewU; ++u) {
                const int32_t p = p0 + u;
                on[u] = p < P && arrived[p] != 0;
                v[u] = on[u] ? fresh[p][j] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kDropFewU; ++u)
                if (on[u]) acc = acc + v[u];
        }
        result[j] = acc;
    }
}

int64_t thr_prefix(double theta, int64_t m) {
    const double x = std::ceil(theta * (double)m);
    return std::min<int64_t>(m, (int64_t)x);
}

int32_t thr_involved(double theta, int32_t P) {
    const int64_t need = std::max<int64_t>(1, (int64_t)std::ceil(theta * (double)P));
    int64_t n = 1;
    while (n < need) n *= 2;
    return (int32_t)std::min<int64_t>(n, P);
}

int32_t thr_grid_once(int64_t elems) {
    const int64_t need = std::max<int64_t>(1, (elems + kThrThreads - 1) / kThrThreads);
    return (int32_t)std::min<int64_t>(need, 0x7fffffff);
}

}  // namespace ecc

using namespace ecc;

extern "C" {

ecc_status_t ecc_bcast_threshold(int32_t P, int32_t root, int64_t m, double theta,
                                 const double *d_src, double *const *d_dst, int64_t *h_count,
                                 void *hip_stream) {
    clear_error();
    ECC_ARG(P >= 1, "P must be >= 1");
    ECC_ARG(root >= 0 && root < P, "root %d outside [0, P)", root);
    ECC_ARG(m >= 0, "m must be >= 0");
    ECC_ARG(theta >= 0.0 && theta <= 1.0, "theta must lie in [0, 1]");
    const int64_t k = thr_prefix(theta, m);
    if (h_count) *h_count = k;
    if (k == 0 || P == 1) return ECC_OK;
    ECC_ARG(d_src != nullptr && d_dst != nullptr, "NULL source or destination array");
    const bool longer = k >= kBcastLong;
    const bool middle = !longer && k >= kBcastMiddle && k > kBcastCached / P;
    const int64_t tile = longer || middle ? kBcastTile : 2 * kThrThreads;
    const int64_t tiles = (k + tile - 1) / tile;
    ECC_ARG(tiles < 0x7fffffff, "too many tiles");
    const int64_t groups = longer || middle ? 1
                                            : std::max<int64_t>(1, std::min<int64_t>(kBcastFill / tiles,
                                                                   ((int64_t)P + kBcastRows - 1) / kBcastRows));
    const int32_t per = (int32_t)((P + groups - 1) / groups);
    const dim3 grid((unsigned)tiles, (unsigned)(((int64_t)P + per - 1) / per));
    hipStream_t st = (hipStream_t)hip_stream;
    if (middle)
        hipLaunchKernelGGL(k_bcast_middle, grid, dim3(kThrThreads), 0, st, P, root, k, d_src,
                           d_dst);
    else if (longer)
        hipLaunchKernelGGL(k_bcast_prefix<kBcastPairs>, grid, dim3(kThrThreads), 0, st, P, root, k, per,
                           d_src, d_dst);
    else
        hipLaunchKernelGGL(k_bcast_prefix<1>, grid, dim3(kThrThreads), 0, st, P, root, k, per,
                           d_src, d_dst);
    ECC_LAUNCH_CHECK();
    return ECC_OK;
}

ecc_status_t ecc_reduce_threshold(int32_t P, int32_t root, int64_t m, double theta, int32_t mode,
                                  const double *const *d_src, double *d_result,
                                  int64_t *h_elements, int32_t *h_processes, void *hip_stream) {
    clear_error();
    ECC_ARG(P >= 1 && P <= (1 << kThrMaxStagesBig), "P = %d must lie in [1, %d]", P,
            1 << kThrMaxStagesBig);
    ECC_ARG(root >= 0 && root < P, "root %d outside [0, P)", root);
    ECC_ARG(m >= 0, "m must be >= 0");
    ECC_ARG(mode == ECC_THRESHOLD_DATA || mode == ECC_THRESHOLD_PROCS, "unknown mode %d", mode);
    int64_t k;
    int32_t n;
    if (mode == ECC_THRESHOLD_DATA) {
        ECC_ARG(theta >= 0.0 && theta <= 1.0, "theta must lie in [0, 1]");
        k = thr_prefix(theta, m);
        n = P;
    } else {
        ECC_ARG(theta > 0.0 && theta <= 1.0, "theta must lie in (0, 1]");
        k = m;
        n = thr_involved(theta, P);
    }
    if (h_elements) *h_elements = k;
    if (h_processes) *h_processes = n;
    if (k == 0) return ECC_OK;
    ECC_ARG(d_src != nullptr && d_result != nullptr, "NULL source array or result");
    int S = 0;
    while ((1 << S) < n) ++S;
    const dim3 grid(thr_grid_once(k)), block(kThrThreads);
    hipStream_t st = (hipStream_t)hip_stream;
    switch (S) {
        case 0: hipLaunchKernelGGL(k_reduce_bst<0>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 1: hipLaunchKernelGGL(k_reduce_bst<1>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 2: hipLaunchKernelGGL(k_reduce_bst<2>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 3: hipLaunchKernelGGL(k_reduce_bst<3>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 4: hipLaunchKernelGGL(k_reduce_bst<4>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 5: hipLaunchKernelGGL(k_reduce_bst<5>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 6: hipLaunchKernelGGL(k_reduce_bst_big<6>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 7: hipLaunchKernelGGL(k_reduce_bst_big<7>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 8: hipLaunchKernelGGL(k_reduce_bst_big<8>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 9: hipLaunchKernelGGL(k_reduce_bst_big<9>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 10: hipLaunchKernelGGL(k_reduce_bst_big<10>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        case 11: hipLaunchKernelGGL(k_reduce_bst_big<11>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
        default: hipLaunchKernelGGL(k_reduce_bst_big<12>, grid, block, 0, st, P, root, n, k, d_src, d_result); break;
    }
    ECC_LAUNCH_CHECK();
    return ECC_OK;
}

ecc_status_t ecc_allreduce_drop(int32_t P, int64_t m, const double *const *d_fresh,
                                const uint8_t *d_arrived, double *d_result, int32_t *d_count,
                                void *hip_stream) {
    clear_error();
    ECC_ARG(P >= 1, "P must be >= 1");
    ECC_ARG(m >= 0, "m must be >= 0");
    ECC_ARG(d_arrived != nullptr, "d_arrived is NULL");
    ECC_ARG(m == 0 || (d_fresh && d_result), "NULL contribution array or result");
    if (m == 0 && !d_count) return ECC_OK;
    if (drop_few(P, m)) {
        const int64_t grid = std::min(kDropFewGrid, (int64_t)thr_grid_once(m));
        hipLaunchKernelGGL(k_allreduce_drop_few, dim3((unsigned)grid), dim3(kThrThreads), 0,
                           (hipStream_t)hip_stream, P, m, d_fresh, d_arrived, d_result, d_count);
        ECC_LAUNCH_CHECK();
        return ECC_OK;
    }
    // (a launch holds fewer than 2^32 threads)
    int64_t e0 = 0;
    do {
        const int64_t grid = std::max<int64_t>(
            1, (std::min(m - e0, kDropLaunch) + kThrThreads - 1) / kThrThreads);
        hipLaunchKernelGGL(drop_cached(P, m) ? k_allreduce_drop<false> : k_allreduce_drop<true>,
                           dim3((unsigned)grid), dim3(kThrThreads), 0, (hipStream_t)hip_stream, P,
                           e0, m, d_fresh, d_arrived, d_result, e0 == 0 ? d_count : nullptr);
        ECC_LAUNCH_CHECK();
        e0 += kDropLaunch;
    } while (e0 < m);
    return ECC_OK;
}

}  // extern "C"
