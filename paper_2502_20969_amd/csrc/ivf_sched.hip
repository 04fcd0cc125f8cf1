// Prefetching scheduler (TeleRAG, arxiv 2502.20969, Sec. 4.2 "Scheduling optimization for
// prefetching"): the queries of a global batch are grouped into micro-batches by a greedy search on
// squared L2 distance, so that the queries of one micro-batch want largely the same clusters.
// Three kernels: all pairwise distances, every query's others in order of distance, then the greedy pick.
#include "ivf_device.h"
#include <algorithm>

namespace ivf {
using namespace dev;

// D[i][j] = sum over t of (q[i][t] - q[j][t])^2 in fp64, added term by term in index order: the
// greedy pick compares these values, and a fixed order of operations makes its decisions
// reproducible down to exact ties.  (x - y)^2 and (y - x)^2 are
// the same value, so only the tiles on and above the diagonal are computed and stored twice.
// One workgroup per 16 x 16 tile of pairs; slabs of 64 components go through LDS, widened to
// double on the way in (once per tile instead of once per pair), the next slab requested while one
// is worked on.  Bound by LDS latency and fp64 issue: 55 -> 35 us for 512 queries x 768 (without
// the reads ahead inside a slab 54 us).
constexpr int kPairTile = 16, kPairSlab = 64;

__global__ __launch_bounds__(256) void pair_dist_kernel(const float* q, int B, int d, double* D) {
    __shared__ __align__(16) double sa[kPairTile][kPairSlab + 2];
    __shared__ __align__(16) double sb[kPairTile][kPairSlab + 2];
    if (blockIdx.x < blockIdx.y) return;                   // below the diagonal: stored by the mirrored tile
    const int tid = threadIdx.x;
    const int ti = tid / kPairTile, tj = tid % kPairTile;
    const int i0 = blockIdx.y * kPairTile, j0 = blockIdx.x * kPairTile;
    double acc = 0.0;
    float va[4], vb[4];                                    // the next slab: on its way while one is worked on
    auto request = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = tid + u * 256, r = e / kPairSlab, t = e % kPairSlab;
            const bool in_k = k0 + t < d;
            va[u] = (in_k && i0 + r < B) ? q[(size_t)(i0 + r) * d + k0 + t] : 0.f;
            vb[u] = (in_k && j0 + r < B) ? q[(size_t)(j0 + r) * d + k0 + t] : 0.f;
        }
    };
    request(0);
    for (int k0 = 0; k0 < d; k0 += kPairSlab) {
        __syncthreads();                                   // the previous slab has been read
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = tid + u * 256;
            sa[e / kPairSlab][e % kPairSlab] = (double)va[u];
            sb[e / kPairSlab][e % kPairSlab] = (double)vb[u];
        }
        __syncthreads();
        if (k0 + kPairSlab < d) request(k0 + kPairSlab);
        const int kn = min(kPairSlab, d - k0);
        if (kn == kPairSlab) {
            // eight terms are read while the eight before them are added: with two wavefronts per
            // SIMD nothing else hides the LDS latency
            double2 xa[2][4], xb[2][4];
            auto read8 = [&](int t0, double2 (&x)[4], double2 (&y)[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) { x[u] = *(const double2*)&sa[ti][t0 + 2 * u]; y[u] = *(const double2*)&sb[tj][t0 + 2 * u]; }
            };
            read8(0, xa[0], xb[0]);
#pragma unroll
            for (int c = 0; c < kPairSlab / 8; ++c) {
                if (c + 1 < kPairSlab / 8) read8(c * 8 + 8, xa[(c + 1) & 1], xb[(c + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double d0 = xa[c & 1][u].x - xb[c & 1][u].x, d1 = xa[c & 1][u].y - xb[c & 1][u].y;
                    acc = __dadd_rn(acc, __dmul_rn(d0, d0));
                    acc = __dadd_rn(acc, __dmul_rn(d1, d1));
                }
            }
        } else {
            for (int t = 0; t < kn; ++t) {
                const double df = sa[ti][t] - sb[tj][t];
                acc = __dadd_rn(acc, __dmul_rn(df, df));
            }
        }
    }
    if (i0 + ti < B && j0 + tj < B) D[(size_t)(i0 + ti) * B + j0 + tj] = acc;
    if (blockIdx.x == blockIdx.y) return;
    __syncthreads();
    sa[tj][ti] = acc;
    __syncthreads();
    if (j0 + ti < B && i0 + tj < B) D[(size_t)(j0 + ti) * B + i0 + tj] = sa[ti][tj];
}

constexpr int kNearStep = 512;

// near[i] = all queries in the order in which seed i would take them: ascending (distance, index).
// A distance is non-negative, so its bit pattern orders like its value.  One workgroup per query,
// a bitonic sort of (bits, index) pairs in LDS over the next power of two.  The sorts of all rows
// run side by side, so that the greedy pick, which is sequential, only walks lists.
// A row of near is a multiple of kNearStep entries, so that one wavefront reads kNearStep of them
// with one 16-byte load per lane; lane l gets entries l, l + 64, ... of them in that order, and entries
// past B are 0xFFFF.
__global__ void sort_near_kernel(const double* D, int B, uint32_t pad, int stride, uint16_t* near) {
    extern __shared__ __align__(16) unsigned char s_raw[];
    unsigned long long* key = (unsigned long long*)s_raw;
    uint16_t* idx = (uint16_t*)(key + pad);
    const uint32_t tid = threadIdx.x, nt = blockDim.x;
    const int row = blockIdx.x;
    for (uint32_t i = tid; i < pad; i += nt) {
        key[i] = (int)i < B ? (unsigned long long)__double_as_longlong(D[(size_t)row * B + i]) : ~0ull;
        idx[i] = (int)i < B ? (uint16_t)i : (uint16_t)0xFFFFu;
    }
    __syncthreads();
    for (uint32_t size = 2; size <= pad; size <<= 1) {
        for (uint32_t st = size >> 1; st > 0; st >>= 1) {
            for (uint32_t p = tid; p < pad / 2; p += nt) {
                const uint32_t i = 2 * p - (p & (st - 1)), j = i + st;      // i has bit st clear
                const unsigned long long ki = key[i], kj = key[j];
                const uint16_t xi = idx[i], xj = idx[j];
                const bool i_after_j = ki > kj || (ki == kj && xi > xj);
                if (i_after_j == ((i & size) == 0)) {
                    key[i] = kj; key[j] = ki;
                    idx[i] = xj; idx[j] = xi;
                }
            }
            __syncthreads();
        }
    }
    for (int o = (int)tid; o < stride; o += (int)nt) {
        const int i = o / kNearStep * kNearStep + o % 8 * 64 + o % kNearStep / 8;
        near[(size_t)row * stride + o] = i < (int)pad ? idx[i] : (uint16_t)0xFFFFu;
    }
}

// Greedy pick by one wavefront.  While queries remain: the remaining query of lowest index seeds a
// micro-batch; the m - 1 remaining queries nearest to it follow, nearest first, equal distances by
// lower index: the first m - 1 entries of its sorted list that are not taken.  Whether they are is read
// for 512 entries at once, then 64 at a time are numbered by one ballot until enough are found.  A
// chain of LDS reads per micro-batch bounds it: the list of the query that will most likely seed next is
// requested one micro-batch ahead, and the order is kept in LDS until the end, because a load waits for
// the stores before it, and stores to host memory take longer than a micro-batch.  (Picking one query at a
// time with a workgroup-wide minimum: 892 us for 512 queries in groups of 8; sorted lists, with the order
// stored as it was found and the places counted by a prefix over the lanes: 67; this: 38.)
__global__ __launch_bounds__(64) void greedy_groups_kernel(const uint16_t* near, int B, int stride, int m, int32_t* order) {
    __shared__ unsigned char taken[kScheduleMaxQueries + 64];
    __shared__ uint16_t found[kScheduleMaxQueries];
    const int lane = threadIdx.x;
    for (int i = lane; i < kScheduleMaxQueries + 64; i += 64) taken[i] = i < B ? 0 : 1;
    __syncthreads();
    // lowest remaining query at or above `from`, B when there is none
    auto lowest_free = [&](int from) -> int {
        for (; from < B; from += 64) {
            const uint64_t free_lanes = __ballot(taken[from + lane] == 0);       // past B: taken
            if (free_lanes) return from + __ffsll((long long)free_lanes) - 1;
        }
        return B;
    };
    auto fetch = [&](int row, int at) { return *(const uint4*)(near + (size_t)row * stride + at + lane * 8); };
    int pos = 0, seed = 0;
    uint4 cur = fetch(0, 0);
    while (seed < B) {
        if (lane == 0) { taken[seed] = 1; found[pos] = (uint16_t)seed; }
        __syncthreads();
        ++pos;
        const int guess = lowest_free(seed + 1);
        uint4 ahead = cur;
        if (guess < B) ahead = fetch(guess, 0);
        int need = min(m - 1, B - pos);
        for (int at = 0; need > 0 && at < stride; at += kNearStep) {
            const uint4 v = at == 0 ? cur : fetch(seed, at);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            uint32_t x[8];
            unsigned char t[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = (w[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = taken[min(x[e], (uint32_t)kScheduleMaxQueries)];      // 0xFFFF: reads as taken
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (need > 0) {
                    const uint64_t is_free = __ballot(t[e] == 0);
                    const int rank = __popcll(is_free & ((1ull << lane) - 1ull));
                    if (t[e] == 0 && rank < need) { taken[x[e]] = 1; found[pos + rank] = (uint16_t)x[e]; }
                    const int got = min(__popcll(is_free), need);
                    pos += got;
                    need -= got;
                }
            }
            __syncthreads();
        }
        const int next = lowest_free(seed + 1);
        cur = next == guess || next >= B ? ahead : fetch(next, 0);
        seed = next;
    }
    __syncthreads();
    for (int i = lane; i < B; i += 64) order[i] = (int32_t)found[i];
}

size_t schedule_near_stride(int B) { return (size_t)((B + kNearStep - 1) / kNearStep) * kNearStep; }

hipError_t launch_schedule(const float* q_dev, int B, int d, int m, double* dist, uint16_t* near, int32_t* order, hipStream_t s) {
    if (B < 1 || B > kScheduleMaxQueries || d < 1 || m < 1) return hipErrorInvalidValue;
    const int tiles = (B + kPairTile - 1) / kPairTile;
    hipLaunchKernelGGL(pair_dist_kernel, dim3(tiles, tiles), dim3(256), 0, s, q_dev, B, d, dist);
    uint32_t pad = 64;
    while (pad < (uint32_t)B) pad <<= 1;
    const unsigned threads = std::min<uint32_t>(1024, std::max<uint32_t>(64, pad / 2));
    const int stride = (int)schedule_near_stride(B);
    hipLaunchKernelGGL(sort_near_kernel, dim3(B), dim3(threads), (size_t)pad * 10, s, dist, B, pad, stride, near);
    hipLaunchKernelGGL(greedy_groups_kernel, dim3(1), dim3(64), 0, s, near, B, stride, m, order);
    return hipGetLastError();
}

}  // namespace ivf
