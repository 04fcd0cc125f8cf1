// Batched list scan for query batches that share probed clusters (TeleRAG Sec. 4.2 "Batching":
// the GPU part of the search becomes a matrix-matrix product).  Each selected list is read from
// HBM once per group of queries that probe it (up to 32 for fp16 / bf16 rows, up to 16 for fp32
// rows); scores come from MFMA (v_mfma_f32_32x32x16 f16 / bf16, or v_mfma_f32_16x16x4 f32 for fp32 rows and
// more than 8 queries; fp32 accumulate) or the vector units and are only used to FILTER rows: a row whose approximate score reaches the query's
// threshold becomes a candidate, and the final ranking is done on fp64 re-scores with the fp32
// query, exactly as in the single-query path.
//
// Scores are "larger is better": <q, y> for the inner product, -|q - y|^2 for squared L2.  The
// MFMA always computes <q, y>; for L2 the filter score is 2 <q, y> - |y|^2 - |q|^2 with |y|^2
// from a table of row norms made when the index is built.
//
// Threshold of a query: the k-th best fp32 score over a sample of its nearest cluster (a lower
// bound of its k-th best score over all selected clusters), lowered by a bound eps on the error
// of the filter score (query rounded to the storage type, fp32 accumulation, rounded norms).
// Every true top-k row passes this filter.
#include "ivf_device.h"
#include "../../include/ivf.h"
#include <hip/hip_ext.h>
#include <algorithm>
#include <type_traits>

namespace ivf {
using namespace dev;

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int kBatchWaves = 8;      // wavefronts of a batched scan workgroup
constexpr int kBatchThreads = kBatchWaves * 64;
constexpr int kTileRows = kBatchWaves * 32;     // rows per task: 32 per wavefront
constexpr int kStageLd = 64 + 8;   // elements per row of a wavefront's staging area: 64 + padding
constexpr int kGroupQ = 32;        // queries per task: one MFMA tile wide
constexpr int kQPad = 8;           // padding (elements) of a staged query row in LDS
constexpr int kStage16 = 2;        // 64-element blocks of a row per pipeline stage (fp16 / bf16 rows)

// ---- row norms of the lists (one-time, at build) ---------------------------------------------------
// Squared norms summed in fp64 and rounded once to fp32; the largest goes to out_bits, all of
// them to out_norm when that is not null.
__global__ void row_norm_kernel(const void* lists, int dtype, int64_t n, int d, unsigned int* out_bits, float* out_norm) {
    const int lane = threadIdx.x & 63;
    int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    float best = 0.f;
    for (int64_t r = wave; r < n; r += nwaves) {
        double s = 0.0;
        for (int t = lane; t < d; t += 64) {
            const double x = widen(lists, dtype, (size_t)r * d + t);
            s = fma(x, x, s);
        }
        const float f = (float)wave_sum(s);
        if (out_norm && lane == 0) out_norm[r] = f;
        best = fmaxf(best, f);
    }
    if (lane == 0) atomicMax(out_bits, __float_as_uint(best));   // non-negative floats order as integers
}

hipError_t launch_row_norms(const void* lists, int dtype, int64_t n, int d, unsigned int* out_bits, float* out_norm, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 3) / 4;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(row_norm_kernel, dim3((unsigned)blocks), dim3(256), 0, s, lists, dtype, n, d, out_bits, out_norm);
    return hipGetLastError();
}

// ---- in front of the scan: threshold sample, queries in the storage type, cluster -> queries map ---------
// One launch for everything that needs only the selected clusters: its workgroups differ in what
// they do (the steps are short, and as launches of their own they cost more than they computed:
// sample, queries, map and task list in seven launches 65, 72 and 260 us for 8 and 32 queries x 768
// fp32 and 256 x 1024 bf16 with 128, 32 and 512 clusters each; the two launches here 15, 21 and 142).
//
// Workgroup 0 builds the map from clusters to the queries that probe them.  Each of the others
// scores one part of a query's threshold sample: fp32 scores (fp32 query; <q, y>, or -sum (q - y)^2
// for L2) of the first rows of the query's (at most 64 nearest) selected clusters, taken in probe order
// (usually all from the nearest cluster; more clusters when those are small).  Any subset of the
// selected rows gives a valid lower bound of the k-th best score over all of them.  How many: the
// k-th best of S rows out of n alike ones lets about k n / S of them pass, so S may be small where
// the clusters are: half the mean size of the eight nearest, but at least 512 and 8 k, and so many
// that a query whose selected rows are all alike fills half of its candidate list; at most 2048.
// The bytes of the sample are what this launch costs (32 queries x 768 fp32: 2048 rows 37 us, 512
// 13; 256 queries x 1024 bf16 with k 100: 2048 rows 190 us, 800 104).
// A wavefront scores four rows, all of them in flight: the sample is bound by the bytes of its
// rows when there are many queries and by the memory round trips in front of them when there are
// few.  One more workgroup per query rounds the query to the storage type.
constexpr int kFrontThreads = 512;
constexpr int kSampleRows = 2048;
constexpr int kSampleStep = kFrontThreads / 64 * 4;          // rows a workgroup scores at a time
// Workgroups per query: one step each for small batches, more steps once the workgroups of the
// batch fill the chip (four resident per compute unit): with 32 per query the starts of 8192
// workgroups took 150 us of a 256-query batch.
static int sample_parts(int nq) { return std::max(4, std::min(kSampleRows / kSampleStep, 1024 / nq)); }
constexpr int kMapLdsLists = 8192;          // up to this many clusters the map is counted in LDS
// With more clusters the pairs are counted in global memory: by the workgroup of the map itself while they
// are few, else by the whole chip in two launches of their own.
// Whole calls, us, map's workgroup / whole chip: 4096 pairs of 16384 clusters 137 / 140, 8192 164 / 162,
// 16384 203 / 184, 131072 (256 queries x 512) 452 / 269; of 65536 clusters 4096 234 / 226, 131072 860 / 663.
constexpr uint32_t kMapSpreadPairs = 8192;
static bool map_counted_before(int nlist, int nq, int nprobe) {
    return nlist > kMapLdsLists && (uint64_t)nq * (uint64_t)nprobe >= kMapSpreadPairs;
}

__global__ __launch_bounds__(256) void clear_counts_kernel(BatchedArgs a) {
    const int c = (int)(blockIdx.x * 256u + threadIdx.x);
    if (c < a.nlist) a.list_count[c] = 0u;
}

__global__ __launch_bounds__(256) void count_pairs_kernel(BatchedArgs a) {
    const uint32_t pairs = (uint32_t)a.nq * (uint32_t)a.nprobe, i = blockIdx.x * 256u + threadIdx.x;
    if (i < pairs) atomicAdd(&a.list_count[a.probe[i]], 1u);
}

// Map: queries per cluster, and their prefix sums qstart (= cursor) and tstart (tasks per cluster).
// One workgroup: LDS atomics and a few rounds of prefix sums, beside the sample.  (The places of the
// queries are filled in by the next launch: 131,072 scattered stores from one compute unit took
// 140 us, from all of them 6.)
template <bool LDS>
__device__ __forceinline__ void build_map(const BatchedArgs& a, uint32_t* cnt, bool counted) {
    __shared__ uint32_t wsum_q[kFrontThreads / 64], wsum_t[kFrontThreads / 64];
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    const uint32_t pairs = (uint32_t)a.nq * (uint32_t)a.nprobe;
    // counters in global memory are read past the L1 and ordered by device-wide fences
    auto meet = [&]() { if (!LDS) __threadfence(); __syncthreads(); };
    auto count_of = [&](int c) -> uint32_t { return LDS ? cnt[c] : __hip_atomic_load(&cnt[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (tid == 0) *a.ticket = 0u;
    if (!counted) {
        for (int c = tid; c <= a.nlist; c += kFrontThreads) {          // one more: pairs past the end count there
            if (LDS) cnt[c] = 0u;
            else __hip_atomic_store(&cnt[c], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        meet();
    }
    // sixteen pairs per thread and pass: all requested before the first is used, and no branches that
    // differ between lanes, so that neither the reads nor the atomics wait for each other
#pragma unroll 1
    for (uint32_t i0 = 0; i0 < pairs && !counted; i0 += kFrontThreads * 16) {
        int32_t c[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) c[u] = a.probe[min(i0 + (uint32_t)(u * kFrontThreads + tid), pairs - 1)];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const uint32_t i = i0 + (uint32_t)(u * kFrontThreads + tid);
            if (i0 + (uint32_t)(u * kFrontThreads) < pairs) atomicAdd(&cnt[i < pairs ? c[u] : a.nlist], 1u);
        }
    }
    meet();
    // prefix sums over all clusters of (queries per cluster) and (tasks per cluster), four clusters per thread
    uint32_t carry_q = 0, carry_t = 0;
    unsigned long long rows = 0;
#pragma unroll 1
    for (int base = 0; base < a.nlist; base += kFrontThreads * 4) {
        uint32_t cq[4], ct[4], sq = 0, st = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = base + tid * 4 + u;
            cq[u] = 0; ct[u] = 0;
            if (c < a.nlist) {
                const uint32_t n = (uint32_t)(a.off[c + 1] - a.off[c]);
                cq[u] = count_of(c);
                ct[u] = cq[u] ? ((n + kTileRows - 1) / kTileRows) * ((cq[u] + a.group_q - 1) / a.group_q) : 0u;
                if (cq[u]) rows += n;
            }
            sq += cq[u]; st += ct[u];
        }
        uint32_t iq = sq, it = st;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t uq = __shfl_up(iq, o), ut = __shfl_up(it, o);
            if (lane >= o) { iq += uq; it += ut; }
        }
        if (lane == 63) { wsum_q[wave] = iq; wsum_t[wave] = it; }
        __syncthreads();
        uint32_t oq = carry_q + iq - sq, ot = carry_t + it - st;
#pragma unroll
        for (int w = 0; w < kFrontThreads / 64; ++w) {
            if (w < wave) { oq += wsum_q[w]; ot += wsum_t[w]; }
            carry_q += wsum_q[w]; carry_t += wsum_t[w];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = base + tid * 4 + u;
            if (c < a.nlist) { a.qstart[c] = oq; a.tstart[c] = ot; a.cursor[c] = oq; }
            oq += cq[u]; ot += ct[u];
        }
        __syncthreads();
    }
    if (tid == 0) { a.qstart[a.nlist] = carry_q; a.tstart[a.nlist] = carry_t; }
    // rows the scan covers once per cluster (for the roofline accounting)
    if (a.rows_counter) {
        for (int m = 32; m >= 1; m >>= 1) rows += __shfl_xor(rows, m);
        if (lane == 0 && rows) atomicAdd(a.rows_counter, rows);
    }
}

// Query `qi` rounded to the storage type, its norm and the bound of |filter score - exact score|
// for any row y.  Inner product from the MFMA: the query rounding contributes |<q~ - q, y>| <=
// |q~ - q| |y| (Cauchy-Schwarz, with the residual norm measured here), the fp32 accumulation at
// most acc_coef |q~| |y|.  The fp32 sample score behind the threshold is off by at most samp_coef
// |q| |y| (inner product) or samp_coef |q - y|^2 (L2: every term of the sum is positive).  The L2
// filter score 2 <q, y> - |y|^2 - |q|^2 doubles the inner-product error and adds the rounding of
// the two norms and of its two operations, each at most 2^-24 (|q| + |y|)^2.  A little slack
// absorbs the rounding of this arithmetic itself.
__device__ __forceinline__ void prepare_query(const BatchedArgs& a, int qi) {
    __shared__ float p_s[kFrontThreads / 64], p_res[kFrontThreads / 64];
    __shared__ double p_qq[kFrontThreads / 64];
    float s = 0.f, res = 0.f;          // |q~|^2 of the rounded query and |q~ - q|^2 of the rounding
    double qq = 0.0;                   // |q|^2
    const int epl = a.dtype == 0 ? 4 : 8, whole = a.d / epl * epl;      // elements in whole 16-byte chunks
    for (int t = threadIdx.x; t < a.dq; t += kFrontThreads) {
        // the scan takes a last, partial chunk from the 16 bytes that end the row, less what the chunk before it has
        const int e = t < whole ? t : t < whole + epl && whole < a.d ? a.d - epl + t - whole : a.d;
        const bool in = t < whole || (e >= whole && e < a.d);
        const float x = in ? a.q[(size_t)qi * a.d + e] : 0.f;
        float xr = x;
        const size_t o = (size_t)qi * a.dq + t;
        if (a.dtype == 1) { _Float16 h = (_Float16)x; ((_Float16*)a.q_store)[o] = h; xr = (float)h; }
        else if (a.dtype == 2) { __bf16 h = (__bf16)x; ((__bf16*)a.q_store)[o] = h; xr = (float)h; }
        else if (a.dq != a.d) ((float*)a.q_store)[o] = x;
        s = fmaf(xr, xr, s);
        res = fmaf(xr - x, xr - x, res);
        qq = fma((double)x, (double)x, qq);
    }
    s = group_sum<64>(s);
    res = group_sum<64>(res);
    qq = wave_sum(qq);
    if (lane_id() == 0) { p_s[wave_id()] = s; p_res[wave_id()] = res; p_qq[wave_id()] = qq; }
    __syncthreads();
    if (threadIdx.x == 0) {
        s = 0.f; res = 0.f; qq = 0.0;
        for (int w = 0; w < kFrontThreads / 64; ++w) { s += p_s[w]; res += p_res[w]; qq += p_qq[w]; }
        const float ymax = sqrtf(__uint_as_float(*a.row_norm_max_bits));
        const float qn = sqrtf((float)qq);
        const float ip_err = (sqrtf(res) + a.acc_coef * sqrtf(s)) * ymax;
        const float eps = a.metric == 0 ? 1.01f * (ip_err + a.samp_coef * qn * ymax)
                                        : 1.01f * (2.f * ip_err + (a.samp_coef + 0x1p-21f) * (qn + ymax) * (qn + ymax));
        a.eps[qi] = eps;
        a.qq[qi] = (float)qq;
        // The bound says nothing when it is no finite number (infinities, values beyond the storage type) or
        // when squares and products underflow; such a query starts with a full candidate list: no row is
        // added to it and it is searched again in fp64.
        const bool bound = eps < INFINITY && (qq == 0.0 || qq >= 1e-25) && ymax * ymax >= 1e-25f;
        a.cand_count[(size_t)qi * kCountStride] = bound || a.keep_all ? 0u : (uint32_t)a.cand_cap + 1u;
    }
}

template <typename T, bool TAIL>
__global__ __launch_bounds__(kFrontThreads) void batch_front_kernel(BatchedArgs a, int parts, int counted) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (blockIdx.x == 0) {
        if (a.nlist <= kMapLdsLists) build_map<true>(a, (uint32_t*)smem, false);
        else build_map<false>(a, a.list_count, counted != 0);
        return;
    }
    constexpr int EPL = T::kPerLoad, U = kSampleStep / (kFrontThreads / 64), V = 4;      // rows of a wavefront, 16-byte loads per lane and row in flight
    const int qi = (int)(blockIdx.x - 1) / (parts + 1), part = (int)(blockIdx.x - 1) % (parts + 1) - 1;
    const int lane = lane_id(), wave = wave_id();
    float* ql = (float*)smem;
    if (part < 0) {
        prepare_query(a, qi);
        return;
    }
    // The rows of the first 64 selected clusters laid end to end: lane i holds cluster i's first
    // row and the running total of rows up to and including it (one parallel prefix, so that
    // finding the cluster of a sample row is a ballot instead of a walk through dependent loads).
    const int32_t* pr = a.probe + (size_t)qi * a.nprobe;
    int64_t my_lo = 0;
    uint32_t my_n = 0;
    if (lane < a.nprobe) {
        const int c = pr[lane];
        my_lo = a.off[c];
        my_n = (uint32_t)(a.off[c + 1] - my_lo);
    }
    for (int i = threadIdx.x; i < a.d; i += kFrontThreads) ql[i] = a.q[(size_t)qi * a.d + i];
    uint32_t my_end = my_n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(my_end, o);
        if (lane >= o) my_end += up;
    }
    auto locate = [&](uint32_t r) -> int64_t {           // global row of sample row r, -1 past the last row
        const uint64_t b = __ballot(r < my_end);
        if (b == 0) return -1;
        const int i = __ffsll((long long)b) - 1;
        const uint32_t end_i = read_lane(my_end, i), n_i = read_lane(my_n, i);
        const int64_t lo_i = ((int64_t)read_lane((uint32_t)((uint64_t)my_lo >> 32), i) << 32) | read_lane((uint32_t)my_lo, i);
        return lo_i + (int64_t)(r - (end_i - n_i));
    };
    __syncthreads();
    const uint32_t rows = a.rprefix[(size_t)qi * (a.nprobe + 1) + a.nprobe];
    const uint32_t at_least = (uint32_t)((uint64_t)rows * (uint64_t)a.k * 2u / (uint64_t)a.cand_cap);
    const uint32_t want = min(max(max(read_lane(my_end, min(7, a.nprobe - 1)) / 16, at_least), max(512u, 8u * (uint32_t)a.k)), (uint32_t)kSampleRows);
    const int chunks = TAIL ? (a.d + EPL - 1) / EPL : a.d / EPL;
#pragma unroll 1
    for (uint32_t r0 = (uint32_t)(part * kSampleStep + wave * U); r0 < (uint32_t)kSampleRows; r0 += (uint32_t)(parts * kSampleStep)) {
        uint32_t key = 0;                                 // lane u < U: the ordered score of sample row r0 + u, 0 = none
        int64_t g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) g[u] = locate(r0 + u);
        if (g[0] >= 0 && r0 < want) {
            const unsigned char* rp[U];
            float s[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                rp[u] = (const unsigned char*)a.lists + (size_t)(g[u] >= 0 ? g[u] : g[0]) * a.d * T::kBytes;      // past the end: a valid row again
                s[u] = 0.f;
            }
#pragma unroll 1
            for (int c0 = lane; c0 < chunks; c0 += 64 * V) {
                uint4 v[V][U];
#pragma unroll
                for (int w = 0; w < V; ++w) {
                    const int ch = min(c0 + 64 * w, chunks - 1);
#pragma unroll
                    for (int u = 0; u < U; ++u) v[w][u] = load_chunk<TAIL>(rp[u] + (size_t)(TAIL ? min(ch * EPL, a.d - EPL) * T::kBytes : ch * 16));
                }
#pragma unroll
                for (int w = 0; w < V; ++w) {
                    const int ch = c0 + 64 * w;
                    if (ch >= chunks) break;
                    // TAIL: the last chunk of a row is the 16 bytes that end it, less what the chunk before has
                    const int skip = TAIL ? max(ch * EPL - (a.d - EPL), 0) : 0;
                    float qv[EPL];
#pragma unroll
                    for (int e = 0; e < EPL; ++e) qv[e] = e < skip ? 0.f : ql[ch * EPL + e - skip];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        float x[EPL];
                        Unpack<T>::run(v[w][u], x);
#pragma unroll
                        for (int e = 0; e < EPL; ++e) {
                            if (TAIL && e < skip) x[e] = 0.f;
                            if (a.metric == 0) s[u] = fmaf(qv[e], x[e], s[u]);
                            else { const float df = qv[e] - x[e]; s[u] = fmaf(df, df, s[u]); }
                        }
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float ck = read_lane(group_total_last_lane<64>(s[u]), 63);
                if (a.metric != 0) ck = -ck;
                if (lane == u && g[u] >= 0 && ck > -INFINITY) key = ordered(ck);      // not a number: no bound from this row
            }
        }
        if (lane < U) a.thr_part[(size_t)qi * kSampleRows + r0 + lane] = key;
    }
}

// Workgroups 0 .. nq - 1: the threshold of a query, the k-th best score of its sample less eps (a
// bucket cut leaves a few more than k, which are ranked by counting).  The others fill the map
// (qidx: the queries grouped by cluster) and write the task list, one wavefront per cluster: tasks
// of a cluster are ordered (query group, row tile), so that tiles of one group are consecutive.
__global__ __launch_bounds__(256) void batch_tasks_kernel(BatchedArgs a) {
    __shared__ uint32_t pool[kSampleRows];
    __shared__ uint32_t hist[256], red[96];
    __shared__ uint32_t s_cnt, s_kth;
    const int tid = threadIdx.x, lane = lane_id();
    if ((int)blockIdx.x >= a.nq) {
        const uint32_t pairs = (uint32_t)a.nq * (uint32_t)a.nprobe, stride = (gridDim.x - (uint32_t)a.nq) * 256u;
        for (uint32_t i = (blockIdx.x - (uint32_t)a.nq) * 256u + (uint32_t)tid; i < pairs; i += stride)
            a.qidx[atomicAdd(&a.cursor[a.probe[i]], 1u)] = i / (uint32_t)a.nprobe;
        const int step = ((int)gridDim.x - a.nq) * 4;
        for (int c = ((int)blockIdx.x - a.nq) * 4 + wave_id(); c < a.nlist; c += step) {
            const uint32_t t0 = a.tstart[c], t1 = a.tstart[c + 1];
            if (t0 == t1) continue;
            const uint32_t n = (uint32_t)(a.off[c + 1] - a.off[c]);
            const uint32_t tiles = (n + kTileRows - 1) / kTileRows, lo = (uint32_t)a.off[c];
            const uint32_t q0 = a.qstart[c], nq = a.qstart[c + 1] - q0, gq = (uint32_t)a.group_q;
            for (uint32_t i = lane; i < t1 - t0; i += 64) {
                const uint32_t group = i / tiles, row = i % tiles * kTileRows;
                a.tasks[t0 + i] = BatchTask{lo + row, min((uint32_t)kTileRows, n - row), q0 + group * gq, min(gq, nq - group * gq)};
            }
        }
        return;
    }
    const int qi = blockIdx.x;
    const uint32_t k = (uint32_t)a.k;
    uint32_t v[kSampleRows / 256];
#pragma unroll
    for (int u = 0; u < kSampleRows / 256; ++u) v[u] = a.thr_part[(size_t)qi * kSampleRows + u * 256 + tid];
#pragma unroll
    for (int u = 0; u < kSampleRows / 256; ++u) pool[u * 256 + tid] = v[u];
    if (tid == 0) { s_cnt = 0; s_kth = 0xFFFFFFFFu; }
    __syncthreads();
    const BucketCut bc = block_bucket_cut([&](uint32_t i) { return pool[i]; }, kSampleRows, k, hist, red);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSampleRows / 256; ++u) {
        const bool ok = v[u] != 0 && bc.pass(v[u]);
        const uint64_t b = __ballot(ok);
        if (b) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&s_cnt, (uint32_t)__popcll(b));
            base = read_lane(base, 0);
            if (ok) pool[base + __popcll(b & ((1ull << lane) - 1ull))] = v[u];
        }
    }
    __syncthreads();
    const uint32_t cnt = s_cnt;
    if (a.cand_count[(size_t)qi * kCountStride] != 0) {        // no bound for this query (prepare_query): nothing passes
        if (tid == 0) a.thr[qi] = INFINITY;
        return;
    }
    if (cnt < k || a.keep_all) {                               // fewer than k rows sampled: everything passes
        if (tid == 0) a.thr[qi] = -INFINITY;
        return;
    }
    // the k-th best: the smallest with fewer than k above it (of a mass of equal ones few are counted)
#pragma unroll 1
    for (uint32_t t = tid; t < cnt; t += 256) {
        const uint32_t me = pool[t];
        if (me >= __hip_atomic_load(&s_kth, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) continue;
        uint32_t above = 0;
#pragma unroll 1
        for (uint32_t j0 = 0; j0 < cnt; j0 += 8) {
            uint32_t o[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u] = pool[min(j0 + u, cnt - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) above += (uint32_t)((o[u] > me) & (j0 + u < cnt));
        }
        if (above < k) atomicMin(&s_kth, me);
    }
    __syncthreads();
    if (tid == 0) a.thr[qi] = unordered(s_kth) - a.eps[qi];
}

// ---- how the scan workgroups get their tasks ---------------------------------------------------------------
// The workgroups resident on the GPU draw runs of consecutive tasks from one counter (a.ticket,
// zero at launch) until the list is used up: compute units, and whole XCDs, differ by several
// per cent in how fast they stream from HBM, and with equal shares the slowest one sets the
// kernel's time.  A run has up to kRunMax tasks (tasks that follow each other mostly share their
// cluster and group of queries, which are staged once) and shrinks towards the end of the list
// (remaining / (4 x workgroups), at least one), so that all workgroups finish within about a task
// of each other.  Every workgroup leaves once a run starts past the end of the list.
constexpr uint32_t kRunMax = 8;

// A load of wave-uniform data that this kernel does not write: through the scalar cache, beside
// the vector loads, which return in order and would hold it back.
template <typename V>
__device__ __forceinline__ V load_scalar(const V* p) {
    return *(const __attribute__((address_space(4))) V*)(uintptr_t)p;
}

struct TaskFeed {
    uint32_t t, t_stop, total;      // same in all threads: next task, end of the run, end of the list
    uint32_t flip;                  // which half of s_run the next run goes to
    uint32_t ahead_t0, ahead_n;     // thread 0: the run reserved ahead
    __device__ __forceinline__ void reserve(const BatchedArgs& a) {
        const uint32_t left = total - min(total, ahead_t0 + ahead_n);
        ahead_n = max(1u, min(kRunMax, left / (4u * gridDim.x)));
        ahead_t0 = atomicAdd(a.ticket, ahead_n);
    }
    __device__ __forceinline__ void start(const BatchedArgs& a) {
        total = load_scalar(&a.tstart[a.nlist]);
        t = t_stop = 0;
        flip = 0;
        ahead_t0 = ahead_n = 0;
        if (threadIdx.x == 0) reserve(a);
    }
    // the next task, or false when the list is used up; all threads of the workgroup call it together.
    // s_run: two halves used in turn, so that one barrier separates writing from reading (16 bytes, so that the
    // dynamic LDS area behind the static one stays 16-byte aligned)
    __device__ __forceinline__ bool next(const BatchedArgs& a, uint32_t (*s_run)[2], BatchTask& task) {
        if (t == t_stop) {
            if (threadIdx.x == 0) {
                s_run[flip][0] = ahead_t0;
                s_run[flip][1] = min(ahead_t0 + ahead_n, total);
            }
            __syncthreads();
            // (read from LDS: the compiler is told that the values are the same in every lane, so
            // that the task and everything derived from it stay in scalar registers)
            t = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_run[flip][0]);
            t_stop = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_run[flip][1]);
            flip ^= 1u;
            if (t >= total) return false;
            // the run after this one: asked for behind the barrier, so that only this wavefront
            // waits for the counter while the others are already at work
            if (threadIdx.x == 0) reserve(a);
        }
        const u4_t v = load_scalar((const u4_t*)(a.tasks + t));
        task = BatchTask{v.x, v.y, v.z, v.w};
        ++t;
        return true;
    }
};

// ---- the MFMA scan -------------------------------------------------------------------------------------
template <typename T> struct Mfma;
template <> struct Mfma<F16> {
    typedef half8_t frag;
    __device__ static __forceinline__ float16_t run(frag a, frag b, float16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};
template <> struct Mfma<BF16> {
    typedef bf16x8_t frag;
    __device__ static __forceinline__ float16_t run(frag a, frag b, float16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};

// One workgroup (8 wavefronts) per task: 256 rows of one cluster against up to 32 of the queries
// that probe it.  The queries (storage type) are staged in LDS once per (cluster, group).  Each
// wavefront streams its 32 rows from HBM with coalesced loads (8 lanes cover one 128-byte line of
// a row, an instruction 8 rows), turns each block of 64 elements into MFMA A fragments (lane l:
// row l % 32, eight elements per step) through a small LDS area of its own, and reads the B
// fragments (lane l: query l % 32, the same elements) from the staged queries.  Scores that reach
// the query's threshold are appended to the query's candidate list.
//
// TAIL: rows that are not whole blocks of 64 elements, or not whole 16-byte chunks and so start at any
// element.  A lane whose chunk reaches past the end of the row loads the 16 bytes that END with the row
// and clears what does not count (the staged queries are laid out the same way): no load leaves the row.
// These loads are cached ones: the 128-byte pieces of such rows straddle lines, which streaming loads
// fetched 1.56 times (48 x 100 fp32: 82 us, 99 with them; 106 x 283 fp16: 238, 268).
template <typename T, int METRIC, bool TAIL>
__global__ __launch_bounds__(kBatchThreads) void batched_scan_kernel(BatchedArgs a, int resident) {
    typedef typename Mfma<T>::frag frag;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t s_q[kGroupQ];
    const int lane = lane_id(), wave = wave_id();
    const int d = a.d, dq = TAIL ? a.dq : a.d, qstride = dq + kQPad;
    // queries, their thresholds and norms: of the whole batch (resident), or of one group
    const int slots = resident ? a.nq : kGroupQ;
    uint16_t* stage = (uint16_t*)smem + (size_t)wave * 32 * kStageLd;    // [32][kStageLd], this wavefront's
    uint16_t* qs = (uint16_t*)smem + (size_t)kBatchWaves * 32 * kStageLd;     // [slots][dq + kQPad] storage-type queries
    float* s_thr = (float*)(qs + (size_t)slots * qstride);
    float* s_qq = s_thr + slots;
    const int chunks = dq / 8;                           // 16-byte chunks per query row
    if (resident) {
        for (int i = threadIdx.x; i < a.nq * chunks; i += blockDim.x) {
            const int qi = i / chunks, ch = i - qi * chunks;
            *(uint4*)(qs + (size_t)qi * qstride + ch * 8) = *(const uint4*)((const uint16_t*)a.q_store + (size_t)qi * dq + ch * 8);
        }
        for (int i = threadIdx.x; i < a.nq; i += blockDim.x) { s_thr[i] = a.thr[i]; s_qq[i] = a.qq[i]; }
        __syncthreads();
    }
    __shared__ __align__(16) uint32_t s_run[2][2];
    TaskFeed feed;
    feed.start(a);
    uint32_t staged = 0xFFFFFFFFu;
    BatchTask task;
    const int col = lane & 31, khalf = lane >> 5;
    while (feed.next(a, s_run, task)) {
        const uint32_t qbase = task.qbase, nqg = task.nq;
        if (!resident && qbase != staged) {
            __syncthreads();                              // everyone is done with the previous queries
            if (threadIdx.x < nqg) {
                const uint32_t qi = a.qidx[qbase + threadIdx.x];
                s_q[threadIdx.x] = qi; s_thr[threadIdx.x] = a.thr[qi]; s_qq[threadIdx.x] = a.qq[qi];
            }
            __syncthreads();
            for (int i = threadIdx.x; i < (int)nqg * chunks; i += blockDim.x) {
                const int p = i / chunks, ch = i - p * chunks;
                *(uint4*)(qs + (size_t)p * qstride + ch * 8) = *(const uint4*)((const uint16_t*)a.q_store + (size_t)s_q[p] * dq + ch * 8);
            }
            __syncthreads();
            staged = qbase;
        }
        const uint32_t lo = task.row0, n = task.rows, r0 = wave * 32;      // first row of this wavefront in the task
        if (r0 >= n) continue;
        // Loading role of a lane: 16-byte chunk lane % 8 of rows lane / 8 + {0, 8, 16, 24} of each
        // 64-element block (rows past the end re-read the last one).  Element order inside the dot
        // product is free, so MFMA step j of a block takes, for the lane half h, elements
        // 32 h + 8 j .. + 7 of the block from both operands.
        const int lrow = lane >> 3, lchunk = lane & 7;
        const uint16_t* lptr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            lptr[u] = (const uint16_t*)a.lists + ((size_t)lo + min(r0 + (uint32_t)(lrow + 8 * u), n - 1)) * d + (TAIL ? 0 : lchunk * 8);
        uint32_t keep[4] = {~0u, ~0u, ~0u, ~0u};          // TAIL: what counts of this lane's chunk in the last block
        if (TAIL) {
            const int at = (d - 1) / 64 * 64 + lchunk * 8, skip = max(at - (d - 8), 0);
#pragma unroll
            for (int e = 0; e < 8; ++e) if (e < skip) keep[e / 2] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
        }
        // the query of this lane's scores (places of the group that no query has: one again), and where it is in LDS
        const uint32_t place = min((uint32_t)col, nqg - 1), qi = a.qidx[qbase + place], slot = resident ? qi : place;
        const uint16_t* brow = qs + (size_t)slot * qstride + khalf * 32;
        uint16_t* wpos = stage + lrow * kStageLd + lchunk * 8;
        const uint16_t* rpos = stage + col * kStageLd + khalf * 32;
        float16_t acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
        float yy[16];                  // L2: squared norms of the rows this lane will hold scores of
        if (METRIC != 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                yy[i] = a.row_norm[(size_t)lo + min(r0 + (uint32_t)((i / 4) * 8 + khalf * 4 + (i % 4)), n - 1)];
        }
        // kStage16 blocks (of 64 elements, 4 MFMA steps) per stage, the next stage's rows in flight
        uint4 av[2][4 * kStage16];
        auto issue = [&](int k0, uint4 (&v)[4 * kStage16]) {
#pragma unroll
            for (int b = 0; b < kStage16; ++b) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (k0 + b * 64 >= d) v[b * 4 + u] = make_uint4(0, 0, 0, 0);
                    else if (TAIL) v[b * 4 + u] = load_chunk<true>(lptr[u] + min(k0 + b * 64 + lchunk * 8, d - 8));
                    else v[b * 4 + u] = load_stream16(lptr[u] + k0 + b * 64);
                }
            }
        };
        auto consume = [&](int k0, const uint4 (&v)[4 * kStage16]) {
#pragma unroll
            for (int b = 0; b < kStage16; ++b) {
                if (k0 + b * 64 < d) {
                    // through LDS: written in the loading layout, read back as fragments.  A
                    // wavefront's LDS operations complete in order, so no barrier is needed.
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        uint4 w = v[b * 4 + u];
                        if (TAIL && k0 + b * 64 + 64 >= d) { w.x &= keep[0]; w.y &= keep[1]; w.z &= keep[2]; w.w &= keep[3]; }
                        *(uint4*)(wpos + u * 8 * kStageLd) = w;
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint4 av4 = *(const uint4*)(rpos + j * 8);
                        const uint4 bv = *(const uint4*)(brow + k0 + b * 64 + j * 8);
                        acc = Mfma<T>::run(__builtin_bit_cast(frag, av4), __builtin_bit_cast(frag, bv), acc);
                    }
                }
            }
        };
        constexpr int kStep = kStage16 * 64;              // elements per stage
        issue(0, av[0]);
        for (int k0 = 0; k0 < d; k0 += 2 * kStep) {
            if (k0 + kStep < d) issue(k0 + kStep, av[1]);
            consume(k0, av[0]);
            if (k0 + kStep >= d) break;
            if (k0 + 2 * kStep < d) issue(k0 + 2 * kStep, av[0]);
            consume(k0 + kStep, av[1]);
        }
        // lane holds query `col`, rows (i / 4) * 8 + khalf * 4 + i % 4
        const float thr = s_thr[slot];
        if (METRIC != 0) {
            const float qq = s_qq[slot];
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = fmaf(2.f, acc[i], -yy[i]) - qq;
        }
        uint32_t pass = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t r = r0 + (i / 4) * 8 + khalf * 4 + (i % 4);
            if (acc[i] >= thr && r < n && (uint32_t)col < nqg) pass |= 1u << i;
        }
        if (pass) {
            // one reservation for all rows of this lane that passed
            uint32_t pos = atomicAdd(&a.cand_count[(size_t)qi * kCountStride], (uint32_t)__popc(pass));
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if ((pass >> i) & 1u) {
                    if (pos < (uint32_t)a.cand_cap) {
                        a.cand_row[(size_t)qi * a.cand_cap + pos] = (uint32_t)(lo + r0 + (i / 4) * 8 + khalf * 4 + (i % 4));
                        a.cand_score[(size_t)qi * a.cand_cap + pos] = acc[i];
                    }
                    ++pos;
                }
            }
        }
    }
}

// fp32 rows.  Eight consecutive lanes take one 128-byte piece of a row (lane l: chunk l % 8 of rows
// l / 8 + {0, 8, 16, 24} of the wavefront's 32), three pieces of the 32 rows are in flight while the
// previous three are multiplied (12 KB per wavefront).
// Groups of up to 8 queries (most: a cluster is selected by one to four queries of a batch) are multiplied by
// the vector units: a lane adds up the products of its chunks for every query, whose chunks it
// reads from LDS, and at the end of a row the eight lanes' sums are added by a butterfly that
// leaves lane l with query l % 8.  The walk comes in sizes M = 1, 2, 4 and 8, each as long as its queries.
// Larger groups go to v_mfma_f32_16x16x4_f32, which is twice as fast for 16 queries and takes as long for fewer:
// a 16 x 4 block of rows (lane l: row l % 16, element l / 16) times a 4 x 16 block of queries (lane l: query
// l % 16, the same element).  The order of the elements inside a dot product is free, so the MFMA lane
// (row i, part p) takes the 16-byte chunk p of each 16-element block of its row and the four values of the
// chunk feed four MFMA steps; register moves across lanes (a DPP row shift and a ds_bpermute per
// value) take each value there.
// What it measured, us, all groups on the matrix cores / this: 32 queries x 768, squared L2 (1.85 GB; rows
// from the cache instead of HBM took 232 of it) 310 / 286, 8 x 768 (4.1 GB) 636 / 608, 199 x 256 with six
// queries per cluster (4.8 GB) 783 / 702, 48 x 100 (287 MB) 101 / 62, 9 x 687 (32 MB) 67 / 36.
// TAIL: as in batched_scan_kernel, for rows that are not whole pieces of 32 elements.
typedef float float4_t __attribute__((ext_vector_type(4)));
constexpr int kGroupQ32 = 16;      // queries per task for fp32 rows
constexpr int kQPad32 = 4;         // padding (floats) of a staged query row
constexpr int kStage32 = 3;        // 32-element pieces of a row per pipeline stage

// Sums of M values over eight consecutive lanes: lane l of the eight ends with value l % M of `v` (M <= 8).
template <int M>
__device__ __forceinline__ float sums_over_8(float (&v)[M]) {
    const int lane = lane_id();
    // partners: 7 - l (row_half_mirror), l ^ 2, l ^ 1; while more than one value is left a lane
    // keeps the half its own bit names and hands the other half over
    auto halve = [&](int n, bool upper, auto move) {
#pragma unroll
        for (int j = 0; j < n; ++j) {
            const float keep = upper ? v[j + n] : v[j], give = upper ? v[j] : v[j + n];
            v[j] = keep + move(give);
        }
    };
    auto m4 = [](float x) { return dpp_move<0x141>(x); };
    auto m2 = [](float x) { return dpp_move<0x4E>(x); };
    auto m1 = [](float x) { return dpp_move<0xB1>(x); };
    if constexpr (M == 8) halve(4, (lane & 4) != 0, m4);
    else {
#pragma unroll
        for (int j = 0; j < M; ++j) v[j] += m4(v[j]);
    }
    if constexpr (M >= 4) halve(2, (lane & 2) != 0, m2);
    else {
#pragma unroll
        for (int j = 0; j < M; ++j) v[j] += m2(v[j]);
    }
    if constexpr (M >= 2) halve(1, (lane & 1) != 0, m1);
    else v[0] += m1(v[0]);
    return v[0];
}

template <int METRIC, bool TAIL>
__global__ __launch_bounds__(kBatchThreads) void batched_scan_f32_kernel(BatchedArgs a, int resident) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t s_q[kGroupQ32];
    const int lane = lane_id(), wave = wave_id();
    const int d = a.d, dq = TAIL ? a.dq : a.d, qstride = dq + kQPad32;
    // queries, their thresholds and norms: of the whole batch (resident), or of one group
    const int slots = resident ? a.nq : kGroupQ32;
    float* qs = (float*)smem;                            // [slots][dq + kQPad32]
    float* s_thr = qs + (size_t)slots * qstride;
    float* s_qq = s_thr + slots;
    const float* q_rows = TAIL && dq != d ? (const float*)a.q_store : a.q;
    __shared__ __align__(16) uint32_t s_run[2][2];
    TaskFeed feed;
    feed.start(a);
    uint32_t staged = 0xFFFFFFFFu;
    BatchTask task;
    const int sub = lane & 7;
    const uint32_t r0 = wave * 32, lrow = (uint32_t)(lane >> 3);
    uint32_t keep[4] = {~0u, ~0u, ~0u, ~0u};              // TAIL: what counts of this lane's chunk in the last piece of a row (nothing past its end)
    if (TAIL) {
        const int at = (d - 1) / 32 * 32 + sub * 4, skip = max(at - (d - 4), 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) if (e < skip) keep[e] = 0u;
    }
    const float* bq = qs + sub * 4;
    const int chunks = dq / 4;                            // 16-byte chunks per query row
    if (resident) {
        for (int i = threadIdx.x; i < a.nq * chunks; i += blockDim.x) {
            const int qi = i / chunks, ch = i - qi * chunks;
            *(uint4*)(qs + (size_t)qi * qstride + ch * 4) = *(const uint4*)(q_rows + (size_t)qi * dq + ch * 4);
        }
        for (int i = threadIdx.x; i < a.nq; i += blockDim.x) { s_thr[i] = a.thr[i]; s_qq[i] = a.qq[i]; }
        __syncthreads();
    }
    while (feed.next(a, s_run, task)) {
        const uint32_t nqg = task.nq;
        if (!resident && task.qbase != staged) {
            __syncthreads();                              // everyone is done with the previous queries
            if (threadIdx.x < nqg) {
                const uint32_t qi = a.qidx[task.qbase + threadIdx.x];
                s_q[threadIdx.x] = qi; s_thr[threadIdx.x] = a.thr[qi]; s_qq[threadIdx.x] = a.qq[qi];
            }
            __syncthreads();
            for (int i = threadIdx.x; i < (int)nqg * chunks; i += blockDim.x) {
                const int p = i / chunks, ch = i - p * chunks;
                *(uint4*)(qs + (size_t)p * qstride + ch * 4) = *(const uint4*)(q_rows + (size_t)s_q[p] * dq + ch * 4);
            }
            __syncthreads();
            staged = task.qbase;
        }
        if (r0 >= task.rows) continue;
        const float* lp[4];                               // rows past the end re-read the last one
#pragma unroll
        for (int u = 0; u < 4; ++u)
            lp[u] = (const float*)a.lists + ((size_t)task.row0 + min(r0 + 8u * u + lrow, task.rows - 1)) * d + (TAIL ? 0 : sub * 4);
        // rows of `task` against M places of the group on the vector units, or (M = 16) on the matrix cores
        auto walk = [&](auto size) __attribute__((always_inline)) {
            constexpr int M = decltype(size)::value;
            constexpr bool MATRIX = M > 8;
            constexpr int N = MATRIX ? 8 : 4;             // scores of a lane
            // query of this lane's scores, and where it is in LDS
            const uint32_t place = MATRIX ? (uint32_t)(lane & 15) : (uint32_t)sub;
            const uint32_t qi = a.qidx[task.qbase + min(place, nqg - 1)], slot = resident ? qi : min(place, nqg - 1);
            // row of score i in the wavefront's 32
            auto row_of = [&](int i) { return MATRIX ? (uint32_t)((i / 4) * 16 + (lane >> 4) * 4 + (i % 4)) : 8u * (uint32_t)i + lrow; };
            float yy[N];                                  // L2: squared norms of those rows
            if (METRIC != 0) {
#pragma unroll
                for (int i = 0; i < N; ++i) yy[i] = a.row_norm[(size_t)task.row0 + min(r0 + row_of(i), task.rows - 1)];
            }
            uint32_t at[MATRIX ? 1 : M];                  // LDS row of place m
            if (!MATRIX) {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const uint32_t p = min((uint32_t)m, nqg - 1);
                    at[m] = (resident ? load_scalar(&a.qidx[task.qbase + p]) : p) * (uint32_t)qstride;
                }
            }
            const float* bm = qs + (size_t)slot * qstride + (lane >> 4) * 4;     // MATRIX: this lane's query operand
            const int from = (((lane & 7) << 3) | (((lane >> 3) & 1) << 2) | (lane >> 4)) << 2;
            float acc[MATRIX ? 1 : 4][MATRIX ? 1 : M];
            float4_t macc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int u = 0; u < (MATRIX ? 1 : 4); ++u)
#pragma unroll
                for (int m = 0; m < (MATRIX ? 1 : M); ++m) acc[u][m] = 0.f;
            uint4 av[2][4 * kStage32];
            auto issue = [&](int k0, uint4 (&v)[4 * kStage32]) __attribute__((always_inline)) {
#pragma unroll
                for (int b = 0; b < kStage32; ++b) {
                    if (k0 + b * 32 >= d) break;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        v[4 * b + u] = TAIL ? load_chunk<true>(lp[u] + min(k0 + b * 32 + sub * 4, d - 4)) : load_stream16(lp[u] + k0 + b * 32);
                }
            };
            // One loaded value to its MFMA lanes.  Lanes with chunk >= 4 hold the second 16-element
            // block of the piece.  A move by four lanes inside each row of 16 lanes (DPP row shift,
            // written only to the lanes of one chunk half) gathers the first block of both row halves
            // in one register (lane (r, c): row r + 8 (c / 4), chunk c % 4) and the second block in
            // another; one lane permutation each then puts them in MFMA order.
            auto to_mfma = [&](uint32_t lo_half, uint32_t hi_half, float& first, float& second) {
                const int f = __builtin_amdgcn_update_dpp((int)lo_half, (int)hi_half, 0x114, 0xF, 0xA, false);   // row_shr:4 into chunks 4..7
                const int g = __builtin_amdgcn_update_dpp((int)hi_half, (int)lo_half, 0x104, 0xF, 0x5, false);   // row_shl:4 into chunks 0..3
                first = __int_as_float(__builtin_amdgcn_ds_bpermute(from, f));
                second = __int_as_float(__builtin_amdgcn_ds_bpermute(from, g));
            };
            auto consume = [&](int k0, const uint4 (&v)[4 * kStage32]) __attribute__((always_inline)) {
#pragma unroll
                for (int b = 0; b < kStage32; ++b) {
                    if (k0 + b * 32 >= d) break;
                    uint4 h[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        h[u] = v[4 * b + u];
                        if (TAIL && k0 + b * 32 + 32 >= d) { h[u].x &= keep[0]; h[u].y &= keep[1]; h[u].z &= keep[2]; h[u].w &= keep[3]; }
                    }
                    if constexpr (MATRIX) {
                        const float4 bv0 = *(const float4*)(bm + k0 + b * 32);
                        const float4 bv1 = *(const float4*)(bm + k0 + b * 32 + 16);
                        float x[2][2][4];          // [row block][16-element block][value of the chunk]
#pragma unroll
                        for (int rb = 0; rb < 2; ++rb) {
                            const uint4 h0 = h[2 * rb], h1 = h[2 * rb + 1];
                            to_mfma(h0.x, h1.x, x[rb][0][0], x[rb][1][0]);
                            to_mfma(h0.y, h1.y, x[rb][0][1], x[rb][1][1]);
                            to_mfma(h0.z, h1.z, x[rb][0][2], x[rb][1][2]);
                            to_mfma(h0.w, h1.w, x[rb][0][3], x[rb][1][3]);
                        }
                        const float q0[4] = {bv0.x, bv0.y, bv0.z, bv0.w}, q1[4] = {bv1.x, bv1.y, bv1.z, bv1.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            macc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0][0][e], q0[e], macc[0], 0, 0, 0);
                            macc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[1][0][e], q0[e], macc[1], 0, 0, 0);
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            macc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0][1][e], q1[e], macc[0], 0, 0, 0);
                            macc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[1][1][e], q1[e], macc[1], 0, 0, 0);
                        }
                    } else {
                        float x[4][4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) Unpack<F32>::run(h[u], x[u]);
#pragma unroll
                        for (int m = 0; m < M; ++m) {
                            const float4 q4 = *(const float4*)(bq + at[m] + k0 + b * 32);
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                acc[u][m] = fmaf(x[u][0], q4.x, acc[u][m]);
                                acc[u][m] = fmaf(x[u][1], q4.y, acc[u][m]);
                                acc[u][m] = fmaf(x[u][2], q4.z, acc[u][m]);
                                acc[u][m] = fmaf(x[u][3], q4.w, acc[u][m]);
                            }
                        }
                    }
                }
            };
            constexpr int kStep = kStage32 * 32;          // elements per stage
            issue(0, av[0]);
#pragma unroll 1
            for (int k0 = 0; k0 < d; k0 += 2 * kStep) {
                if (k0 + kStep < d) issue(k0 + kStep, av[1]);
                consume(k0, av[0]);
                if (k0 + kStep >= d) break;
                if (k0 + 2 * kStep < d) issue(k0 + 2 * kStep, av[0]);
                consume(k0 + kStep, av[1]);
            }
            float sc[N];
            if constexpr (MATRIX) {
#pragma unroll
                for (int i = 0; i < 4; ++i) { sc[i] = macc[0][i]; sc[4 + i] = macc[1][i]; }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) sc[u] = sums_over_8<M>(acc[u]);
            }
            if (place >= nqg) return;
            const float thr = s_thr[slot];
            if (METRIC != 0) {
                const float qq = s_qq[slot];
#pragma unroll
                for (int i = 0; i < N; ++i) sc[i] = fmaf(2.f, sc[i], -yy[i]) - qq;
            }
            uint32_t pass = 0;
#pragma unroll
            for (int i = 0; i < N; ++i) if (sc[i] >= thr && r0 + row_of(i) < task.rows) pass |= 1u << i;
            if (pass) {
                // one reservation for all rows of this lane that passed
                uint32_t pos = atomicAdd(&a.cand_count[(size_t)qi * kCountStride], (uint32_t)__popc(pass));
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    if ((pass >> i) & 1u) {
                        if (pos < (uint32_t)a.cand_cap) {
                            a.cand_row[(size_t)qi * a.cand_cap + pos] = task.row0 + r0 + row_of(i);
                            a.cand_score[(size_t)qi * a.cand_cap + pos] = sc[i];
                        }
                        ++pos;
                    }
                }
            }
        };
        if (nqg > 8) walk(std::integral_constant<int, 16>{});
        else if (nqg > 4) walk(std::integral_constant<int, 8>{});
        else if (nqg > 2) walk(std::integral_constant<int, 4>{});
        else if (nqg > 1) walk(std::integral_constant<int, 2>{});
        else walk(std::integral_constant<int, 1>{});
    }
}

// ---- final ranking of a query's candidates ------------------------------------------------------------------
// One workgroup per query.  Candidates are pruned by their approximate scores, each within eps of the
// exact one: with t = the k-th best of them, a row of the true top k has an approximate score of at
// least t - 2 eps.  The survivors are re-scored in fp64 (fp32 query), in the order of operations of
// the query-by-query merge, and the k best by (score, id) are ranked by counting.  When there are
// many survivors those that reach t go first: with s = the smallest of their exact scores the true
// k-th best is at least s, and of the others only the rows that reach s - eps can matter (about half
// of them).  Everything lives in LDS and nothing is sorted: bucket cuts leave a few more than k.
// What bounds it: the re-scores' trips to memory (two rows per group of lanes in flight), and in a
// batch the query with the most survivors.  (Radix selects over candidates and re-scores in global
// memory, one row in flight per group: 13, 17 and 140 us for 8, 32 and 256 queries with k 3, 10 and
// 100; this: 10, 12 and 58.)
// A query whose candidates or survivors do not fit sets its overflow flag and is searched again.
constexpr int kRescoreInFlight = 2;
constexpr uint32_t kSurvivorsAtOnce = kSelectThreads / kRescoreLanes * kRescoreInFlight * 2;     // up to here: no second look

__global__ __launch_bounds__(kSelectThreads) void batched_merge_kernel(BatchedArgs a) {
    __shared__ uint64_t s_key[kBatchSurvivors];     // ordered(fp64 score): larger is nearer
    __shared__ uint32_t s_row[kBatchSurvivors];
    __shared__ uint32_t hist[256], red[96];
    __shared__ uint32_t s_n, s_m, s_kth;
    __shared__ unsigned long long s_low;
    __shared__ int64_t o_id[IVF_MAX_K];
    __shared__ float o_dist[IVF_MAX_K];
    constexpr uint16_t kNoTie = 0xFFFFu;
    __shared__ uint16_t s_tie[kBatchSurvivors];     // survivors that share their score: how many are above them
    __shared__ uint64_t o_key[IVF_MAX_K];           // the score of those with this many above them
    __shared__ uint32_t s_ties, s_edge_n, s_edge_above;     // any; those on the edge of the k best
    __shared__ uint64_t s_edge_key;
    __shared__ unsigned long long s_top_id;
    const int tid = threadIdx.x, lane = lane_id();
    constexpr int nt = kSelectThreads;
    const int qi = blockIdx.x;
    const uint32_t k = (uint32_t)a.k;
    const uint32_t n0 = a.cand_count[(size_t)qi * kCountStride];
    // too many candidates or survivors: the query is searched again, by the host or, with redo_flag, by the
    // exact pass that follows on the stream (rows below `at_least` do not count)
    auto search_again = [&](uint32_t again, double at_least) {
        if (tid != 0) return;
        a.overflow[qi] = (int32_t)again;
        if (a.redo_flag) {
            a.redo_flag[qi] = again;
            a.redo_thr[qi] = at_least;
            a.redo_ticket[qi] = 0u;
        }
    };
    if (n0 > (uint32_t)a.cand_cap) {
        search_again(1u, -INFINITY);
        return;
    }
    const float* sc = a.cand_score + (size_t)qi * a.cand_cap;
    const uint32_t* rows0 = a.cand_row + (size_t)qi * a.cand_cap;
    // reserves a place behind counter `n` for every lane with ok
    auto place = [&](uint32_t& n, bool ok) -> uint32_t {
        const uint64_t b = __ballot(ok);
        if (!b) return 0;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&n, (uint32_t)__popcll(b));
        return read_lane(base, 0) + __popcll(b & ((1ull << lane) - 1ull));
    };
    // four candidates per thread are requested together; the first four stay in registers
    constexpr int C = 4;
    auto read_scores = [&](uint32_t i0, float (&v)[C]) {
#pragma unroll
        for (int u = 0; u < C; ++u)
            if (i0 + (uint32_t)(u * nt) < n0) v[u] = sc[min(i0 + (uint32_t)(u * nt + tid), n0 - 1)];
    };
    float first[C];
    read_scores(0, first);
    const uint32_t row_first = n0 ? rows0[min((uint32_t)tid, n0 - 1)] : 0u;
    auto for_scores = [&](auto&& use) {
#pragma unroll
        for (int u = 0; u < C; ++u)
            if ((uint32_t)(u * nt) < n0) use((uint32_t)(u * nt + tid), first[u]);
#pragma unroll 1
        for (uint32_t i0 = C * nt; i0 < n0; i0 += C * nt) {
            float v[C];
            read_scores(i0, v);
#pragma unroll
            for (int u = 0; u < C; ++u)
                if (i0 + (uint32_t)(u * nt) < n0) use(i0 + (uint32_t)(u * nt + tid), v[u]);
        }
    };
    const float eps = a.eps[qi];
    const uint32_t sub8 = (uint32_t)tid & 7u;
    // 1. the k-th best approximate score
    float kth = -INFINITY;
    if (tid == 0) { s_n = 0; s_m = 0; s_kth = 0xFFFFFFFFu; s_low = ~0ull; s_ties = 0; s_edge_n = 0; s_top_id = 0; }
    if (n0 > k) {
        // the candidates are dealt to the threads: as many threads' best reach the cut of those as
        // were asked for, so at least k candidates do, and not many more
        uint32_t mine = 0;
        for_scores([&](uint32_t i, float v) { mine = max(mine, i < n0 ? ordered(v) : 0u); });
        const BucketCut bc = block_bucket_cut([&](uint32_t) { return mine; }, (uint32_t)nt, k, hist, red);
        __syncthreads();
        uint32_t* pool = s_row;                        // ordered scores that pass the cut
        for_scores([&](uint32_t i, float v) {
            const bool ok = i < n0 && bc.pass(ordered(v));
            const uint32_t pos = place(s_n, ok);
            if (ok && pos < (uint32_t)kBatchSurvivors) pool[pos] = ordered(v);
        });
        __syncthreads();
        // masses of equal scores may let more pass than the pool holds: the smallest of those stored
        // that has fewer than k above it is then still a lower bound of the k-th best
        const uint32_t m = min(s_n, (uint32_t)kBatchSurvivors);
        for (uint32_t t = (uint32_t)tid / 8; t < m; t += nt / 8) {
            const uint32_t me = pool[t];
            // only a smaller value can still lower the result: of a mass of equal ones few are counted
            if (me >= __hip_atomic_load(&s_kth, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) continue;
            uint32_t above, equal;
            count_above(pool, m, me, sub8, above, equal);
            if (sub8 == 0 && above < k) atomicMin(&s_kth, me);
        }
        __syncthreads();
        kth = unordered(s_kth);
        if (tid == 0) s_n = 0;
    }
    __syncthreads();
    // 2. survivors: those that reach the k-th best from the front, the others from the back, these
    //    with their approximate score in the place of the exact one
    const float cut = kth - 2.f * eps;
    for_scores([&](uint32_t i, float v) {
        const bool ok = i < n0 && v >= cut, top = ok && v >= kth;
        const uint32_t row = i < (uint32_t)nt ? row_first : ok ? rows0[i] : 0u;
        const uint32_t front = place(s_n, top), back = place(s_m, ok && !top);
        if (top && front < (uint32_t)kBatchSurvivors) s_row[front] = row;
        if (ok && !top && back < (uint32_t)kBatchSurvivors) {
            s_row[kBatchSurvivors - 1 - back] = row;
            s_key[kBatchSurvivors - 1 - back] = ordered(v);
        }
    });
    __syncthreads();
    const uint32_t n_top = s_n, n_back = s_m;
    if (n_top + n_back > (uint32_t)kBatchSurvivors) {  // cannot happen unless scores are massively tied
        search_again(1u, (double)kth - 1.0001 * (double)eps);       // k rows have scores of at least kth, each within eps
        return;
    }
    // 3. fp64 re-scores of survivors c0 .. c1 - 1: a group of lanes per survivor, two rows in flight
    const float* q = a.q + (size_t)qi * a.d;
    const int sub = tid % kRescoreLanes;
    auto rescore = [&](uint32_t c0, uint32_t c1) {
        constexpr uint32_t groups = nt / kRescoreLanes;
#pragma unroll 1
        for (uint32_t c = c0 + (uint32_t)(tid / kRescoreLanes); c < c1; c += groups * kRescoreInFlight) {
            double s[kRescoreInFlight];
            uint32_t row[kRescoreInFlight];
#pragma unroll
            for (int r = 0; r < kRescoreInFlight; ++r) row[r] = s_row[min(c + groups * r, c1 - 1)];
            rescore_rows<kRescoreInFlight>(a.lists, q, a.d, a.dtype, a.metric, row, sub, s);
#pragma unroll
            for (int r = 0; r < kRescoreInFlight; ++r)
                if (sub == 0 && c + groups * r < c1) s_key[c + groups * r] = ordered(a.metric == 0 ? s[r] : -s[r]);
        }
    };
    // the others come to the front, all of them or those that reach `low`
    auto gather_back = [&](float low) -> uint32_t {
        uint32_t row[kBatchSurvivors / nt];
        bool ok[kBatchSurvivors / nt];
#pragma unroll
        for (int u = 0; u < kBatchSurvivors / nt; ++u) {
            const uint32_t i = (uint32_t)(u * nt + tid);
            ok[u] = i < n_back && unordered((uint32_t)s_key[kBatchSurvivors - 1 - min(i, (uint32_t)kBatchSurvivors - 1)]) >= low;
            row[u] = s_row[kBatchSurvivors - 1 - min(i, (uint32_t)kBatchSurvivors - 1)];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kBatchSurvivors / nt; ++u) {
            const uint32_t pos = place(s_n, ok[u]);
            if (ok[u]) s_row[pos] = row[u];
        }
        __syncthreads();
        return s_n;
    };
    const bool at_once = n_top + n_back <= kSurvivorsAtOnce;
    uint32_t done = 0, n = n_top;
#pragma unroll 1
    for (int look = at_once ? 1 : 0; look < 2; ++look) {
        if (look == 1) {
            float low = -INFINITY;
            if (!at_once) {
                for (uint32_t t = tid; t < n_top; t += nt) atomicMin(&s_low, (unsigned long long)s_key[t]);
                __syncthreads();
                low = nextafterf((float)(unordered((uint64_t)s_low) - 1.0001 * (double)eps), -INFINITY);
            }
            n = gather_back(low);
        }
        rescore(done, n);
        done = n;
        __syncthreads();
    }
    // 4. many: only those that pass a bucket cut over the high halves can be among the k best
    BucketCut bc;
    bc.lo = 0u; bc.scale = 0.f; bc.cut = 0u; bc.passing = n;
    if (n > 512) bc = block_bucket_cut([&](uint32_t i) { return (uint32_t)(s_key[i] >> 32); }, n, k, hist, red);
    // 5. rank by counting, nearest first; a score that several survivors have is left to step 6
    auto id_at = [&](uint32_t i) { return a.ids ? a.ids[s_row[i]] : (int64_t)s_row[i]; };
    auto put = [&](uint32_t rank, int64_t id, double key) { o_id[rank] = id; o_dist[rank] = (float)(a.metric == 0 ? key : -key); };
    // masses of equal scores pass every cut: those that hold the k-th place are counted by the first
    // of them only
    const bool mass = n > 512 && bc.passing > 512;
#pragma unroll 1
    for (uint32_t t0 = 0; t0 < n; t0 += nt / 8) {
        const uint32_t t = t0 + (uint32_t)tid / 8;
        const uint32_t edge_n = s_edge_n, edge_above = s_edge_above;
        const uint64_t edge_key = s_edge_key;
        if (mass) __syncthreads();
        if (t < n) {
            const uint64_t me = s_key[t];
            uint32_t above = k, equal = 0;
            if (bc.pass((uint32_t)(me >> 32))) {
                if (mass && edge_n != 0 && me == edge_key) { above = edge_above; equal = edge_n; }
                else count_above(s_key, n, me, sub8, above, equal);
            }
            if (sub8 == 0) {
                s_tie[t] = above < k && equal > 1 ? (uint16_t)above : kNoTie;
                if (above < k && equal == 1) put(above, id_at(t), unordered(me));
                if (above < k && equal > 1) {
                    s_ties = 1;
                    o_key[above] = me;
                    if (above + equal > k) { s_edge_key = me; s_edge_above = above; s_edge_n = equal; }
                }
            }
        }
        if (mass) __syncthreads();
    }
    __syncthreads();
    // 6. ties by smaller id.  Survivors of one score have the same number above them, which takes the
    //    place of the score, so that the ids fit LDS in the place of the scores.  More than 512 on the
    //    edge of the k best are cut by their ids first.  (32 queries with 1000 and 3500 copies of the
    //    best row, the whole call with k 10: 0.21 and 0.47 ms; each of them asking every survivor of its
    //    score for its id from memory took 1.6 and 15.9.)
    if (__builtin_expect(s_ties != 0, 0)) {
        const uint32_t edge_n = s_edge_n, edge_above = s_edge_above;
#pragma unroll 1
        for (uint32_t i0 = 0; i0 < n; i0 += 4 * nt) {
            int64_t id[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) id[u] = id_at(min(i0 + (uint32_t)(u * nt + tid), n - 1));
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t i = i0 + (uint32_t)(u * nt + tid);
                if (i < n && s_tie[i] != kNoTie) {
                    s_key[i] = (uint64_t)id[u];
                    if (edge_n > 512 && s_tie[i] == edge_above) atomicMax(&s_top_id, (unsigned long long)id[u]);
                }
            }
        }
        __syncthreads();
        const int bits = 64 - __clzll((long long)s_top_id), shift = max(bits - 31, 0);
        auto level = [&](uint32_t i) -> uint32_t { return s_tie[i] == edge_above ? 0x80000000u - (uint32_t)(s_key[i] >> shift) : 0u; };
        if (edge_n > 512) bc = block_bucket_cut(level, n, k - edge_above, hist, red);
#pragma unroll 1
        for (uint32_t t = (uint32_t)tid / 8; t < n; t += nt / 8) {
            const uint32_t tie = s_tie[t];
            if (tie == kNoTie || (edge_n > 512 && tie == edge_above && !bc.pass(level(t)))) continue;
            const uint64_t id = s_key[t];
            uint32_t ahead = 0;
#pragma unroll 1
            for (uint32_t j0 = sub8; j0 < n; j0 += 32) {
                uint64_t o[4];
                uint32_t w[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) { const uint32_t j = min(j0 + 8u * u, n - 1); o[u] = s_key[j]; w[u] = s_tie[j]; }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t j = j0 + 8u * u;
                    ahead += (uint32_t)((j < n) & (w[u] == tie) & ((o[u] < id) | ((o[u] == id) & (j < t))));
                }
            }
            const uint32_t rank = tie + sum_of_8(ahead);
            if (sub8 == 0 && rank < k) put(rank, (int64_t)id, unordered(o_key[tie]));
        }
    }
    search_again(0u, 0.0);
    __syncthreads();
    // in order: the outputs may be host memory
    for (uint32_t i = tid; i < k; i += nt) {
        a.out_ids[(size_t)qi * k + i] = i < n ? o_id[i] : -1;
        a.out_dists[(size_t)qi * k + i] = i < n ? o_dist[i] : (a.metric == 0 ? -INFINITY : INFINITY);
    }
}

// ---- launch sequence ---------------------------------------------------------------------------------------
int batched_group_q(int dtype) { return dtype == 0 ? kGroupQ32 : kGroupQ; }

int batched_query_stride(int d, int dtype) { return dtype == 0 ? (d + 31) / 32 * 32 : (d + 63) / 64 * 64; }

// LDS of the scan with the queries, thresholds and norms of `slots` queries, beside its staging area (2-byte rows)
static size_t batched_lds_for(int slots, int dq, int dtype) {
    if (dtype == 0) return (size_t)slots * ((size_t)(dq + kQPad32) * 4 + 8);
    return (size_t)slots * ((size_t)(dq + kQPad) * 2 + 8) + (size_t)kBatchWaves * 32 * kStageLd * 2;
}
size_t batched_scan_lds(int d, int dtype) { return batched_lds_for(batched_group_q(dtype), batched_query_stride(d, dtype), dtype); }

// The scan keeps the queries of the whole batch in LDS when they fit and rows are narrow: tasks are then
// short (256 rows of 400 bytes: 3.7 us of streaming), and staging the queries of every group anew, three
// barriers and two trips to memory, is a large part of them: 48 queries x 100 fp32 (287 MB) 69 us with
// groups, 62 so; 106 x 283 fp16 (994 MB) 282, 238; 134 x 46 fp16 (726 MB) 285, 245.  Rows of 1536 and 4096
// bytes lose by it: 32 x 768 fp16 (4.3 GB) 625, 633; 20 x 1024 fp32 (1.9 GB) 308, 316; of 1024 bytes nothing.
constexpr size_t kResidentRowBytes = 1024;
constexpr size_t kScanStaticLds = 512;          // what the scan kernels hold beside that (at most)
static bool queries_resident(const BatchedArgs& a) {
    return (size_t)a.d * (a.dtype == 0 ? 4 : 2) <= kResidentRowBytes && batched_lds_for(a.nq, a.dq, a.dtype) + kScanStaticLds <= a.max_lds;
}

uint64_t batched_task_bound(const int64_t* off_host, int nlist, int nq, int dtype) {
    // every cluster may be probed, by every query
    uint64_t tiles = 0;
    for (int c = 0; c < nlist; ++c) tiles += (uint64_t)((off_host[c + 1] - off_host[c] + kTileRows - 1) / kTileRows);
    const uint64_t gq = (uint64_t)batched_group_q(dtype);
    return tiles * (((uint64_t)nq + gq - 1) / gq) + 1;
}

size_t batched_sample_words(int nq) { return (size_t)nq * kSampleRows; }

typedef void (*BatchedScanFn)(BatchedArgs, int);
template <bool TAIL>
static BatchedScanFn batched_scan_fn_for(int dtype, int metric) {
    if (dtype == 0) return metric == 0 ? batched_scan_f32_kernel<0, TAIL> : batched_scan_f32_kernel<1, TAIL>;
    if (dtype == 1) return metric == 0 ? batched_scan_kernel<F16, 0, TAIL> : batched_scan_kernel<F16, 1, TAIL>;
    return metric == 0 ? batched_scan_kernel<BF16, 0, TAIL> : batched_scan_kernel<BF16, 1, TAIL>;
}
static BatchedScanFn batched_scan_fn(int dtype, int metric, int d) {
    return d % 64 != 0 ? batched_scan_fn_for<true>(dtype, metric) : batched_scan_fn_for<false>(dtype, metric);
}

int batched_resident_grid(int dtype, int metric, int d, int n_cu) {
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)batched_scan_fn(dtype, metric, d), kBatchThreads,
                                                                batched_scan_lds(d, dtype));
    if (e != hipSuccess || per_cu < 1) per_cu = 1;
    if (per_cu > 4) per_cu = 4;
    return per_cu * n_cu;
}

// rounding of an fp32 sum made like the threshold sample's: terms per lane, six additions across
// the lanes, and for L2 the rounded difference and its square
float batched_sample_coef(int d, int dtype, int metric) {
    const int epl = dtype == 0 ? 4 : 8;
    const int chunks = (d + epl - 1) / epl;
    const int terms = epl * ((chunks + 63) / 64) + 6 + (metric != 0 ? 3 : 0);
    return 1.05f * (float)(terms + 2) * 0x1p-24f;
}

hipError_t launch_batched(const BatchedArgs& a, int grid, hipStream_t s, hipEvent_t scan_start, hipEvent_t scan_stop, bool with_merge) {
    const size_t front_lds = std::max((size_t)a.d * 4, a.nlist <= kMapLdsLists ? ((size_t)a.nlist + 1) * 4 : (size_t)0);
    const int parts = sample_parts(a.nq), counted = map_counted_before(a.nlist, a.nq, a.nprobe);
    if (counted) {
        hipLaunchKernelGGL(clear_counts_kernel, dim3((unsigned)(a.nlist + 255) / 256), dim3(256), 0, s, a);
        hipLaunchKernelGGL(count_pairs_kernel, dim3((unsigned)(((uint64_t)a.nq * (uint64_t)a.nprobe + 255) / 256)), dim3(256), 0, s, a);
    }
    const dim3 front(1 + (unsigned)a.nq * (unsigned)(parts + 1)), tasks((unsigned)a.nq + (unsigned)std::min((a.nlist + 3) / 4, 1024));
    typedef void (*FrontFn)(BatchedArgs, int, int);
    const bool tail = a.d % (a.dtype == 0 ? 4 : 8) != 0;
    const FrontFn front_fn = a.dtype == 0 ? (tail ? (FrontFn)batch_front_kernel<F32, true> : (FrontFn)batch_front_kernel<F32, false>)
                           : a.dtype == 1 ? (tail ? (FrontFn)batch_front_kernel<F16, true> : (FrontFn)batch_front_kernel<F16, false>)
                                          : (tail ? (FrontFn)batch_front_kernel<BF16, true> : (FrontFn)batch_front_kernel<BF16, false>);
    hipLaunchKernelGGL(front_fn, front, dim3(kFrontThreads), front_lds, s, a, parts, counted);
    hipLaunchKernelGGL(batch_tasks_kernel, tasks, dim3(256), 0, s, a);
    const BatchedScanFn scan = batched_scan_fn(a.dtype, a.metric, a.d);
    const int resident = queries_resident(a) ? 1 : 0;
    const size_t scan_lds = resident ? batched_lds_for(a.nq, a.dq, a.dtype) : batched_scan_lds(a.d, a.dtype);
    IVF_LAUNCH(scan, dim3(grid), dim3(kBatchThreads), scan_lds, s, scan_start, scan_stop, a, resident);
    if (with_merge) hipLaunchKernelGGL(batched_merge_kernel, dim3(a.nq), dim3(kSelectThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace ivf
