// HIP kernels of the IVF search path for gfx950 (wave64): coarse scoring, top-nprobe
// selection, list scan with per-workgroup top-k', and the fp64 re-score + merge.
// The operations are those of TeleRAG (arxiv 2502.20969) App. B: coarse search over the
// centroids, fine search over the rows of the selected clusters, k nearest by a sort.
#include "ivf_device.h"
#include "../../include/ivf.h"
#include <hip/hip_ext.h>
#include <algorithm>
#include <type_traits>

namespace ivf {
using namespace dev;

// =============================================================================================
// Coarse scoring (App. B, first step): scores[q][j] = d(x_q, c_j) for every centroid, in fp64
// (products of fp32 values are exact in fp64, so the selection below sees the same order as a
// plain fp64 loop up to the last bits of the sums).
//
// Few queries: one wavefront per centroid row, all loads of a row and of the query requested
// at once; HBM-bound on the nlist*d*4 bytes of the centroid matrix, in practice one memory
// latency.  A batch of queries: a dense contraction Q x C^T on the fp64 matrix cores.
// =============================================================================================
// Sums per pair of query and centroid, by the vector units; measured against the matrix cores (us; the row kernel
// walked the queries one after the other then): 3
// queries x 4096 x 768 7.4 / 6.2, x 1024 x 768 5.2 / 5.9, x 1024 x 2048 7.5 / 10.4, x 32768 x 1024 41 / 35;
// 4 x 1024 x 768 6.4 / 6.2, x 1024 x 2048 9.2 / 10.4; 5 x 1024 x 2048 10.8 / 10.4; 8 x 4096 x 768 15 / 6.4.  So
// it takes 3 and 4 queries of few centroids and wide rows (a wavefront of the matrix kernel then has a
// longer chain), and always one or two.  Squared L2 keeps the direct sum of squared differences up to 15 queries, and
// for any number when d is no multiple of 4 (the matrix cores need the three norms form, which is less exact
// where distances are small).
static bool coarse_by_rows(const CoarseArgs& a) {
    if (a.metric != 0) return a.nq < 16 || (a.d & 3) != 0;
    return a.nq < 3 || (a.nq <= 4 && a.nq * 256 <= a.d && a.nlist <= 2048);
}
// queries per wavefront of the row kernel (at most 65535 workgroups side by side in the grid's second direction)
constexpr int kCoarseRowWaves = 8192;
static int coarse_rows_queries(const CoarseArgs& a) {
    const int64_t per = std::max(((int64_t)a.nq * a.nlist + kCoarseRowWaves - 1) / kCoarseRowWaves, ((int64_t)a.nq + 65534) / 65535);
    return (int)std::min<int64_t>(per, a.nq);
}
// From this many pairs on the row kernel's batches go four by four (coarse_pairs_kernel).  Squared L2, us, one pair at a
// time / four by four: 8 queries x 1000 x 100 5.1 / 5.2, 15 x 300 x 64 4.3 / 5.4, 15 x 1024 x 768 9.0 / 8.2, 4 x 4096 x
// 768 8.7 / 7.9, 143 x 307 x 265 17.8 / 14.3, 36 x 1740 x 42 17.4 / 8.8, 37 x 3819 x 158 38 / 17, 4 x 65536 x 65
// 57 / 23, 256 x 8192 x 747 785 / 356.
constexpr int64_t kPairsMin = 12288;
constexpr int kPairTile = 4;
constexpr int64_t kCoarsePairWgs = 2048;         // workgroups of that kernel; more pairs make their walks longer
// (inner products that come here are at most 4 queries of 2048 centroids)
static bool coarse_in_pairs(const CoarseArgs& a) { return a.metric != 0 && a.d >= 4 && a.nq >= 3 && (int64_t)a.nq * a.nlist >= kPairsMin; }

// RAGGED: d is no multiple of 4, rows start at any element.
// A wavefront takes one centroid for `per` queries, one after the other: as few as still make no more
// wavefronts than the chip holds at once.  What bounds it is the length of that chain.
template <bool RAGGED>
__global__ __launch_bounds__(256) void coarse_rows_kernel(CoarseArgs a, int per) {
    const int lane = lane_id(), wave = wave_id();
    const int row = blockIdx.x * 4 + wave;
    if (row >= a.nlist) return;
    const float* c = a.centroids + (size_t)row * a.d;
#pragma unroll 1
    for (int qi = (int)blockIdx.y * per; qi < min(a.nq, ((int)blockIdx.y + 1) * per); ++qi) {
        const float* q = a.q + (size_t)qi * a.d;
        double acc = 0.0;
        if (!RAGGED || a.d >= 4) {
            // a chunk that the end of the row cuts short is taken from the four elements that end it,
            // less those that the lane before has
#pragma unroll 1
            for (int t0 = lane * 4; t0 < a.d; t0 += 1024) {
                float4 cv[4], qv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int t = min(t0 + u * 256, a.d - 4);
                    cv[u] = RAGGED ? load_float4_any(c + t) : *(const float4*)(c + t);
                    qv[u] = RAGGED ? load_float4_any(q + t) : *(const float4*)(q + t);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (t0 + u * 256 < a.d) {
                        const int skip = RAGGED ? max(t0 + u * 256 - (a.d - 4), 0) : 0;
                        const float ce[4] = {cv[u].x, cv[u].y, cv[u].z, cv[u].w};
                        const float qe[4] = {qv[u].x, qv[u].y, qv[u].z, qv[u].w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const bool out = RAGGED && e < skip;
                            const double x = out ? 0.0 : (double)qe[e], y = out ? 0.0 : (double)ce[e];
                            if (a.metric == 0) acc = fma(x, y, acc);
                            else { const double df = x - y; acc = fma(df, df, acc); }
                        }
                    }
                }
            }
        } else {
            for (int t = lane; t < a.d; t += 64) {
                const double x = (double)q[t], y = (double)c[t];
                if (a.metric == 0) acc = fma(x, y, acc);
                else { const double df = x - y; acc = fma(df, df, acc); }
            }
        }
        const double s = wave_sum(acc);
        if (lane == 0) a.scores[(size_t)qi * a.nlist + row] = s;
    }
}

// The same sums for squared L2, four centroids by four queries to a wavefront: for batches, where one pair at a time is bound by
// the rows' way from the caches (two rows per pair; here half a row) and by the wavefront's sum.  A
// pair's products are added in the order of the row kernel and the lanes' sums by the same
// butterfly, which hands the halves of the sixteen values on as it goes: bit for bit the same scores.
template <bool RAGGED>
__global__ __launch_bounds__(256) void coarse_pairs_kernel(CoarseArgs a, int per) {
    constexpr int T = kPairTile;
    const int lane = lane_id(), c0 = (int)(blockIdx.x * 4 + wave_id()) * T;
    if (c0 >= a.nlist) return;
    const int q_tiles = (a.nq + T - 1) / T;
    const float* crow[T];
#pragma unroll
    for (int i = 0; i < T; ++i) crow[i] = a.centroids + (size_t)min(c0 + i, a.nlist - 1) * a.d;
#pragma unroll 1
    for (int g = (int)blockIdx.y * per; g < min(q_tiles, ((int)blockIdx.y + 1) * per); ++g) {
        const float* qrow[T];
#pragma unroll
        for (int j = 0; j < T; ++j) qrow[j] = a.q + (size_t)min(g * T + j, a.nq - 1) * a.d;
        double acc[T * T];
#pragma unroll
        for (int p = 0; p < T * T; ++p) acc[p] = 0.0;
#pragma unroll 2
        for (int t0 = lane * 4; t0 < a.d; t0 += 256) {
            const int t = RAGGED ? min(t0, a.d - 4) : t0, skip = t0 - t;      // as in the row kernel
            float4 cv[T], qv[T];
#pragma unroll
            for (int i = 0; i < T; ++i) cv[i] = RAGGED ? load_float4_any(crow[i] + t) : *(const float4*)(crow[i] + t);
#pragma unroll
            for (int j = 0; j < T; ++j) qv[j] = RAGGED ? load_float4_any(qrow[j] + t) : *(const float4*)(qrow[j] + t);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool out = RAGGED && e < skip;
                double x[T], y[T];
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    const float ce = e == 0 ? cv[i].x : e == 1 ? cv[i].y : e == 2 ? cv[i].z : cv[i].w;
                    const float qe = e == 0 ? qv[i].x : e == 1 ? qv[i].y : e == 2 ? qv[i].z : qv[i].w;
                    y[i] = out ? 0.0 : (double)ce;
                    x[i] = out ? 0.0 : (double)qe;
                }
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j) {
                        const double df = x[j] - y[i];
                        acc[i * T + j] = fma(df, df, acc[i * T + j]);
                    }
            }
        }
        // lane l ends with pair l / 4
        auto halve = [&](auto size, int m) {
            constexpr int n = decltype(size)::value;
            const bool upper = (lane & m) != 0;
#pragma unroll
            for (int p = 0; p < n; ++p) {
                const double keep = upper ? acc[p + n] : acc[p], give = upper ? acc[p] : acc[p + n];
                acc[p] = keep + __shfl_xor(give, m);
            }
        };
        halve(std::integral_constant<int, 8>{}, 32);
        halve(std::integral_constant<int, 4>{}, 16);
        halve(std::integral_constant<int, 2>{}, 8);
        halve(std::integral_constant<int, 1>{}, 4);
        double s = acc[0];
        s += __shfl_xor(s, 2);
        s += __shfl_xor(s, 1);
        const int i = lane >> 4, j = (lane >> 2) & 3;
        if ((lane & 3) == 0 && c0 + i < a.nlist && g * T + j < a.nq) a.scores[(size_t)(g * T + j) * a.nlist + c0 + i] = s;
    }
}

// Q x C^T with v_mfma_f64_16x16x4_f64.  Operand layout of the instruction: lane l supplies
// A[i = l % 16][k = l / 16] and B[k = l / 16][j = l % 16]; result register r of lane l is
// C[i = 4 r + l / 16][j = l % 16].  The order of the elements inside a dot product is free, so lane
// (row i, part p) loads the 16 bytes p of each 16-element block of its row straight from memory
// and the four values feed four instructions: no LDS on the way in.  A workgroup covers QT * 16
// queries by CT * 16 centroids; its W wavefronts take every W-th 32-element block of the rows (the
// next block in flight while one is multiplied) and their sums are added through LDS, in order.
// Why this split: batches are tens of queries, and what bounds them is the length of the chain
// through the elements, not the matrix cores.  (Tiles of 32 x 128 that walked all elements through
// LDS slabs, a barrier pair per 32: 52.7, 55.5 and 117 us for 16 queries x 1024 x 768, 32 x 4096 x 768
// and 256 x 8192 x 1024; this: 6.1, 10 and 105; the fp64 matrix peak for the last is 55 us.)
// W = 1: a tile is one wavefront's, its sums go straight to memory and no LDS is used.
// RAGGED: d is no multiple of 4, rows start at any element (the row kernel served such batches with
// single elements: 272 and 1120 us for 256 queries x 2678 x 295 and x 8192 x 747; this: 18 and 86).
// Workgroups that follow each other on one XCD share their centroids (blockIdx % 8 is the XCD):
// each L2 then holds one eighth of the centroids instead of all of them.
// For the squared distance the norms are accumulated beside the products: |q - c|^2 = |q|^2 + |c|^2 - 2 q.c.
typedef double double4_t __attribute__((ext_vector_type(4)));
template <int QT, int CT, int W, bool RAGGED>
__global__ __launch_bounds__(W * 64) void coarse_mfma_kernel(CoarseArgs a, int q_tiles) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    typedef double SumTile[QT * CT][4][64];
    SumTile* s_acc = (SumTile*)smem_raw;               // [W]
    double (*s_nq)[QT * 16] = (double (*)[QT * 16])(s_acc + W);
    double (*s_nc)[CT * 16] = (double (*)[CT * 16])(s_nq + W);
    const int lane = lane_id(), wave = wave_id();
    const int xcd = blockIdx.x & 7, in_xcd = blockIdx.x >> 3;
    const int c0 = ((in_xcd / q_tiles) * 8 + xcd) * (CT * 16), q0 = (in_xcd % q_tiles) * (QT * 16);
    if (c0 >= a.nlist) return;
    const int fi = lane & 15, fk = lane >> 4;
    const float* qrow[QT];
    const float* crow[CT];
#pragma unroll
    for (int x = 0; x < QT; ++x) qrow[x] = a.q + (size_t)min(q0 + x * 16 + fi, a.nq - 1) * a.d + fk * 4;
#pragma unroll
    for (int y = 0; y < CT; ++y) crow[y] = a.centroids + (size_t)min(c0 + y * 16 + fi, a.nlist - 1) * a.d + fk * 4;
    double4_t acc[QT][CT];
    double nq2[QT], nc2[CT];
#pragma unroll
    for (int x = 0; x < QT; ++x) {
        nq2[x] = 0.0;
#pragma unroll
        for (int y = 0; y < CT; ++y) acc[x][y] = double4_t{0.0, 0.0, 0.0, 0.0};
    }
#pragma unroll
    for (int y = 0; y < CT; ++y) nc2[y] = 0.0;
    struct Stage { float4 q[2][QT], c[2][CT]; };       // a 32-element block: two 16-element halves
    auto request = [&](int k0, Stage& s) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = k0 + h * 16;
            const int left = a.d - (k + fk * 4);       // elements from this lane's first on
            auto take = [&](const float* p) {
                if (!RAGGED) return left > 0 ? *(const float4*)p : make_float4(0.f, 0.f, 0.f, 0.f);
                if (left >= 4) return load_float4_any(p);
                // the row ends inside the chunk or before it
                return make_float4(left > 0 ? p[0] : 0.f, left > 1 ? p[1] : 0.f, left > 2 ? p[2] : 0.f, 0.f);
            };
#pragma unroll
            for (int x = 0; x < QT; ++x) s.q[h][x] = take(qrow[x] + k);
#pragma unroll
            for (int y = 0; y < CT; ++y) s.c[h][y] = take(crow[y] + k);
        }
    };
    auto multiply = [&](const Stage& s) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double fa[QT], fb[CT];
#pragma unroll
                for (int x = 0; x < QT; ++x) {
                    fa[x] = (double)(e == 0 ? s.q[h][x].x : e == 1 ? s.q[h][x].y : e == 2 ? s.q[h][x].z : s.q[h][x].w);
                    if (a.metric != 0) nq2[x] = fma(fa[x], fa[x], nq2[x]);
                }
#pragma unroll
                for (int y = 0; y < CT; ++y) {
                    fb[y] = (double)(e == 0 ? s.c[h][y].x : e == 1 ? s.c[h][y].y : e == 2 ? s.c[h][y].z : s.c[h][y].w);
                    if (a.metric != 0) nc2[y] = fma(fb[y], fb[y], nc2[y]);
                }
#pragma unroll
                for (int x = 0; x < QT; ++x)
#pragma unroll
                    for (int y = 0; y < CT; ++y)
                        acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[x], fb[y], acc[x][y], 0, 0, 0);
            }
        }
    };
    Stage st[2];
    const int step = W * 32;
    int k = wave * 32;
    if (k < a.d) request(k, st[0]);
#pragma unroll 1
    for (; k < a.d; k += 2 * step) {
        if (k + step < a.d) request(k + step, st[1]);
        multiply(st[0]);
        if (k + step >= a.d) break;
        if (k + 2 * step < a.d) request(k + 2 * step, st[0]);
        multiply(st[1]);
    }
    if (W == 1) {
#pragma unroll
        for (int y = 0; y < CT; ++y) if (a.metric != 0) { nc2[y] += __shfl_xor(nc2[y], 16); nc2[y] += __shfl_xor(nc2[y], 32); }
#pragma unroll
        for (int x = 0; x < QT; ++x) {
            if (a.metric != 0) { nq2[x] += __shfl_xor(nq2[x], 16); nq2[x] += __shfl_xor(nq2[x], 32); }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = x * 16 + 4 * r + fk;
                const double qn = a.metric != 0 ? __shfl(nq2[x], 4 * r + fk) : 0.0;
#pragma unroll
                for (int y = 0; y < CT; ++y) {
                    const int j = y * 16 + fi;
                    const double s = a.metric != 0 ? fma(-2.0, acc[x][y][r], qn + nc2[y]) : acc[x][y][r];
                    if (q0 + i < a.nq && c0 + j < a.nlist) a.scores[(size_t)(q0 + i) * a.nlist + c0 + j] = s;
                }
            }
        }
        return;
    }
    // the wavefronts' sums, added in order
#pragma unroll
    for (int x = 0; x < QT; ++x)
#pragma unroll
        for (int y = 0; y < CT; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) s_acc[wave][x * CT + y][r][lane] = acc[x][y][r];
    if (a.metric != 0) {
        // over the four parts of a row; then lane l < 16 holds the norm of row l
#pragma unroll
        for (int x = 0; x < QT; ++x) {
            nq2[x] += __shfl_xor(nq2[x], 16); nq2[x] += __shfl_xor(nq2[x], 32);
            if (lane < 16) s_nq[wave][x * 16 + lane] = nq2[x];
        }
#pragma unroll
        for (int y = 0; y < CT; ++y) {
            nc2[y] += __shfl_xor(nc2[y], 16); nc2[y] += __shfl_xor(nc2[y], 32);
            if (lane < 16) s_nc[wave][y * 16 + lane] = nc2[y];
        }
    }
    __syncthreads();
    // result registers (tile, r) of the workgroup, dealt to the wavefronts
#pragma unroll
    for (int n0 = 0; n0 < QT * CT * 4; n0 += W) {
        const int n = n0 + wave, t = n >> 2, r = n & 3, x = t / CT, y = t % CT;
        if (n >= QT * CT * 4) break;
        double s = s_acc[0][t][r][lane];
#pragma unroll
        for (int w = 1; w < W; ++w) s += s_acc[w][t][r][lane];
        const int i = x * 16 + 4 * r + fk, j = y * 16 + fi;
        if (a.metric != 0) {
            double qn = s_nq[0][i], cn = s_nc[0][j];
#pragma unroll
            for (int w = 1; w < W; ++w) { qn += s_nq[w][i]; cn += s_nc[w][j]; }
            s = fma(-2.0, s, qn + cn);
        }
        if (q0 + i < a.nq && c0 + j < a.nlist) a.scores[(size_t)(q0 + i) * a.nlist + c0 + j] = s;
    }
}

template <int QT, int CT, int W>
static void launch_coarse_mfma(const CoarseArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const int q_tiles = (a.nq + QT * 16 - 1) / (QT * 16), c_tiles = (a.nlist + CT * 16 - 1) / (CT * 16);
    const size_t lds = W == 1 ? 0 : (size_t)W * (QT * CT * 4 * 64 + QT * 16 + CT * 16) * sizeof(double);
    const dim3 grid((unsigned)((c_tiles + 7) / 8 * 8 * q_tiles));
    if (a.d & 3) IVF_LAUNCH((coarse_mfma_kernel<QT, CT, W, true>), grid, dim3(W * 64), lds, s, e0, e1, a, q_tiles);
    else IVF_LAUNCH((coarse_mfma_kernel<QT, CT, W, false>), grid, dim3(W * 64), lds, s, e0, e1, a, q_tiles);
}

hipError_t launch_coarse(const CoarseArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (coarse_by_rows(a)) {
        if (coarse_in_pairs(a)) {
            const int c_wgs = (a.nlist + 4 * kPairTile - 1) / (4 * kPairTile), q_tiles = (a.nq + kPairTile - 1) / kPairTile;
            const int per = (int)std::min<int64_t>(std::max<int64_t>(((int64_t)q_tiles * c_wgs + kCoarsePairWgs - 1) / kCoarsePairWgs, (q_tiles + 65534) / 65535), q_tiles);
            const dim3 grid((unsigned)c_wgs, (unsigned)((q_tiles + per - 1) / per));
            if (a.d & 3) IVF_LAUNCH(coarse_pairs_kernel<true>, grid, dim3(256), 0, s, e0, e1, a, per);
            else IVF_LAUNCH(coarse_pairs_kernel<false>, grid, dim3(256), 0, s, e0, e1, a, per);
            return hipGetLastError();
        }
        const int per = coarse_rows_queries(a);
        const dim3 grid((unsigned)(a.nlist + 3) / 4, (unsigned)((a.nq + per - 1) / per));
        if (a.d & 3) IVF_LAUNCH(coarse_rows_kernel<true>, grid, dim3(256), 0, s, e0, e1, a, per);
        else IVF_LAUNCH(coarse_rows_kernel<false>, grid, dim3(256), 0, s, e0, e1, a, per);
    } else {
        // Small tiles while they leave the chip short of work, measured with 1024, 4096 and 8192 lists:
        // 512 of them 12.9, 12.6, 14.3 us against 15.7, 16.1, 19.1 of the large ones; 768: 16.0 against
        // 17.0; 1024: 19.3, 19.2, 22.5 against 17.0, 17.0, 19.5; 8192 (256 x 8192 x 768): 107 against 81.  And for any number of
        // lists when the queries fit one of them (4 queries x 65536 x 64, 128, 768: 11.5, 14.6, 51 us against
        // 14.2, 18.2, 76).
        // Large ones: split over four wavefronts while the chain counts.  One wavefront per tile when
        // there are more than eight tiles per compute unit, or half of the four had no elements (256 queries x
        // 16384 x 64, 65536 x 64, 16384 x 256, 65536 x 768: 26, 66, 58, 552 us against 31, 94, 64, 593; 2048
        // tiles of 256 x 8192 x 768 85 against 81, but x 64 17.8 against 20.2).
        const size_t small_tiles = (size_t)((a.nlist + 15) / 16) * ((a.nq + 15) / 16);
        const size_t large_tiles = (size_t)((a.nlist + 31) / 32) * ((a.nq + 31) / 32);
        if (small_tiles <= 768 || a.nq <= 16) launch_coarse_mfma<1, 1, 8>(a, s, e0, e1);
        else if (large_tiles > 2048 || (a.d <= 64 && large_tiles >= 1024)) launch_coarse_mfma<2, 2, 1>(a, s, e0, e1);
        else launch_coarse_mfma<2, 2, 4>(a, s, e0, e1);
    }
    return hipGetLastError();
}

// =============================================================================================
// Top-nprobe selection (App. B: the L nearest centroids), ordered nearest first with ties by
// smaller cluster index, plus the tables the scan walks: per selected cluster ("slot") its
// placement and rows, and per scan workgroup its share of the rows.  One workgroup per query.
// =============================================================================================
__device__ __forceinline__ uint64_t coarse_key(double score, int metric) {
    uint64_t o = ordered(score);
    return metric == 0 ? ~o : o;       // ascending key = nearest first
}

// Fills keys/idx (LDS or global, `pad` entries) with the nprobe best (key, index) pairs sorted
// ascending.  Inlined once per memory kind so that LDS accesses compile to LDS instructions.
__device__ __forceinline__ void select_sorted(const SelectArgs& a, const double* sc, uint64_t* keys,
                                              uint32_t* idx, uint32_t pad, uint32_t* hist, uint32_t* sh) {
    const int tid = threadIdx.x, nt = blockDim.x;
    const uint32_t nlist = a.nlist, nprobe = a.nprobe;
    if (nlist <= pad) {
        // every centroid fits the sort: no selection pass needed
        for (uint32_t i = tid; i < pad; i += nt) {
            keys[i] = i < nlist ? coarse_key(sc[i], a.metric) : ~0ull;
            idx[i] = i < nlist ? i : 0xFFFFFFFFu;
        }
        __syncthreads();
    } else {
        // radix-select the nprobe best, then sort only those
        uint64_t mask, prefix; uint32_t need, group;
        auto key_at = [&](uint32_t i) { return coarse_key(sc[i], a.metric); };
        block_radix_select<uint64_t>(key_at, nlist, nprobe, hist, sh, mask, prefix, need, group);
        if (tid == 0) sh[4] = 0;
        for (uint32_t i = tid; i < pad; i += nt) { keys[i] = ~0ull; idx[i] = 0xFFFFFFFFu; }
        __syncthreads();
        const bool take_group = need == group;
        for (uint32_t i = tid; i < nlist; i += nt) {
            uint64_t k = key_at(i);
            uint64_t hi = k & mask;
            if (hi < prefix || (take_group && hi == prefix)) {
                uint32_t p = atomicAdd(&sh[4], 1u);
                keys[p] = k; idx[p] = i;
            }
        }
        __syncthreads();
        if (!take_group) {
            // the boundary group holds fully equal scores: keep the `need` smallest indices.
            // Entries are visited in index order by one wavefront so the choice is ordered.
            if (tid < 64) {
                uint32_t taken = 0;
                for (uint32_t base = 0; base < nlist && taken < need; base += 64) {
                    uint32_t i = base + tid;
                    bool tie = i < nlist && (key_at(i) & mask) == prefix;
                    uint64_t b = __ballot(tie);
                    uint32_t rank = taken + __popcll(b & ((1ull << tid) - 1ull));
                    if (tie && rank < need) {
                        uint32_t p = sh[4] + rank;
                        keys[p] = key_at(i); idx[p] = i;
                    }
                    taken += __popcll(b);
                }
            }
            __syncthreads();
        }
    }
    block_bitonic_sort(keys, idx, pad);
}

// ---- up to 64 clusters of up to four per thread -----------------------------------------------------
// The order is (key, index) with key = the order-preserving image of the 64-bit score, larger = nearer, equal keys by smaller
// index.  Clusters are dealt to 64 groups by their numbers (128 when more than 32 are wanted); T, the largest of the
// maxima's high words that at least nprobe of them reach, lets at least nprobe candidates pass and, with groups
// unrelated to the scores, about nprobe (1 + nprobe / 128) of them.  Those are pooled, and each finds its rank by
// ballots over the pool: exact, whatever ties there are.
// What bounds it: two trips to memory and the instructions of one workgroup.  Ranks by ballots are dealt to the
// wavefronts, where a sorting network is one wavefront's chain (a kernel of its own, us, before / now: 8 of 64 clusters
// 5.4 / 4.2, 32 of 1024 5.9 / 4.9; a search that selects 64 of 4096 whose best are all in one of eight groups 60 / 26).
constexpr int kFewPerThread = 4;
constexpr int kFewThreads = 256;         // up to 1024 clusters; more: kSelectThreads
struct FewLds {
    uint32_t red[128];
    uint32_t n, cut, above, pad;
    uint32_t pick[64];           // the selected clusters, nearest first
    // behind it: uint64_t key[NT * kFewPerThread], uint32_t idx[NT * kFewPerThread]
};
static size_t few_lds(int threads) { return sizeof(FewLds) + (size_t)threads * kFewPerThread * 12; }

// Leaves the clusters in L.pick[0 .. nprobe - 1]; all threads of the workgroup (NT) call it, nprobe <= min(64, nlist) and
// nlist <= NT * kFewPerThread.
template <int NT>
__device__ __forceinline__ void select_few(const double* sc, int nlist, int nprobe, int metric, FewLds& L) {
    constexpr int C = kFewPerThread, NW = NT / 64, G = NT / 128;       // G lanes hold one of 128 groups
    uint64_t* pkey = (uint64_t*)(&L + 1);
    uint32_t* pidx = (uint32_t*)(pkey + NT * C);
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    // cluster c belongs to group c % 128: scores that rise or fall with the number, or come in runs, spread over the groups
    const int first = (tid & (G - 1)) * 128 + tid / G;
    double v[C];
#pragma unroll
    for (int j = 0; j < C; ++j) v[j] = sc[min(first + j * NT, nlist - 1)];
    if (tid == 0) { L.n = 0; L.cut = 0; L.above = 0; }
    uint64_t key[C];
    uint32_t idx[C];
#pragma unroll
    for (int j = 0; j < C; ++j) { key[j] = ~coarse_key(v[j], metric); idx[j] = (uint32_t)(first + j * NT); }
    // T for the words of those in `active` (bit j: candidate j of the thread) and `want` of them
    auto cut_of = [&](const uint32_t (&word)[C], uint32_t active, int want) __attribute__((always_inline)) -> uint32_t {
        uint32_t best = 0;
#pragma unroll
        for (int j = 0; j < C; ++j) if ((active >> j) & 1u) best = max(best, word[j]);
        if (G >= 2) best = max(best, xor_lane_u32<1>(best));
        if (G >= 4) best = max(best, xor_lane_u32<2>(best));
        if (G >= 8) best = max(best, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)best, 0x141, 0xF, 0xF, true));      // row_half_mirror
        if ((lane & (G - 1)) == 0) L.red[tid / G] = best;
        __syncthreads();
        uint32_t g0 = L.red[2 * lane], g1 = L.red[2 * lane + 1];
        const bool fine = want > 32;                 // all 128 groups; else two of them together
        if (!fine) { g0 = max(g0, g1); g1 = 0; }
        uint32_t t = 0;
#pragma unroll
        for (int i = 0; i < 64 / NW; ++i) {
            const uint32_t u = read_lane(g0, wave * (64 / NW) + i);
            int reach = __popcll(__ballot(g0 >= u));
            if (fine) {
                const uint32_t w = read_lane(g1, wave * (64 / NW) + i);
                reach += __popcll(__ballot(g1 >= u));
                const int reach1 = __popcll(__ballot(g0 >= w)) + __popcll(__ballot(g1 >= w));
                t = reach1 >= want ? max(t, w) : t;
            }
            t = reach >= want ? max(t, u) : t;
        }
        if (lane == 0 && t) atomicMax(&L.cut, t);
        __syncthreads();
        return L.cut;                                // 0: fewer than `want` groups hold anything, all pass
    };
    auto pool = [&](uint32_t which) __attribute__((always_inline)) {
        uint64_t b[C];
        uint32_t n = 0;
#pragma unroll
        for (int j = 0; j < C; ++j) { b[j] = __ballot((which >> j) & 1u); n += (uint32_t)__popcll(b[j]); }
        if (n) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&L.n, n);
            base = read_lane(base, 0);
            const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
            for (int j = 0; j < C; ++j) {
                const uint32_t pos = base + __popcll(b[j] & below);
                if ((b[j] >> lane) & 1u) { pkey[pos] = key[j]; pidx[pos] = idx[j]; }
                base += (uint32_t)__popcll(b[j]);
            }
        }
        __syncthreads();
        return (int)L.n;
    };
    uint32_t active = 0, taken = 0;
    uint32_t word[C];
#pragma unroll
    for (int j = 0; j < C; ++j) { word[j] = (uint32_t)(key[j] >> 32); active |= first + j * NT < nlist ? 1u << j : 0u; }
    int want = nprobe;
    uint32_t cut = cut_of(word, active, want);
    auto passing = [&]() __attribute__((always_inline)) {
        uint32_t m = 0;
#pragma unroll
        for (int j = 0; j < C; ++j) m |= word[j] >= cut ? 1u << j : 0u;
        return (m & active) | taken;
    };
    int cnt = pool(passing());                       // at least nprobe
#pragma unroll 1
    for (int round = 0, level = 0; __builtin_expect(cnt > 128 && round < 5, 0); ++round) {
        // Many.  Those above the cut word are in, when they are fewer than wanted (masses of scores with the same high
        // word, as of a query of zeros); of those with the cut word the low words decide, then the numbers of the clusters.
        // Else only those above it matter (scores that run with the groups): they are dealt anew, in the order of the pool.
        uint32_t over = 0, same = 0;
#pragma unroll
        for (int j = 0; j < C; ++j) {
            if ((active >> j) & 1u) { over |= word[j] > cut ? 1u << j : 0u; same |= word[j] == cut ? 1u << j : 0u; }
        }
        const uint32_t mine = (uint32_t)__popc(over);
        if (mine) atomicAdd(&L.above, mine);
        __syncthreads();
        const int above = (int)L.above;
        __syncthreads();
        if (tid == 0) { L.n = 0; L.cut = 0; L.above = 0; }
        __syncthreads();
        if (above >= want) {
            cnt = pool(over | taken);
            active = 0;
#pragma unroll
            for (int j = 0; j < C; ++j) {
                const int at = first + j * NT;
                if (at < cnt) { key[j] = pkey[at]; idx[j] = pidx[at]; active |= 1u << j; }
            }
            taken = 0; want = nprobe; level = 0;
            __syncthreads();
            if (tid == 0) L.n = 0;
        } else {
            want -= above;
            taken |= over;
            active = same;
            ++level;
        }
#pragma unroll
        for (int j = 0; j < C; ++j) word[j] = level == 0 ? (uint32_t)(key[j] >> 32) : level == 1 ? (uint32_t)key[j] : ~idx[j];
        cut = cut_of(word, active, want);
        cnt = pool(passing());
    }
    if (__builtin_expect(cnt <= 128, 1)) {
        // (places past the end: below every score, behind every index)
        const uint64_t k0 = lane < cnt ? pkey[lane] : 0, k1 = lane + 64 < cnt ? pkey[lane + 64] : 0;
        const uint32_t i0 = lane < cnt ? pidx[lane] : ~0u, i1 = lane + 64 < cnt ? pidx[lane + 64] : ~0u;
        auto rank_of = [&](uint64_t k, uint32_t i) __attribute__((always_inline)) {
            int rank = __popcll(__ballot(k0 > k));
            uint64_t e0 = __ballot(k0 == k), e1 = 0;
            if (cnt > 64) { rank += __popcll(__ballot(k1 > k)); e1 = __ballot(k1 == k); }
            if (__builtin_expect(__popcll(e0) + __popcll(e1) > 1, 0)) rank += __popcll(__ballot(k0 == k && i0 < i)) + __popcll(__ballot(k1 == k && i1 < i));
            if (rank < nprobe && lane == 0) L.pick[rank] = i;
        };
#pragma unroll 1
        for (int j = wave; j < min(cnt, 64); j += NW) rank_of(read_lane(k0, j), read_lane(i0, j));
#pragma unroll 1
        for (int j = 64 + wave; j < cnt; j += NW) rank_of(read_lane(k1, j - 64), read_lane(i1, j - 64));
    } else {
        // (scores that five cuts did not thin out)
#pragma unroll 1
        for (int t = tid; t < cnt; t += NT) {
            const uint64_t k = pkey[t];
            const uint32_t i = pidx[t];
            int rank = 0;
#pragma unroll 1
            for (int j0 = 0; j0 < cnt && rank < nprobe; j0 += 8) {
                uint64_t o[8];
                uint32_t w[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) { o[u] = pkey[min(j0 + u, cnt - 1)]; w[u] = pidx[min(j0 + u, cnt - 1)]; }
#pragma unroll
                for (int u = 0; u < 8; ++u) rank += (int)((j0 + u < cnt) & ((o[u] > k) | ((o[u] == k) & (w[u] < i))));
            }
            if (rank < nprobe) L.pick[rank] = i;
        }
    }
    __syncthreads();
}

// Inclusive sum over the lanes of a wavefront.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);        // row_shr:1, 2, 4, 8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);       // row_bcast:15 into rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);       // row_bcast:31 into rows 2 and 3
    return v;
}

// The slot table of a query that selected up to 64 clusters, one slot per lane (L.pick), by one wavefront.
struct LaneSlot { uint32_t cluster, grow, nrows, end; int64_t base; };     // end: rows of the resident slots up to and with this one
__device__ __forceinline__ LaneSlot slot_of_lane(const FewLds& L, int nprobe, const int64_t* off, const int64_t* res_off) {
    LaneSlot s;
    const int lane = lane_id();
    s.cluster = L.pick[min(lane, nprobe - 1)];
    const int64_t lo = off[s.cluster], hi = off[s.cluster + 1];
    s.base = res_off[s.cluster];
    s.grow = (uint32_t)lo;
    s.nrows = (uint32_t)(hi - lo);
    s.end = wave_prefix(lane < nprobe && s.base >= 0 ? s.nrows : 0u);
    return s;
}
// ... written where the merge, the second pass and the caller look for it.
__device__ __forceinline__ void store_slots(const LaneSlot& s, int nprobe, int qi, const SlotTables& slots, int32_t* probe, uint32_t* used,
                                            unsigned long long* rows_counter) {
    const int lane = lane_id();
    if (lane < nprobe) {
        const size_t o = (size_t)qi * nprobe + lane;
        probe[o] = (int32_t)s.cluster;
        slots.base[o] = s.base;
        slots.grow[o] = s.grow;
        slots.nrows[o] = s.nrows;
        slots.rprefix[o + qi + 1] = s.end;
        if (used && s.base >= 0) used[s.cluster] = 1u;            // cache bookkeeping: resident and selected
    }
    if (lane == 0) slots.rprefix[(size_t)qi * (nprobe + 1)] = 0u;
    if (rows_counter && lane == 63) atomicAdd(rows_counter, (unsigned long long)s.end);
}

template <int NT>
__global__ __launch_bounds__(NT) void select_few_kernel(SelectArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    FewLds& L = *(FewLds*)smem_raw;
    select_few<NT>(a.scores + (size_t)blockIdx.x * a.nlist, a.nlist, a.nprobe, a.metric, L);
    if (wave_id() == 0) store_slots(slot_of_lane(L, a.nprobe, a.off, a.res_off), a.nprobe, (int)blockIdx.x, a.slots, a.probe, a.used, a.rows_counter);
}
// up to 64 of up to 4096 clusters
static bool selects_few(int nlist, int nprobe) { return nprobe <= 64 && nlist <= kSelectThreads * kFewPerThread; }

// The nprobe nearest by packed candidates (top 40 bits of the descending key image, complement of
// the cluster index: larger = nearer).  The candidates are dealt to the threads; a bucket cut over
// the threads' best lets at least nprobe of those pass, so at least nprobe candidates do, and, with
// 8 candidates per thread and half the threads' best wanted, about a third more than that.  Those are
// pooled, sorted in runs of 64 by the wavefronts (registers only), and each finds its place by a
// binary search in every run.  The order of the prefixes is the order of the scores wherever
// prefixes differ; where they tie among the selected clusters or across the cut, the pooled
// candidates of one prefix are ordered by the low bits of their keys.  When more pass than the pool
// holds, or a score is no number or infinite, the result is not used: returns false (for the
// whole workgroup), idx is then undefined.  Bound by barriers and dependent LDS reads of one workgroup.
// (Ranking the pool by counting on 64-bit keys, with the histogram taken over all scores: 18, 31 and
// 95 us for 8 queries of 2048 lists with nprobe 128, 32 of 4096 with 128 and 256 of 8192 with 512;
// this: 11, 12 and 24.  With two equal scores among the selected, one query of 1000, 4096 and 8192
// lists with nprobe 100, 128 and 512: 13, 14 and 22 us, and 24, 31 and 54 when ties went to the exact
// path.  256 queries of 65536 lists with nprobe 512: 63 us, 225 with their scores read one by one.)
constexpr int kSelectPoolCap = 2048;
__device__ __forceinline__ bool select_pooled(const SelectArgs& a, const double* sc, uint32_t* idx, Cand* pool, Cand* in_order,
                                              uint32_t* hist, uint32_t* red, uint32_t* sh) {
    const int tid = threadIdx.x, nt = blockDim.x, lane = lane_id(), wave = wave_id();
    const uint32_t nprobe = a.nprobe;
    auto packed = [&](int i, double s) {
        return (~coarse_key(s, a.metric) & ~0xFFFFFFull) | (uint64_t)(0xFFFFFFu - (uint32_t)i);
    };
    // the first eight scores of a thread are requested together and stay in registers
    constexpr int C = 8;
    double s8[C];
#pragma unroll
    for (int j = 0; j < C; ++j) s8[j] = sc[min(tid + j * nt, a.nlist - 1)];
    if (tid == 0) { sh[4] = 0; sh[6] = 0; }
    auto nearness = [&](double s) { return (float)(a.metric == 0 ? s : -s); };
    // not a number: infinite here, which sends the selection to the exact path
    auto better = [](float b, float f) { return f == f ? fmaxf(b, f) : INFINITY; };
    float best = -INFINITY;
#pragma unroll
    for (int j = 0; j < C; ++j) if (tid + j * nt < a.nlist) best = better(best, nearness(s8[j]));
    // the others four at a time
    constexpr int M = 4;
    auto request = [&](int i0, double (&v)[M]) {
#pragma unroll
        for (int j = 0; j < M; ++j) v[j] = sc[min(i0 + j * nt + tid, a.nlist - 1)];
    };
#pragma unroll 1
    for (int i0 = C * nt; i0 < a.nlist; i0 += M * nt) {
        double v[M];
        request(i0, v);
#pragma unroll
        for (int j = 0; j < M; ++j) if (i0 + j * nt + tid < a.nlist) best = better(best, nearness(v[j]));
    }
    // the cut is taken on scores mapped linearly to integers: bit images of scores around zero leave
    // all the exponents between them to one bucket
    float lo = tid < a.nlist ? best : INFINITY, hi = best;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) { lo = fminf(lo, __shfl_xor(lo, m)); hi = fmaxf(hi, __shfl_xor(hi, m)); }
    float* ends = (float*)red;
    if (lane == 0) { ends[wave] = lo; ends[16 + wave] = hi; }
    __syncthreads();
    for (int w = 0; w < nt >> 6; ++w) { lo = fminf(lo, ends[w]); hi = fmaxf(hi, ends[16 + w]); }
    const float scale = hi > lo ? 4.0e9f / (hi - lo) : 0.f;
    if (!(hi - lo < INFINITY) || !(scale < INFINITY)) return false;       // infinities, or all but equal scores
    auto level = [&](float f) -> uint32_t { return f > lo ? 1u + (uint32_t)((f - lo) * scale) : 1u; };
    __syncthreads();                                    // ends has been read
    const BucketCut bc = block_bucket_cut([&](uint32_t) { return tid < a.nlist ? level(best) : 0u; }, (uint32_t)nt, nprobe, hist, red);
    auto offer = [&](int i, double s) {
        const bool ok = i < a.nlist && bc.pass(level(nearness(s)));
        const uint64_t bal = __ballot(ok);
        if (!bal) return;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&sh[4], (uint32_t)__popcll(bal));
        base = read_lane(base, 0);
        const uint32_t pos = base + __popcll(bal & ((1ull << lane) - 1ull));
        if (ok && pos < (uint32_t)kSelectPoolCap) pool[pos] = packed(i, s);
    };
#pragma unroll
    for (int j = 0; j < C; ++j) offer(tid + j * nt, s8[j]);
#pragma unroll 1
    for (int i0 = C * nt; i0 < a.nlist; i0 += M * nt) {
        double v[M];
        request(i0, v);
#pragma unroll
        for (int j = 0; j < M; ++j) offer(i0 + j * nt + tid, v[j]);
    }
    __syncthreads();
    const uint32_t cnt = sh[4];
    if (cnt > (uint32_t)kSelectPoolCap) return false;
    const int runs = (int)((cnt + 63) / 64);
#pragma unroll 1
    for (int r = wave; r < runs; r += nt >> 6) {
        const uint32_t e = (uint32_t)(r * 64 + lane);
        pool[e] = bitonic_sort64<true>(e < cnt ? pool[e] : (Cand)0);
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t t = tid; t < (uint32_t)runs * 64; t += nt) {
        const Cand me = pool[t];
        uint32_t rank = 0;                              // candidates ahead of this one
#pragma unroll 1
        for (int r0 = 0; r0 < runs; r0 += 4) {
            // four runs at a time: their reads overlap
            uint32_t at[4] = {0, 0, 0, 0};
#pragma unroll
            for (int st = 32; st >= 1; st >>= 1) {
                Cand o[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) o[u] = pool[min(r0 + u, runs - 1) * 64 + at[u] + st - 1];
#pragma unroll
                for (int u = 0; u < 4; ++u) at[u] += o[u] > me ? st : 0;
            }
            Cand o[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] = pool[min(r0 + u, runs - 1) * 64 + at[u]];
#pragma unroll
            for (int u = 0; u < 4; ++u) rank += r0 + u < runs ? at[u] + (o[u] > me ? 1u : 0u) : 0u;
        }
        if (me != 0) in_order[rank] = me;
    }
    __syncthreads();
    auto cluster_of = [](Cand c) { return 0xFFFFFFu - (uint32_t)(c & 0xFFFFFFull); };
#pragma unroll 1
    for (uint32_t i = tid; i < nprobe; i += nt) {
        const Cand c = in_order[i];
        idx[i] = cluster_of(c);
        if (i + 1 < cnt && (c >> 24) == (in_order[i + 1] >> 24)) sh[6] = 1;
    }
    __syncthreads();
    if (__builtin_expect(sh[6] != 0, 0)) {
        uint32_t* low = (uint32_t*)pool;
        // the low bits of the keys, larger = nearer; candidates of one prefix stand in order of their index
#pragma unroll 1
        for (uint32_t t = tid; t < cnt; t += nt) low[t] = (uint32_t)(~coarse_key(sc[cluster_of(in_order[t])], a.metric)) & 0xFFFFFFu;
        __syncthreads();
#pragma unroll 1
        for (uint32_t t = tid; t < cnt; t += nt) {
            const uint64_t prefix = in_order[t] >> 24;
            if (!((t > 0 && (in_order[t - 1] >> 24) == prefix) || (t + 1 < cnt && (in_order[t + 1] >> 24) == prefix))) continue;
            // first .. last - 1: those of this prefix
            auto count_until = [&](auto&& before) {
                uint32_t lo = 0, hi = cnt;
                while (lo < hi) { const uint32_t m = (lo + hi) >> 1; if (before(in_order[m] >> 24)) lo = m + 1; else hi = m; }
                return lo;
            };
            const uint32_t first = count_until([&](uint64_t p) { return p > prefix; });
            const uint32_t last = count_until([&](uint64_t p) { return p >= prefix; });
            const uint32_t me = low[t];
            uint32_t at = first;
#pragma unroll 1
            for (uint32_t j0 = first; j0 < last; j0 += 8) {
                uint32_t o[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) o[u] = low[min(j0 + u, last - 1)];
#pragma unroll
                for (int u = 0; u < 8; ++u) at += (uint32_t)((j0 + u < last) & ((o[u] > me) | ((o[u] == me) & (j0 + u < t))));
            }
            if (at < nprobe) idx[at] = cluster_of(in_order[t]);
        }
        __syncthreads();
    }
    return true;
}

__global__ __launch_bounds__(kSelectThreads) void select_kernel(SelectArgs a, uint32_t pad, int in_lds,
                                                                int prefix_in_lds, int pooled) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t sh[8];
    __shared__ uint32_t red[96];
    __shared__ uint32_t scan_buf[kSelectThreads / 64 + 1];
    const int tid = threadIdx.x, nt = blockDim.x;
    const int qi = blockIdx.x;
    const double* sc = a.scores + (size_t)qi * a.nlist;
    const uint32_t nprobe = a.nprobe;
    const size_t sort_bytes = in_lds ? (size_t)pad * 12 : 0;
    uint32_t* idx;
    if (in_lds) {
        uint64_t* keys = (uint64_t*)smem_raw;
        idx = (uint32_t*)(smem_raw + sizeof(uint64_t) * pad);
        bool done = false;
        if (pooled) {
            Cand* pool = (Cand*)(((uintptr_t)(smem_raw + sort_bytes + (size_t)(nprobe + 1) * 4) + 15) & ~(uintptr_t)15);
            done = select_pooled(a, sc, idx, pool, pool + kSelectPoolCap, hist, red, sh);
        }
        if (!done) {
            __syncthreads();
            select_sorted(a, sc, keys, idx, pad, hist, sh);
        }
    } else {
        uint64_t* keys = a.sort_keys + (size_t)qi * pad;
        idx = a.sort_idx + (size_t)qi * pad;
        select_sorted(a, sc, keys, idx, pad, hist, sh);
    }

    // slot tables: per selected cluster its placement and its rows
    const int64_t* off = a.off;
    int64_t* s_base = a.slots.base + (size_t)qi * nprobe;
    uint32_t* s_grow = a.slots.grow + (size_t)qi * nprobe;
    uint32_t* s_n = a.slots.nrows + (size_t)qi * nprobe;
    uint32_t* s_rp = a.slots.rprefix + (size_t)qi * (nprobe + 1);
    uint32_t* l_rp = (uint32_t*)(smem_raw + sort_bytes);     // LDS copy of the row prefix
    uint32_t carry = 0;
    // one selected cluster: its table entries; returns the rows it contributes to the scan
    auto fill_slot = [&](uint32_t i) -> uint32_t {
        uint32_t c = in_lds ? ((uint32_t*)(smem_raw + sizeof(uint64_t) * pad))[i] : idx[i];
        a.probe[(size_t)qi * nprobe + i] = (int32_t)c;
        int64_t lo = off[c];
        uint32_t n = (uint32_t)(off[c + 1] - lo);
        int64_t ro = a.res_off[c];
        s_base[i] = ro;
        s_grow[i] = (uint32_t)lo;
        s_n[i] = n;
        if (a.used && ro >= 0) a.used[c] = 1u;            // cache bookkeeping: resident and selected
        return ro >= 0 ? n : 0;
    };
    if (nprobe <= 64) {
        // the whole table fits one wavefront: prefix inside it, no LDS round trips
        if (wave_id() == 0) {
            const uint32_t i = (uint32_t)tid;
            const uint32_t rows = i < nprobe ? fill_slot(i) : 0;
            uint32_t incl = rows;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                uint32_t up = __shfl_up(incl, o);
                if (tid >= o) incl += up;
            }
            if (i < nprobe) {
                s_rp[i] = incl - rows;
                if (prefix_in_lds) l_rp[i] = incl - rows;
            }
            const uint32_t total = read_lane(incl, 63);
            if (tid == 0) {
                scan_buf[0] = total;
                s_rp[nprobe] = total;
                if (prefix_in_lds) l_rp[nprobe] = total;
                if (a.rows_counter) atomicAdd(a.rows_counter, (unsigned long long)total);
            }
        }
        __syncthreads();
        carry = scan_buf[0];
    } else {
        for (uint32_t base = 0; base < nprobe; base += nt) {
            uint32_t i = base + tid;
            uint32_t rows = i < nprobe ? fill_slot(i) : 0;
            // block-wide exclusive scan of `rows`
            uint32_t incl = rows;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                uint32_t up = __shfl_up(incl, o);
                if ((tid & 63) >= o) incl += up;
            }
            if ((tid & 63) == 63) scan_buf[tid >> 6] = incl;
            __syncthreads();
            uint32_t wave_off = 0, total = 0;
#pragma unroll
            for (int w = 0; w < kSelectThreads / 64; ++w) {        // all sums read at once
                const uint32_t v = w < nt / 64 ? scan_buf[w] : 0;
                total += v;
                wave_off += w < (tid >> 6) ? v : 0;
            }
            if (i < nprobe) {
                uint32_t ex = carry + wave_off + incl - rows;
                s_rp[i] = ex;
                if (prefix_in_lds) l_rp[i] = ex;
            }
            carry += total;
            __syncthreads();
        }
        if (tid == 0) {
            s_rp[nprobe] = carry;
            if (prefix_in_lds) l_rp[nprobe] = carry;
            if (a.rows_counter) atomicAdd(a.rows_counter, (unsigned long long)carry);
        }
        __syncthreads();
    }

    // workgroup shares: rows split evenly, each share starting inside some slot
    const uint32_t R = carry;
    const uint32_t per = R / (uint32_t)a.grid, extra = R % (uint32_t)a.grid;
    const uint32_t* rp = prefix_in_lds ? l_rp : s_rp;
    for (int b = tid; b < (nprobe > kLaneTableSlots ? a.grid : 0); b += nt) {   // few slots: the scan finds its share itself
        WgDesc ds;
        ds.r_begin = per * (uint32_t)b + min((uint32_t)b, extra);        // the first `extra` shares get one more row
        ds.r_end = per * (uint32_t)(b + 1) + min((uint32_t)(b + 1), extra);
        uint32_t slot = 0;
        if (ds.r_begin < ds.r_end) {
            uint32_t lo = 0, hi = nprobe;        // invariant: rp[lo] <= r_begin < rp[hi]
            while (hi - lo > 1) {
                uint32_t mid = (lo + hi) >> 1;
                if (rp[mid] <= ds.r_begin) lo = mid; else hi = mid;
            }
            slot = lo;
        }
        ds.slot = slot;
        ds.slot_rbegin = rp[slot];
        ds.slot_rend = rp[slot + 1];
        ds.slot_grow = s_grow[slot];
        ds.slot_base = s_base[slot];
        a.desc[(size_t)qi * a.grid + b] = ds;
    }
}

static uint32_t next_pow2(uint32_t v) { uint32_t p = 1; while (p < v) p <<= 1; return p; }

// power-of-two length of the select kernel's sort array for (nlist, nprobe)
uint32_t select_sort_pad(int nlist, int nprobe) {
    uint32_t full = next_pow2((uint32_t)nlist), part = next_pow2((uint32_t)nprobe);
    return part < full ? part : full;     // sort only the selected clusters when that is fewer
}

hipError_t launch_select(const SelectArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (selects_few(a.nlist, a.nprobe)) {
        if (a.nlist <= kFewThreads * kFewPerThread) IVF_LAUNCH(select_few_kernel<kFewThreads>, dim3(a.nq), dim3(kFewThreads), few_lds(kFewThreads), s, e0, e1, a);
        else IVF_LAUNCH(select_few_kernel<kSelectThreads>, dim3(a.nq), dim3(kSelectThreads), few_lds(kSelectThreads), s, e0, e1, a);
        return hipGetLastError();
    }
    uint32_t pad = select_sort_pad(a.nlist, a.nprobe);
    int in_lds = pad <= (uint32_t)kSortLdsCap;
    int prefix_in_lds = a.nprobe <= kPrefixLdsCap;
    const int threads = kSelectThreads;
    size_t lds = (in_lds ? (size_t)pad * 12 : 0) + (prefix_in_lds ? (size_t)(a.nprobe + 1) * 4 : 0);
    // the pool holds what passes the cut for up to 512 of any number of clusters, and all of 1024 (for
    // 1000 of 2048 lists it would rank 2048: 50 us against 32 of the sorting network below)
    const int pooled = in_lds && a.nlist <= 0xFFFFFF && (a.nprobe <= 512 || a.nlist <= 1024);
    if (pooled) lds += 16 + (size_t)kSelectPoolCap * 16;           // the pool, as it came and in order
    IVF_LAUNCH(select_kernel, dim3(a.nq), dim3(threads), lds, s, e0, e1, a, pad, in_lds, prefix_in_lds, pooled);
    return hipGetLastError();
}

// =============================================================================================
// List scan (App. B, second step): d(x, y) for every row y of every selected, resident list,
// reduced in the kernel to the best rows each wavefront saw.  HBM-bound: each row is read once
// with 16-byte streaming loads; only candidate lists are written.
//
// A row is covered by LPR lanes with SEG 16-byte loads each, so one wavefront instruction
// covers 64/LPR rows; a batch is U such row groups; each wavefront has kScanBatches batches in
// flight (one: a compute unit's eight wavefronts overlap each other).  The resident rows of
// a query's clusters form one sequence.  With up to kLaneTableSlots selected clusters the
// sequence is cut into windows of one batch and wavefront w of all W takes the windows
// w, w + W, ...: every wavefront then reads the same mix of addresses.  With more clusters the
// sequence is split evenly over the workgroups (the select kernel wrote where each share begins)
// and inside a workgroup over its wavefronts.
//
// Every wavefront writes its own candidate list (kCandSlots per list, unordered, 0 = empty) and
// the list's best entry again into a dense array of heads: no LDS, no barrier.
// =============================================================================================
// Position of a wavefront in the row sequence of its query.
struct Cursor {
    uint32_t r, r_end;           // next row and end of the current range (a window, or the wavefront's share)
    uint32_t win, win_step;      // windows: start of the current one, distance to the next (0: one contiguous range)
    uint32_t total;              // rows in the sequence (windows only)
    uint32_t slot, s_rb, s_re;   // current slot and its row range
    uint32_t s_grow;
    int64_t s_base;
};

struct Batch {
    const unsigned char* rows;   // first row of the batch in the device buffer
    uint32_t nr;                 // rows in the batch (0: none left)
    uint32_t grow;               // global row of the first row
};

// With at most kLaneTableSlots selected clusters a wavefront keeps the query's slot table in its
// lanes: lane i holds the end of slot i in the row sequence, its first global row and its place
// in the device buffer.  Finding the slot of a row is then one ballot, and stepping to the next
// slot costs no memory access.
struct LaneTable {
    bool on;
    int nprobe;
    uint32_t end, grow;
    int64_t base;
    __device__ __forceinline__ void load(const ScanArgs& p, int qi) {
        on = p.nprobe <= kLaneTableSlots;
        nprobe = p.nprobe;
        end = 0; grow = 0; base = 0;
        const int lane = lane_id();
        if (on && lane < p.nprobe) {
            const size_t o = (size_t)qi * p.nprobe + lane;
            end = p.slots.rprefix[o + qi + 1];
            grow = p.slots.grow[o];
            base = p.slots.base[o];
        }
    }
    // Every workgroup selects the clusters for itself, from the coarse scores; the first of a query also leaves the tables.
    // When they are all resident at once, selecting side by side takes as long as once, and the
    // launch in between and the way of the tables through memory go (whole search, us, select kernel / here: 8 of 64
    // clusters, 2500 rows of 128 18.0 / 15.6; 48 of 700, 41,000 of 300 fp16 43.1 / 42.0; 32 of 1024, 30,000 of 768 33.3 / 33.0).
    __device__ __forceinline__ void select(const ScanArgs& p, int qi) {
        extern __shared__ __align__(16) unsigned char smem_raw[];
        FewLds& L = *(FewLds*)smem_raw;
        select_few<kScanThreads>(p.scores + (size_t)qi * p.nlist, p.nlist, p.nprobe, p.metric, L);
        const LaneSlot s = slot_of_lane(L, p.nprobe, p.off, p.res_off);
        on = true;
        nprobe = p.nprobe;
        end = s.end; grow = s.grow; base = s.base;
        if (blockIdx.x == 0 && wave_id() == 0) store_slots(s, p.nprobe, qi, p.slots, p.probe, nullptr, p.rows_counter);
    }
    __device__ __forceinline__ uint32_t total() const { return read_lane(end, nprobe - 1); }
    // points the cursor at the slot that holds row c.r (c.r below the total)
    __device__ __forceinline__ void seek(Cursor& c) const {
        const int slot = __popcll(__ballot(lane_id() < nprobe && end <= c.r));     // ends are non-decreasing
        c.slot = (uint32_t)slot;
        c.s_rb = slot ? read_lane(end, slot - 1) : 0u;
        c.s_re = read_lane(end, slot);
        c.s_grow = read_lane(grow, slot);
        c.s_base = (int64_t)(((uint64_t)read_lane((uint32_t)((uint64_t)base >> 32), slot) << 32) | read_lane((uint32_t)base, slot));
    }
};

__device__ __forceinline__ Batch next_batch(Cursor& c, const ScanArgs& p, int qi, int rows_per_batch,
                                            size_t row_bytes, const LaneTable& tab) {
    Batch b{nullptr, 0, 0};
    if (c.r >= c.r_end) {
        if (c.win_step == 0) return b;
        if (c.total - c.win <= c.win_step) { c.win_step = 0; return b; }
        c.win += c.win_step;                 // the wavefront's next window
        c.r = c.win;
        c.r_end = c.total - c.win < (uint32_t)rows_per_batch ? c.total : c.win + (uint32_t)rows_per_batch;
    }
    if (tab.on) {
        if (c.r >= c.s_re) tab.seek(c);
    } else {
        while (c.r >= c.s_re) {      // step to the slot that holds row r (skips empty / absent lists)
            c.slot += 1;
            const size_t o = (size_t)qi * p.nprobe + c.slot;
            c.s_rb = c.s_re;
            c.s_re = p.slots.rprefix[o + qi + 1];
            c.s_grow = p.slots.grow[o];
            c.s_base = p.slots.base[o];
        }
    }
    const uint32_t in_slot = c.r - c.s_rb;
    b.nr = min((uint32_t)rows_per_batch, min(c.r_end, c.s_re) - c.r);      // a window that crosses into the next slot comes in two batches
    b.rows = (const unsigned char*)p.buf + ((size_t)c.s_base + in_slot) * row_bytes;
    b.grow = c.s_grow + in_slot;
    c.r += b.nr;
    return b;
}

__device__ __forceinline__ Cursor start_cursor(const ScanArgs& p, int qi, const LaneTable& tab, int rows_per_batch) {
    const int wave = wave_id();
    Cursor c;
    c.win = 0; c.win_step = 0; c.total = 0;
    if (tab.on) {
        const uint32_t R = tab.total();
        const uint32_t w = blockIdx.x * kScanWaves + (uint32_t)wave;
        c.total = R;
        c.win = w * (uint32_t)rows_per_batch;
        c.win_step = (uint32_t)p.grid * kScanWaves * (uint32_t)rows_per_batch;
        c.r = min(c.win, R);
        c.r_end = R - c.r < (uint32_t)rows_per_batch ? R : c.r + (uint32_t)rows_per_batch;
        c.slot = 0; c.s_rb = 0; c.s_re = 0; c.s_grow = 0; c.s_base = 0;
        if (c.r >= c.r_end) c.win_step = 0;        // beyond the last window: nothing to do
        return c;
    }
    const WgDesc ds = p.desc[(size_t)qi * p.grid + blockIdx.x];
    const uint32_t cnt = ds.r_end - ds.r_begin;
    c.r = ds.r_begin + (uint32_t)((uint64_t)cnt * wave / kScanWaves);
    c.r_end = ds.r_begin + (uint32_t)((uint64_t)cnt * (wave + 1) / kScanWaves);
    c.slot = ds.slot; c.s_rb = ds.slot_rbegin; c.s_re = ds.slot_rend;
    c.s_grow = ds.slot_grow; c.s_base = ds.slot_base;
    return c;
}

// What a wavefront leaves behind: its candidates as a list of 64 * KL entries (the sorted list when it has one,
// else the loose candidates as they stand) and the best of them as the list's head.
template <int KL>
__device__ __forceinline__ void write_wave_list(WaveTopK<KL, false>& top, const ScanArgs& p, int qi) {
    const int lane = lane_id();
    const size_t list = ((size_t)qi * p.grid + blockIdx.x) * kScanWaves + (size_t)wave_id();
    Cand* out = p.part + list * (size_t)(64 * KL);
    const bool has_list = read_lane(top.top[0], 0) != 0;
    Cand head;
    if (KL == 1 && !has_list) {
        const Cand c = lane < top.pcount ? top.pend : (Cand)0;
        out[lane] = c;
        head = wave_max(c);
    } else {
        top.flush(p.kprime);
#pragma unroll
        for (int j = 0; j < KL; ++j) {
            const int e = j * 64 + lane;
            out[e] = e < p.kprime ? top.top[j] : (Cand)0;
        }
        head = read_lane(top.top[0], 0);
    }
    if (lane == 0) p.heads[list] = head;
}

// TAIL: rows that are not whole 16-byte chunks, and therefore start at any element.  The lane with
// the last, partial chunk of a row loads the 16 bytes that END with the row and clears the elements
// that the lane before it has already, in its slice of the query and in every chunk it loads: no
// load leaves the row.  (One element per lane and row at a time, 34,500 rows of 300 fp16: 30.1 us;
// this: 12.4.)
// SEL: the scan selects the clusters itself.  A kernel of its own: with both ways in one the scan of given tables lost 4
// to 14 per cent (269 of 6988 clusters of 1024 bf16 32.1 -> 36.5 us).
template <typename T, int LPR, int SEG, int U, int METRIC, int KL, bool TAIL, bool SEL>
__global__ __launch_bounds__(kScanThreads) void scan_kernel(ScanArgs p) {
    constexpr int EPL = T::kPerLoad;
    constexpr int RPI = 64 / LPR;
    constexpr int RPB = U * RPI;
    const int lane = lane_id();
    const int sub = lane % LPR, rsel = lane / LPR;
    const int qi = blockIdx.y;
    const size_t row_bytes = (size_t)p.d * T::kBytes;

    // first element of this lane's chunk `sg` in memory: the chunk's place, or for a partial one EPL
    // elements before the end of the row (TAIL; d is at least EPL, else a multiple of it)
    auto place = [&](int col) { return TAIL ? min(col, p.d - EPL) : col; };
    const int tail_seg = TAIL ? ((p.d + EPL - 1) / EPL - 1) / LPR : 0;
    uint32_t keep[4] = {~0u, ~0u, ~0u, ~0u};          // TAIL: the elements of the chunk in segment tail_seg that count
    if (TAIL) {
        const int col = (tail_seg * LPR + sub) * EPL, skip = col - place(col);       // above EPL: the lane has no chunk
#pragma unroll
        for (int e = 0; e < EPL; ++e)
            if (e < skip) keep[e * T::kBytes / 4] &= T::kBytes == 4 ? 0u : (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
    }

    // This lane's slice of the query.  It is requested right AFTER the tables: loads return in order, and the
    // tables decide where the rows are, so nothing should arrive before them; the query is needed
    // only when the first rows are there.  (Measured: query first 16.8 us, tables first 16.5,
    // query after the first rows 16.6 - 16.9.)
    float qv[SEG][EPL];
    const float* q = p.q + (size_t)qi * p.d;
    auto load_query = [&]() {
#pragma unroll
        for (int sg = 0; sg < SEG; ++sg) {
            const int col = (sg * LPR + sub) * EPL;
            if (TAIL) {
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    const int c = place(col) + e;
                    qv[sg][e] = col < p.d && c >= col ? q[c] : 0.f;
                }
            } else {
#pragma unroll
                for (int e = 0; e < EPL; e += 4) {
                    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (col < p.d) t = *(const float4*)(q + col + e);
                    qv[sg][e] = t.x; qv[sg][e + 1] = t.y; qv[sg][e + 2] = t.z; qv[sg][e + 3] = t.w;
                }
            }
        }
    };

    LaneTable tab;
    if (SEL) {
        load_query();                 // (behind the selection: 0.4 us longer, and 8 registers more)
        tab.select(p, qi);
    } else {
        tab.load(p, qi);
        load_query();
    }
    Cursor cur = start_cursor(p, qi, tab, RPB);

    WaveTopK<KL, false> top;
    top.init();

    // `tie` receives the global row of batch row `lane` (lanes < RPB): equal keys come out by smaller row
    auto issue = [&](const Batch& b, uint4 (&v)[U][SEG], uint32_t& tie) {
        tie = b.grow + min((uint32_t)lane, b.nr - 1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t r = min((uint32_t)(u * RPI + rsel), b.nr - 1);   // rows past the end re-read the last one
            const unsigned char* rp = b.rows + (size_t)r * row_bytes;
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg) {
                int col = (sg * LPR + sub) * EPL;
                if (col < p.d) v[u][sg] = TAIL ? load_stream16_any(rp + (size_t)place(col) * T::kBytes) : load_stream16(rp + (size_t)col * T::kBytes);
                else v[u][sg] = make_uint4(0, 0, 0, 0);
            }
        }
    };
    auto consume = [&](const Batch& b, const uint4 (&v)[U][SEG], uint32_t tie) {
        float acc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float s = 0.f;
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg) {
                float x[EPL];
                uint4 w = v[u][sg];
                if (TAIL && sg == tail_seg) { w.x &= keep[0]; w.y &= keep[1]; w.z &= keep[2]; w.w &= keep[3]; }
                Unpack<T>::run(w, x);
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    if (METRIC == 0) s = fmaf(qv[sg][e], x[e], s);
                    else { float df = qv[sg][e] - x[e]; s = fmaf(df, df, s); }
                }
            }
            s = group_total_last_lane<LPR>(s);
            acc[u] = METRIC == 0 ? s : -s;        // key: larger is nearer
        }
        // almost every row fails the threshold: one ballot decides whether to look closer
        bool any = false;
        const bool leader = sub == LPR - 1;
#pragma unroll
        for (int u = 0; u < U; ++u) any |= leader && (uint32_t)(u * RPI + rsel) < b.nr && acc[u] >= top.thr;
        if (__ballot(any)) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int j = 0; j < RPI; ++j) {
                    const uint32_t r = u * RPI + j;
                    const float ck = read_lane(acc[u], j * LPR + LPR - 1);
                    if (r < b.nr && ck >= top.thr) top.push(ck, read_lane(tie, (int)r));
                }
            }
            if (top.pcount > 64 - RPB) top.flush(p.kprime);   // room for a whole batch stays free
        }
    };

    // kScanBatches batches in flight: the oldest is consumed, its buffer takes the next one
    uint4 v[kScanBatches][U][SEG];
    uint32_t tie[kScanBatches];
    Batch bt[kScanBatches];
#pragma unroll
    for (int i = 0; i < kScanBatches; ++i) {
        tie[i] = 0;
        bt[i] = next_batch(cur, p, qi, RPB, row_bytes, tab);
        if (bt[i].nr) issue(bt[i], v[i], tie[i]);
    }
    bool more = true;
    while (more) {
#pragma unroll
        for (int i = 0; i < kScanBatches; ++i) {
            if (bt[i].nr == 0) { more = false; break; }     // batches arrive in order: an empty buffer ends the walk
            consume(bt[i], v[i], tie[i]);
            bt[i] = next_batch(cur, p, qi, RPB, row_bytes, tab);
            if (bt[i].nr) issue(bt[i], v[i], tie[i]);
        }
    }
    write_wave_list<KL>(top, p, qi);
}

// Fallback for rows of less than 16 bytes and of more than 8 KB: element-wise loads, query in LDS, 4 rows per batch.
template <int METRIC, int KL>
__global__ __launch_bounds__(kScanThreads) void scan_generic_kernel(ScanArgs p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_id();
    const int qi = blockIdx.y;
    float* ql = (float*)smem;
    for (int i = threadIdx.x; i < p.d; i += blockDim.x) ql[i] = p.q[(size_t)qi * p.d + i];
    __syncthreads();
    const int esz = p.dtype == 0 ? 4 : 2;
    const size_t row_bytes = (size_t)p.d * esz;
    LaneTable tab;
    tab.load(p, qi);
    Cursor cur = start_cursor(p, qi, tab, 4);
    WaveTopK<KL, false> top;
    top.init();
    for (Batch b = next_batch(cur, p, qi, 4, row_bytes, tab); b.nr; b = next_batch(cur, p, qi, 4, row_bytes, tab)) {
        for (uint32_t r = 0; r < b.nr; ++r) {
            const unsigned char* rp = b.rows + (size_t)r * row_bytes;
            float s = 0.f;
            for (int c = lane; c < p.d; c += 64) {
                float x;
                if (p.dtype == 0) x = ((const float*)rp)[c];
                else {
                    uint16_t h = ((const uint16_t*)rp)[c];
                    x = p.dtype == 1 ? (float)__builtin_bit_cast(_Float16, h) : __uint_as_float((uint32_t)h << 16);
                }
                if (METRIC == 0) s = fmaf(ql[c], x, s);
                else { float df = ql[c] - x; s = fmaf(df, df, s); }
            }
            s = group_total_last_lane<64>(s);
            float ck = read_lane(METRIC == 0 ? s : -s, 63);
            if (ck >= top.thr) {
                top.push(ck, b.grow + r);
                if (top.pcount == 64) top.flush(p.kprime);
            }
        }
    }
    write_wave_list<KL>(top, p, qi);
}

// ---- shape selection ---------------------------------------------------------------------
// (lanes per row, 16-byte segments per lane, row groups per batch), keyed by the number of
// 16-byte chunks in a row.  A batch is about 6 KB and a wavefront has one in flight: with eight
// wavefronts per compute unit that keeps the memory path busy, and measured against two batches
// of 12 KB in flight it ends every scan about a microsecond earlier (shorter queues, a finer
// grain at the end).
struct ShapeOpt { int lpr, seg, u; };
static const ShapeOpt kShapes[] = {{16, 1, 6}, {32, 1, 6}, {64, 1, 6}, {32, 3, 2}, {64, 2, 3},
                                   {64, 3, 2}, {64, 4, 2}, {64, 8, 1}};

ScanShape pick_scan_shape(int d, int dtype) {
    const int esz = dtype == 0 ? 4 : 2;
    const size_t row_bytes = (size_t)d * esz;
    if (row_bytes < 16) return ScanShape{0, 0, 0, 4, 0};
    const int chunks = (int)((row_bytes + 15) / 16);
    int best = -1, best_waste = 1 << 30;
    for (int i = 0; i < (int)(sizeof(kShapes) / sizeof(kShapes[0])); ++i) {
        int cap = kShapes[i].lpr * kShapes[i].seg;
        if (cap < chunks) continue;
        int waste = cap - chunks;
        if (waste < best_waste) { best = i; best_waste = waste; }
    }
    if (best < 0) return ScanShape{0, 0, 0, 4, 0};
    return ScanShape{kShapes[best].lpr, kShapes[best].seg, kShapes[best].u,
                     kShapes[best].u * (64 / kShapes[best].lpr), row_bytes % 16 != 0};
}

// The same shape with two row groups per batch: for scans whose rows would keep less than a quarter of
// the wavefronts busy in batches of six groups, which then run long code for few rows.  Measured on
// one query (us, two groups against six): 600 to 6000 rows of 128 fp32 4.2-4.5 / 5.0-5.6, 12000 5.0 /
// 4.9; 2500 rows of 300 fp16 4.5 / 5.6, 6000 5.2 / 4.7; 2500 of 256 fp32 4.4 / 5.3, 6000 4.6 / 4.6.
// (rows of several segments have two or three groups per batch as they are.)
constexpr int kFewGroups = 2;
ScanShape scan_shape_for_rows(const ScanShape& shape, uint64_t rows, int kprime, int n_cu) {
    if (shape.lanes_per_row == 0 || shape.segments != 1 || kprime > 64) return shape;
    if (rows / (uint64_t)shape.rows_per_batch > (uint64_t)(n_cu * kScanMaxWgPerCu * kScanWaves / 4)) return shape;
    ScanShape few = shape;
    few.unroll = kFewGroups;
    few.rows_per_batch = kFewGroups * (64 / shape.lanes_per_row);
    return few;
}

typedef void (*ScanFn)(ScanArgs);

template <typename T, int LPR, int SEG, int U, bool TAIL>
static ScanFn scan_fn_shape(int metric, bool big, bool sel) {
    if (sel) return metric == 0 ? (ScanFn)scan_kernel<T, LPR, SEG, U, 0, 1, TAIL, true> : (ScanFn)scan_kernel<T, LPR, SEG, U, 1, 1, TAIL, true>;
    if (metric == 0) return big ? (ScanFn)scan_kernel<T, LPR, SEG, U, 0, 2, TAIL, false> : (ScanFn)scan_kernel<T, LPR, SEG, U, 0, 1, TAIL, false>;
    return big ? (ScanFn)scan_kernel<T, LPR, SEG, U, 1, 2, TAIL, false> : (ScanFn)scan_kernel<T, LPR, SEG, U, 1, 1, TAIL, false>;
}

template <typename T, int LPR, bool TAIL>
static ScanFn scan_fn_few(int metric, bool sel) {
    if (sel) return metric == 0 ? (ScanFn)scan_kernel<T, LPR, 1, kFewGroups, 0, 1, TAIL, true> : (ScanFn)scan_kernel<T, LPR, 1, kFewGroups, 1, 1, TAIL, true>;
    return metric == 0 ? (ScanFn)scan_kernel<T, LPR, 1, kFewGroups, 0, 1, TAIL, false> : (ScanFn)scan_kernel<T, LPR, 1, kFewGroups, 1, 1, TAIL, false>;
}

// sel: the variant that selects the clusters itself (kprime up to 64)
template <typename T>
static ScanFn scan_fn_dtype(const ScanShape& sh, int metric, bool big, bool sel) {
    const int l = sh.lanes_per_row, g = sh.segments;
#define IVF_FEW(L) if (l == L && g == 1 && !big && sh.unroll == kFewGroups) return sh.tail ? scan_fn_few<T, L, true>(metric, sel) : scan_fn_few<T, L, false>(metric, sel);
    IVF_FEW(16) IVF_FEW(32) IVF_FEW(64)
#undef IVF_FEW
#define IVF_SHAPE(L, G, UU) if (l == L && g == G) return sh.tail ? scan_fn_shape<T, L, G, UU, true>(metric, big, sel) : scan_fn_shape<T, L, G, UU, false>(metric, big, sel);
    IVF_SHAPE(16, 1, 6) IVF_SHAPE(32, 1, 6) IVF_SHAPE(64, 1, 6) IVF_SHAPE(32, 3, 2)
    IVF_SHAPE(64, 2, 3) IVF_SHAPE(64, 3, 2) IVF_SHAPE(64, 4, 2) IVF_SHAPE(64, 8, 1)
#undef IVF_SHAPE
    return nullptr;
}

static ScanFn scan_fn(const ScanShape& sh, int dtype, int metric, int kprime, bool sel = false) {
    const bool big = kprime > 64;
    if (sel && (big || sh.lanes_per_row == 0)) return nullptr;
    if (sh.lanes_per_row == 0) {
        if (metric == 0) return big ? (ScanFn)scan_generic_kernel<0, 2> : (ScanFn)scan_generic_kernel<0, 1>;
        return big ? (ScanFn)scan_generic_kernel<1, 2> : (ScanFn)scan_generic_kernel<1, 1>;
    }
    if (dtype == 0) return scan_fn_dtype<F32>(sh, metric, big, sel);
    if (dtype == 1) return scan_fn_dtype<F16>(sh, metric, big, sel);
    return scan_fn_dtype<BF16>(sh, metric, big, sel);
}

static size_t scan_lds_bytes(const ScanShape& sh, int d) {
    return sh.lanes_per_row == 0 ? (size_t)d * 4 : 0;      // only the fallback kernel stages the query
}

bool scan_selects(const ScanShape& shape, int nlist, int nprobe, int kprime) {
    return shape.lanes_per_row != 0 && kprime <= 64 && nprobe <= kLaneTableSlots && nlist <= kScanThreads * kFewPerThread;
}

float scan_error_coef(const ScanShape& shape, int d, int dtype, int metric) {
    // roundings on the longest path of one row's sum: the fused multiply-adds of a lane, then the tree over the lanes
    int terms;
    if (shape.lanes_per_row == 0) terms = (d + 63) / 64 + 6;
    else {
        int tree = 0;
        for (int l = shape.lanes_per_row; l > 1; l >>= 1) ++tree;
        terms = shape.segments * (dtype == 0 ? 4 : 8) + tree;
    }
    if (metric != 0) terms += 2;          // the difference is rounded before it is squared
    return 1.05f * (float)(terms + 2) * 0x1p-24f;
}

int scan_resident_grid(const ScanShape& shape, int dtype, int metric, int kprime, int d, int n_cu) {
    ScanFn fn = scan_fn(shape, dtype, metric, kprime);
    if (!fn) return n_cu;
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)fn, kScanThreads,
                                                                scan_lds_bytes(shape, d));
    if (e != hipSuccess || per_cu < 1) per_cu = 1;
    if (per_cu > kScanMaxWgPerCu) per_cu = kScanMaxWgPerCu;
    return per_cu * n_cu;
}

hipError_t launch_scan(const ScanArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    ScanFn fn = scan_fn(a.shape, a.dtype, a.metric, a.kprime, a.scores != nullptr);
    if (!fn) return hipErrorInvalidValue;
    dim3 grid(a.grid, a.nq);
    IVF_LAUNCH(fn, grid, dim3(kScanThreads), a.scores ? few_lds(kScanThreads) : scan_lds_bytes(a.shape, a.d), s, e0, e1, a);
    return hipGetLastError();
}

// =============================================================================================
// Merge (App. B: "this involves sorting"; Sec. 4.1 step 4: results of the GPU and the host part
// are merged on the GPU).  One workgroup per query: finds the kprime best fp32 candidates of
// all workgroup lists, re-scores those rows in fp64 from the stored rows, adds the host's
// candidates (already fp64), orders everything by (score, id) and writes the k nearest.
// =============================================================================================
constexpr int kMergeCandCap = 4096;    // candidates that can be pooled
constexpr int kMergeThreads = 1024;    // kprime up to 64, one search at a time
constexpr int kMergeBesideThreads = 512;       // ... with other searches in flight, up to 48 candidates
constexpr int kMergeWideThreads = 1024;

struct MergeLds {
    uint32_t red[96];                      // the groups' maxima; scratch of the bucket cut
    uint32_t hist[256];                    // bucket cut, radix select
    uint32_t sh[8];
    uint32_t f_last;                       // key image of the last candidate that counts as kept
    Cand c_cand[kMaxKPrime];
    uint64_t f_key[2 * kMaxKPrime];        // ordered fp64 scores: larger is nearer
    int64_t f_id[2 * kMaxKPrime];
    double q_part[kMergeWideThreads / 64]; // |q|^2, by wavefronts
};

// Last resort: radix select over all entries of all lists (candidates are distinct, so the
// selection ends with exactly kprime of them).  Returns their number.
__device__ __forceinline__ int gather_radix(const MergeArgs& a, const Cand* part, MergeLds& L) {
    const int tid = threadIdx.x, nt = blockDim.x, lane = lane_id();
    const uint32_t n = (uint32_t)a.nparts * (uint32_t)a.list_len, kp = a.kprime;
    auto key_at = [&](uint32_t i) { return ~part[i]; };      // ascending = best first; all ones = empty
    __syncthreads();                       // everyone has read the words of L.sh that brought them here
    uint32_t my_valid = 0;
    for (uint32_t i = tid; i < n; i += nt) my_valid += part[i] != 0;
    if (tid == 0) { L.sh[4] = 0; L.sh[5] = 0; L.f_last = 0xFFFFFFFFu; }
    __syncthreads();
#pragma unroll
    for (int m2 = 32; m2 >= 1; m2 >>= 1) my_valid += __shfl_xor(my_valid, m2);
    if (lane == 0) atomicAdd(&L.sh[5], my_valid);
    __syncthreads();
    const uint32_t n_valid = L.sh[5];
    uint64_t mask = 0, prefix = 0; uint32_t need, group;      // all valid ones: those below the all-ones key
    if (n_valid > kp) block_radix_select<uint64_t>(key_at, n, kp, L.hist, L.sh, mask, prefix, need, group);
    // need == group here: distinct keys leave a boundary group of one
    for (uint32_t i = tid; i < n; i += nt) {
        const uint64_t key = key_at(i);
        if (key != ~0ull && (key & mask) <= prefix) {
            uint32_t p = atomicAdd(&L.sh[4], 1u);
            if (p < (uint32_t)kMaxKPrime) L.c_cand[p] = part[i];
            atomicMin(&L.f_last, (uint32_t)(part[i] >> 32));
        }
    }
    __syncthreads();
    return (int)min(L.sh[4], (uint32_t)kMaxKPrime);
}

// Can a row that the scan or the gathering dropped still belong to the k nearest?  Everything
// dropped anywhere has an fp32 key of at most f_last, the key of the last candidate kept, so its
// exact score is at most f_last + E, E bounding the rounding of the fp32 accumulation:
//   inner product   |fl(sum) - sum| <= g |q| |y|        squared distance   |fl(sum) - sum| <= g sum
// with g = err_coef (a little above (terms + 2) 2^-24 for sums whose terms pass through at most
// `terms` roundings).  The k-th best exact score found, s_k, is a lower bound of the true one;
// the result is exact when s_k > f_last + E.
__device__ __forceinline__ bool result_is_safe(double s_k, float f_last, const MergeArgs& a, double qq) {
    // single precision is enough for the bound itself: it is rounded upwards
    const float e = a.metric == 0 ? a.err_coef * (sqrtf((float)qq) * 1.0001f) * a.row_norm_max * 1.0001f
                                  : a.err_coef * fabsf(f_last) * 1.0001f;
    return s_k > (double)f_last + (double)e;
}
// The verdict on query qi: redo_flag and, for the second pass, the k-th best score found.
__device__ __forceinline__ void conclude(const MergeArgs& a, int qi, bool unsafe, double kth) {
    if (a.redo_flag) {
        a.redo_flag[qi] = unsafe ? 1u : 0u;
        if (unsafe) {
            a.redo_thr[qi] = kth;
            a.redo_ticket[qi] = 0u;
        }
    }
    if (a.host_flag) a.host_flag[qi] = unsafe ? 1u : 0u;       // pinned: read behind the completion word or the end of the kernel
}
// The completion word, behind everything that the workgroup has stored: results and verdict come from several wavefronts.
__device__ __forceinline__ void signal_done(const MergeArgs& a) {
    if (!a.done) return;
    wait_for_stores();
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence_system();
        __hip_atomic_store(a.done, a.done_value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Places in the buffer of R rows (global row numbers) of query qi, by a group of kRescoreLanes lanes: the slots whose
// range of global rows holds them.  false: none does.
template <int R>
__device__ __forceinline__ void find_rows(const MergeArgs& a, int qi, int sub, const uint32_t (&row)[R], size_t (&brow)[R], bool (&found)[R]) {
    const int np = a.nprobe;
    const int64_t* s_base = a.slots.base + (size_t)qi * np;
    const uint32_t* s_grow = a.slots.grow + (size_t)qi * np;
    const uint32_t* s_n = a.slots.nrows + (size_t)qi * np;
    int at[R];
#pragma unroll
    for (int r = 0; r < R; ++r) at[r] = -1;
#pragma unroll 1
    for (int s = sub; s < np; s += kRescoreLanes) {
        const uint32_t g = s_grow[s], n = s_n[s];
#pragma unroll
        for (int r = 0; r < R; ++r) if (row[r] >= g && row[r] - g < n) at[r] = s;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll 1
        for (int o = 1; o < kRescoreLanes; o <<= 1) at[r] = max(at[r], __shfl_xor(at[r], o));
        found[r] = at[r] >= 0;
        brow[r] = found[r] ? (size_t)(s_base[at[r]] + (int64_t)(row[r] - s_grow[at[r]])) : 0;
    }
}
// Candidates c0, c0 + step, ... (R of them, below m) of query qi re-scored by a group of kRescoreLanes lanes.  The order of
// operations is fixed (see rescore_rows), so a row has the same fp64 score whichever kernel, or the host,
// computes it.
template <int R>
__device__ __forceinline__ void score_candidates(const MergeArgs& a, int qi, MergeLds& L, const Cand* cands, uint32_t c0, uint32_t step, uint32_t m, int sub) {
    uint32_t row[R];
    int64_t id[R];
    size_t brow[R];
    bool found[R];
    double s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        row[r] = cand_tie(cands[min(c0 + step * r, m - 1)]);
        id[r] = a.ids ? a.ids[row[r]] : (int64_t)row[r];
        brow[r] = row[r]; found[r] = true;
    }
    if (!a.identity) find_rows<R>(a, qi, sub, row, brow, found);
    rescore_rows<R>(a.buf, a.q + (size_t)qi * a.d, a.d, a.dtype, a.metric, brow, sub, s);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t c = c0 + step * r;
        if (sub == 0 && c < m) {
            L.f_key[c] = ordered(!found[r] ? -INFINITY : (a.metric == 0 ? s[r] : -s[r]));
            L.f_id[c] = id[r];
        }
    }
}
// The host's candidates behind the m that were re-scored; returns their number.
__device__ __forceinline__ uint32_t add_host_candidates(const MergeArgs& a, int qi, MergeLds& L, uint32_t m) {
    if (!a.host_cand) return 0;
    const uint32_t kp = (uint32_t)a.kprime, nh = min((uint32_t)a.host_count[qi], kp);
    for (uint32_t i = threadIdx.x; i < nh; i += blockDim.x) {
        L.f_key[m + i] = ordered(a.host_cand[(size_t)qi * kp + i].key);
        L.f_id[m + i] = a.host_cand[(size_t)qi * kp + i].id;
    }
    return nh;
}
__device__ __forceinline__ void pad_results(const MergeArgs& a, int qi, uint32_t have) {
    for (uint32_t i = have + threadIdx.x; i < (uint32_t)a.k; i += blockDim.x) {
        a.out_ids[(size_t)qi * a.k + i] = -1;
        a.out_dists[(size_t)qi * a.k + i] = a.metric == 0 ? -INFINITY : INFINITY;
    }
}

// ---- kprime up to 64 -----------------------------------------------------------------------------
// The scan left one unordered list of 64 candidates per wavefront and each list's best entry in `heads` (0: empty
// list).  Candidates are distinct.  The heads are dealt to 64 groups (list l to group l % 64); the kprime-th largest
// group maximum T is not above the kprime-th largest head, so at least kprime candidates reach T and the
// kprime best overall are among those that do, in lists whose head does.  With heads spread at
// random over the groups, about kprime (1 + kprime / 128) heads reach T.  A wavefront pools the passing entries of
// the lists whose heads it holds.  Up to 32 are all re-scored, up to 512 are ranked first, more are cut
// again (the pool dealt anew) while that thins them out; what does not fit the pool is left to gather_radix.  The result is exact when nothing that was dropped can matter: result_is_safe.
//
// What bounds it: a chain of four trips to memory (heads, lists, rows, results; what the scan wrote comes from other
// XCDs, 0.8 us a trip) and the steps between them, whose instructions sixteen wavefronts issue in turn, four to a SIMD.  So: ranks
// by ballots (every lane holds one of 64 values, a value's rank is the number of lanes above it) dealt to the
// wavefronts, where a sorting network is one wavefront's chain of 21 exchanges; groups of sixteen lanes, so that one LDS
// read brings all maxima; no division by the list length; |q|^2 by a wavefront beside the others; the verdict by the lane
// that holds the k-th result, which needs no barrier behind the ranks.  Whole kernel, us, before / now: 2500 rows of 128 fp32 7.8 / 6.5, 30,000 of
// 768 fp32 8.4 / 6.9, 34,000 of 300 fp16 in squared L2 10.2 / 8.1.  Eight wavefronts with two rows of a group of lanes in flight:
// 7.5, 8.6, 8.6; four with four rows: 8.6, 9.4, 10.0; four lists always requested together: 7.0, 7.4, 8.5.
constexpr int kNormLds = 1024;                            // elements of the query that go through LDS to the wavefront that sums |q|^2
constexpr int kMergeCut = 512;                            // pooled candidates above which another cut is tried
// ... up to which they are ranked by counting; more are sorted.  Whole searches with that many copies of the best row among 400,000 of
// 128 fp32, k 10, us (400 of them the exact pass), counted / sorted: 150 415 / 420, 250 421 / 423, 400 436 / 433, 900 475 / 440.
constexpr int kMergeRanked = 384;

// NT threads.  With other searches in flight half of them (a.beside): a workgroup of sixteen wavefronts finds no room on a
// compute unit beside two workgroups of a scan (four wavefronts of 96 registers and two of 72 on a SIMD of 512) and waits
// for a scan to end.  (Re-scored 32 at a time either way, so that more than 48 candidates make it too long by itself.)
template <int NT>
__global__ __launch_bounds__(NT) void merge_kernel(MergeArgs a) {
    extern __shared__ __align__(16) unsigned char m_dyn[];
    __shared__ MergeLds L;
    __shared__ float s_q[kNormLds];
    constexpr int nt = NT, nw = nt / 64, slots = 64;
    constexpr int H = 2048 / nt;                  // heads of a thread that stay in registers: all of one query's lists
    constexpr int G = nt / 64;                    // lanes that hold a group's heads
    constexpr int kRows = 1024 / nt;              // rows of a group of lanes in flight: 32 candidates in one go
    Cand* pool = (Cand*)m_dyn;
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    const int qi = blockIdx.x, np = a.nparts, kp = a.kprime;
    const Cand* part = a.part + (size_t)qi * (size_t)np * slots;
    const Cand* heads = a.heads + (size_t)qi * np;
    const float* q = a.q + (size_t)qi * a.d;
    const uint64_t below = (1ull << lane) - 1ull;
    // head i of a thread: G consecutive lanes take the lists g, g + 64, g + 128, ... of group g
    auto list_of = [&](int t, int i) __attribute__((always_inline)) { return (i * G + (t & (G - 1))) * 64 + t / G; };
    auto head_at = [&](int i) __attribute__((always_inline)) -> Cand {
        const int l = list_of(tid, i);
        const Cand c = heads[min(l, np - 1)];
        return l < np ? c : (Cand)0;
    };
    Cand h[H];
#pragma unroll
    for (int i = 0; i < H; ++i) h[i] = head_at(i);
    float x[kNormLds / nt];
#pragma unroll
    for (int u = 0; u < kNormLds / nt; ++u) x[u] = q[min(tid + u * nt, a.d - 1)];
    if (tid == 0) { L.sh[4] = 0; L.sh[6] = 0; }

    // 1. the cut: T is the largest of the 64 maxima that at least kprime of them reach (0: fewer than kprime groups hold
    //    anything, all pass).  A wavefront tries an equal share of the 64, each by one ballot.
    auto group_max = [&](uint32_t v) __attribute__((always_inline)) {
        v = max(v, xor_lane_u32<1>(v));
        v = max(v, xor_lane_u32<2>(v));
        if (G > 4) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));      // row_half_mirror
        if (G > 8) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));      // row_mirror
        if ((lane & (G - 1)) == 0) L.red[tid / G] = v;
    };
    auto cut_of_groups = [&]() __attribute__((always_inline)) -> uint32_t {
        __syncthreads();
        const uint32_t g = L.red[lane];
        uint32_t best = 0;
#pragma unroll
        for (int i = 0; i < 64 / nw; ++i) {
            const uint32_t v = read_lane(g, wave * (64 / nw) + i);
            best = __popcll(__ballot(g >= v)) >= kp ? max(best, v) : best;
        }
        if (lane == 0 && best) atomicMax(&L.sh[6], best);
        __syncthreads();
        return L.sh[6];
    };
    {
        uint32_t best = 0;
#pragma unroll
        for (int i = 0; i < H; ++i) best = max(best, (uint32_t)(h[i] >> 32));
#pragma unroll 1
        for (int i = H; i * nt < np; ++i) best = max(best, (uint32_t)(head_at(i) >> 32));
        group_max(best);
#pragma unroll
        for (int u = 0; u < kNormLds / nt; ++u) s_q[tid + u * nt] = tid + u * nt < a.d ? x[u] : 0.f;
    }
    const uint32_t cut = cut_of_groups();

    // 2. the entries that pass, of the lists whose heads do (mostly one or two of a wavefront's)
    constexpr int C = 4;
    Cand c[C];
    auto offer = [&](uint32_t at_least) __attribute__((always_inline)) {
        uint64_t b[C];
        uint32_t n = 0;
#pragma unroll
        for (int u = 0; u < C; ++u) { b[u] = __ballot(c[u] != 0 && (uint32_t)(c[u] >> 32) >= at_least); n += (uint32_t)__popcll(b[u]); }
        if (n == 0) return;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&L.sh[4], n);
        base = read_lane(base, 0);
#pragma unroll
        for (int u = 0; u < C; ++u) {
            const uint32_t pos = base + __popcll(b[u] & below);
            if (((b[u] >> lane) & 1u) && pos < (uint32_t)kMergeCandCap) pool[pos] = c[u];
            base += (uint32_t)__popcll(b[u]);
        }
    };
    auto pool_lists = [&](Cand head, int i) __attribute__((always_inline)) {
        uint64_t lists = __ballot(head != 0 && (uint32_t)(head >> 32) >= cut);
        auto entry = [&](int l) __attribute__((always_inline)) { return part[(size_t)list_of(wave * 64 + l, i) * slots + lane]; };
#pragma unroll 1
        while (lists) {
            if ((lists & (lists - 1)) == 0) {
                c[0] = entry(__builtin_ctzll(lists));
#pragma unroll
                for (int u = 1; u < C; ++u) c[u] = 0;
                lists = 0;
            } else {
                // several: all requested before the first is looked at, the last one again where there are fewer (a load
                // behind a branch of its own is waited for where the branch ends)
                bool own[C];
                int l = 0;
#pragma unroll
                for (int u = 0; u < C; ++u) {
                    own[u] = lists != 0;
                    l = own[u] ? __builtin_ctzll(lists) : l;
                    lists &= lists - 1;
                    c[u] = entry(l);
                }
#pragma unroll
                for (int u = 0; u < C; ++u) c[u] = own[u] ? c[u] : (Cand)0;
            }
            offer(cut);
        }
    };
#pragma unroll
    for (int i = 0; i < H; ++i) pool_lists(h[i], i);
#pragma unroll 1
    for (int i = H; i * nt < np; ++i) pool_lists(head_at(i), i);
    if (wave == nw - 1) {
        // |q|^2 for the error bound
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < kNormLds / 64; ++u) { const double y = (double)s_q[u * 64 + lane]; s = fma(y, y, s); }
#pragma unroll 1
        for (int t = lane + kNormLds; t < a.d; t += 64) { const double y = (double)q[t]; s = fma(y, y, s); }
        s = wave_sum(s);
        if (lane == 0) L.q_part[0] = s;
    }
    __syncthreads();
    int cnt = (int)L.sh[4];
    const Cand* cands = pool;
    uint32_t m = 0;
#pragma unroll 1
    for (int before = kMergeCandCap + 1; __builtin_expect(cnt > kMergeCut && cnt < before, 0);) {
        before = cnt;
        // many (rows that are all alike, a few lists that hold them all): another cut, the pool dealt anew
        constexpr int R = kMergeCandCap / nt;
        Cand v[R];
        uint32_t best = 0;
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int at = u * nt + (tid & (G - 1)) * 64 + tid / G;       // (a sorted list's entries stand side by side)
            v[u] = at < cnt ? pool[at] : (Cand)0;
            best = max(best, (uint32_t)(v[u] >> 32));
        }
        group_max(best);
        if (tid == 0) L.sh[6] = 0;
        const uint32_t tighter = cut_of_groups();      // (behind its barrier everyone has read the pool and its size)
        if (tid == 0) L.sh[4] = 0;
        __syncthreads();
#pragma unroll
        for (int u0 = 0; u0 < R; u0 += C) {
#pragma unroll
            for (int u = 0; u < C; ++u) c[u] = u0 + u < R ? v[u0 + u] : (Cand)0;
            offer(tighter);
        }
        __syncthreads();
        cnt = (int)L.sh[4];
    }
    if (cnt <= 32) {
        m = (uint32_t)cnt;
        const Cand other = lane < cnt ? pool[lane] : (Cand)0;
#pragma unroll
        for (int i = 0; i < 32 / nw; ++i) {
            const Cand v = read_lane(other, wave * (32 / nw) + i);
            if (v != 0 && __popcll(__ballot(other > v)) == kp - 1 && lane == 0) L.f_last = (uint32_t)(v >> 32);
        }
    } else if (cnt <= kMergeCandCap) {
        // the first kprime take their places.  Up to 64: a value's rank is the number of lanes above it; up to
        // kMergeRanked: eight lanes per candidate count those ahead of it
        auto place = [&](Cand v, uint32_t rank) __attribute__((always_inline)) {
            if (rank < (uint32_t)kp) L.c_cand[rank] = v;
            if (rank == (uint32_t)kp - 1) L.f_last = (uint32_t)(v >> 32);
        };
        if (cnt <= 64) {
            const Cand other = lane < cnt ? pool[lane] : (Cand)0;
#pragma unroll
            for (int i = 0; i < 64 / nw; ++i) {
                const Cand v = read_lane(other, wave * (64 / nw) + i);
                const uint32_t rank = (uint32_t)__popcll(__ballot(other > v));
                if (lane == 0 && v != 0) place(v, rank);
            }
        } else if (cnt <= kMergeRanked) {
#pragma unroll 1
            for (int t = tid / 8; t < cnt; t += nt / 8) {
                const Cand me = pool[t];
                uint32_t rank, equal;
                count_above(pool, (uint32_t)cnt, me, (uint32_t)tid & 7u, rank, equal);
                if ((tid & 7) == 0) place(me, rank);
            }
        } else {
            // more, which no cut thins out: every wavefront sorts and merges its runs of 64, then wavefront 0 what the
            // wavefronts have (1500 and 3000 copies as above: 443 and 453 us, by the radix select over all lists 830 and 841)
            auto run = [&](int c) __attribute__((always_inline)) { return bitonic_sort64<true>(c * 64 + lane < cnt ? pool[c * 64 + lane] : (Cand)0); };
            Cand best = run(wave);
#pragma unroll 1
            for (int c = wave + nw; c * 64 < cnt; c += nw) best = merge_best64<true>(best, run(c));
            __syncthreads();
            pool[tid] = best;
            __syncthreads();
            if (wave == 0) {
#pragma unroll 1
                for (int w = 1; w < nw; ++w) best = merge_best64<true>(best, pool[w * 64 + lane]);
                place(best, (uint32_t)lane);
            }
        }
        __syncthreads();
        m = (uint32_t)min(cnt, kp);
        cands = L.c_cand;
    } else {
        m = (uint32_t)gather_radix(a, part, L);
        cands = L.c_cand;
    }

    // 3. fp64 re-score
    constexpr uint32_t groups = nt / kRescoreLanes;
#pragma unroll 1
    for (uint32_t c0 = (uint32_t)(tid / kRescoreLanes); c0 < m; c0 += kRows * groups)
        score_candidates<kRows>(a, qi, L, cands, c0, groups, m, tid % kRescoreLanes);
    const uint32_t tot = m + add_host_candidates(a, qi, L, m);
    __syncthreads();
    // 4. ranked by ballots, every wavefront an equal share of the results against all: nearest first, ties by smaller
    //    id (and, with an id that occurs more than once, by place); the lane whose result is the k-th proves it
    const int k = a.k;
#pragma unroll 1
    for (uint32_t t0 = 0; t0 < tot; t0 += 64) {
        const uint32_t at = min(t0 + (uint32_t)lane, tot - 1), last = min(tot - t0, 64u);
        const uint64_t mk = L.f_key[at];
        const int64_t mi = L.f_id[at];
        uint32_t rank = 0;                           // of result t0 + lane, for lanes of this wavefront's share
#pragma unroll 1
        for (uint32_t j0 = 0; j0 < tot; j0 += 64) {
            const uint32_t j = j0 + (uint32_t)lane;
            const bool in = j < tot;
            const uint64_t ok = t0 == j0 ? mk : L.f_key[min(j, tot - 1)];
            const int64_t oi = t0 == j0 ? mi : L.f_id[min(j, tot - 1)];
#pragma unroll 1
            for (uint32_t t = (uint32_t)wave; t < last; t += nw) {
                const uint64_t v = read_lane(mk, (int)t);
                uint64_t ahead = __ballot(in && ok > v);
                const uint64_t tie = __ballot(in && ok == v);
                if (__builtin_expect((tie & (tie - 1)) != 0 || t0 != j0, 0)) {
                    const int64_t vi = (int64_t)read_lane((uint64_t)mi, (int)t);
                    ahead |= __ballot(in && ok == v && (oi < vi || (oi == vi && j < t0 + t)));
                }
                if (lane == (int)t) rank += (uint32_t)__popcll(ahead);
            }
        }
        if (lane % nw == wave && t0 + (uint32_t)lane < tot && rank < (uint32_t)k) {
            const double key = unordered(mk);
            a.out_ids[(size_t)qi * k + rank] = mi;
            a.out_dists[(size_t)qi * k + rank] = (float)(a.metric == 0 ? key : -key);
            // Rows were dropped only if kprime candidates were kept (a wavefront of the scan drops nothing before
            // it holds kprime, the gathering nothing before it has kprime).
            if (rank == (uint32_t)k - 1 && m >= (uint32_t)kp) conclude(a, qi, !result_is_safe(key, unordered(L.f_last), a, L.q_part[0]), key);
        }
    }
    if (tid == 0 && m < (uint32_t)kp) conclude(a, qi, false, 0.0);
    pad_results(a, qi, tot);
    signal_done(a);
}

// ---- kprime above 64 -----------------------------------------------------------------------------
// Wide path (kprime above 64: every list holds 128 entries, best first).  A first cut is taken from
// the heads (block_bucket_cut: at least kprime of them pass, so at least kprime candidates do), the
// lists whose head passes are walked 16 entries at a time while their last entry read still passes,
// and what passes is pooled.  When the best rows sit in few lists the kprime-th largest head is a
// loose cut and the pool overflows; any kPoolCap entries that were pooled then give a tighter cut
// and the walk starts over.  A pool of more than 512 is narrowed once more, and every pooled
// candidate counts those ahead of it: the first kprime take their places.
// What bounds it: one workgroup, a handful of dependent L2 reads and barriers.  (The radix select
// over all entries reads 2 MB up to ten times from one compute unit: 494 us at 2048 lists against
// 27 us here, k 100 on 4 M x 768 fp16 rows.)
// Returns the number of candidates in L.c_cand, with the key of the kprime-th in L.f_last; -1 (for the whole
// workgroup) when the lists do not fit or masses of equal keys keep overflowing the pool.
constexpr int kWideLists = 2048;           // lists the wide path can visit: all of one query's scan wavefronts
constexpr int kWideRounds = 4;             // cuts tried before the radix select takes over
__device__ __forceinline__ int gather_wide(const MergeArgs& a, const Cand* part, const Cand* heads, MergeLds& L,
                                            Cand* pool, uint16_t* alive) {
    constexpr int nt = kMergeWideThreads;
    const int tid = threadIdx.x, lane = lane_id();
    const int np = a.nparts, slots = a.list_len;
    const uint32_t kp = (uint32_t)a.kprime;
    if (np > kWideLists) return -1;
    const Cand h0 = tid < np ? heads[tid] : (Cand)0;
    const Cand h1 = tid + nt < np ? heads[tid + nt] : (Cand)0;
    auto head_key = [&](uint32_t l) -> uint32_t { return (uint32_t)((l == (uint32_t)tid ? h0 : l == (uint32_t)(tid + nt) ? h1 : heads[l]) >> 32); };
    auto pool_key = [&](uint32_t i) -> uint32_t { return (uint32_t)(pool[i] >> 32); };
    // appends c of every lane with ok to the pool; entries past the end are counted, not stored
    auto append = [&](Cand c, bool ok) {
        const uint64_t b = __ballot(ok);
        if (!b) return;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&L.sh[4], (uint32_t)__popcll(b));
        base = read_lane(base, 0);
        const uint32_t pos = base + __popcll(b & ((1ull << lane) - 1ull));
        if (ok && pos < (uint32_t)kMergeCandCap) pool[pos] = c;
    };
    BucketCut bc = block_bucket_cut(head_key, (uint32_t)np, kp, L.hist, L.red);
    uint32_t cnt = 0;
#pragma unroll 1
    for (int round = 0;; ++round) {
        __syncthreads();                       // the cut has been read by everyone
        if (tid == 0) { L.sh[4] = 0; L.sh[5] = 0; }
        __syncthreads();
#pragma unroll 1
        for (int l = tid; l < np; l += nt) {
            const uint32_t key = head_key((uint32_t)l);
            if (key != 0 && bc.pass(key)) alive[atomicAdd(&L.sh[5], 1u)] = (uint16_t)l;
        }
        __syncthreads();
        uint32_t na = L.sh[5];
        uint16_t* cur = alive;
        uint16_t* nxt = alive + kWideLists;
#pragma unroll 1
        for (int lvl = 0; lvl < slots && na; lvl += 16) {
            __syncthreads();                   // the count of this level has been read
            if (tid == 0) L.sh[5] = 0;
            __syncthreads();
            const uint32_t total = na * 16;
#pragma unroll 1
            for (uint32_t e0 = 0; e0 < total; e0 += 2 * nt) {
                Cand c[2]; uint32_t l[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t e = e0 + u * nt + tid;
                    l[u] = cur[min(e, total - 1) / 16];
                    c[u] = e < total ? part[(size_t)l[u] * slots + lvl + e % 16] : (Cand)0;
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const bool ok = c[u] != 0 && bc.pass((uint32_t)(c[u] >> 32));
                    if (ok && (tid & 15) == 15) nxt[atomicAdd(&L.sh[5], 1u)] = (uint16_t)l[u];
                    append(c[u], ok);
                }
            }
            __syncthreads();
            na = L.sh[5];
            uint16_t* t = cur; cur = nxt; nxt = t;
        }
        __syncthreads();
        cnt = L.sh[4];
        if (cnt <= (uint32_t)kMergeCandCap) break;
        if (round == kWideRounds - 1) return -1;
        bc = block_bucket_cut(pool_key, (uint32_t)kMergeCandCap, kp, L.hist, L.red);
    }
    if (cnt > 512) {
        // kMergeCandCap / kMergeWideThreads entries per thread stay in registers while the pool is rebuilt
        bc = block_bucket_cut(pool_key, cnt, kp, L.hist, L.red);
        Cand mine[kMergeCandCap / kMergeWideThreads];
#pragma unroll
        for (int u = 0; u < kMergeCandCap / kMergeWideThreads; ++u) mine[u] = (uint32_t)(tid + u * nt) < cnt ? pool[tid + u * nt] : (Cand)0;
        __syncthreads();
        if (tid == 0) L.sh[4] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kMergeCandCap / kMergeWideThreads; ++u) append(mine[u], mine[u] != 0 && bc.pass((uint32_t)(mine[u] >> 32)));
        __syncthreads();
        cnt = L.sh[4];
    }
    // eight lanes per candidate count those ahead of it
#pragma unroll 1
    for (uint32_t t = (uint32_t)tid / 8; t < cnt; t += (uint32_t)nt / 8) {
        const Cand me = pool[t];
        uint32_t rank, equal;
        count_above(pool, cnt, me, (uint32_t)tid & 7u, rank, equal);
        if ((tid & 7) == 0 && rank < kp) L.c_cand[rank] = me;
        if ((tid & 7) == 0 && rank == kp - 1) L.f_last = (uint32_t)(me >> 32);
    }
    __syncthreads();
    return (int)min(cnt, kp);
}

__global__ __launch_bounds__(kMergeWideThreads) void merge_wide_kernel(MergeArgs a) {
    extern __shared__ __align__(16) unsigned char m_dyn[];
    __shared__ MergeLds L;
    constexpr int nt = kMergeWideThreads;
    const int tid = threadIdx.x;
    const int qi = blockIdx.x;
    const Cand* part = a.part + (size_t)qi * (size_t)a.nparts * (size_t)a.list_len;
    const Cand* heads = a.heads + (size_t)qi * a.nparts;
    const uint32_t kp = a.kprime;
    const float* q = a.q + (size_t)qi * a.d;

    // |q|^2 for the error bound, summed while the heads travel
    {
        double s = 0.0;
        for (int t = tid; t < a.d; t += nt) { const double x = (double)q[t]; s = fma(x, x, s); }
        s = wave_sum(s);
        if (lane_id() == 0) L.q_part[wave_id()] = s;
    }
    // 1. the kprime best fp32 candidates
    Cand* pool = (Cand*)m_dyn;
    int got = gather_wide(a, part, heads, L, pool, (uint16_t*)(pool + kMergeCandCap));
    if (__builtin_expect(got < 0, 0)) got = gather_radix(a, part, L);
    const uint32_t m = (uint32_t)got;
    // 2. fp64 re-score, two candidates of a group of lanes in flight (112 of 1.5 KB: 29.4 -> 27.0 us for the whole kernel)
    {
        constexpr uint32_t groups = nt / kRescoreLanes;
#pragma unroll 1
        for (uint32_t c = (uint32_t)(tid / kRescoreLanes); c < m; c += 2 * groups)
            score_candidates<2>(a, qi, L, L.c_cand, c, groups, m, tid % kRescoreLanes);
    }
    // 3. host candidates
    const uint32_t tot = m + add_host_candidates(a, qi, L, m);
    __syncthreads();
    // 4. rank by counting, eight lanes per candidate; nearest first, ties by smaller id
    const int k = a.k;
    for (uint32_t t = (uint32_t)tid / 8; t < tot; t += (uint32_t)nt / 8) {
        const uint64_t mk = L.f_key[t];
        const int64_t mi = L.f_id[t];
        uint32_t rank = 0;
        // four others per lane and pass, all read before any is compared, and no branches: a compare that
        // waits for its own LDS read every time costs more than the whole pass
#pragma unroll 1
        for (uint32_t j0 = (uint32_t)tid & 7u; j0 < tot; j0 += 32) {
            uint64_t ok[4]; int64_t oi[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = min(j0 + 8u * u, tot - 1);
                ok[u] = L.f_key[j]; oi[u] = L.f_id[j];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = j0 + 8u * u;
                const bool ahead = (ok[u] > mk) | ((ok[u] == mk) & ((oi[u] < mi) | ((oi[u] == mi) & (j < t))));
                rank += (uint32_t)(ahead & (j < tot));
            }
        }
        rank = sum_of_8(rank);
        if ((tid & 7) == 0 && rank < (uint32_t)k) {
            const double key = unordered(mk);
            a.out_ids[(size_t)qi * k + rank] = mi;
            a.out_dists[(size_t)qi * k + rank] = (float)(a.metric == 0 ? key : -key);
            if (rank == (uint32_t)k - 1 && m >= kp) {
                double qq = 0.0;
#pragma unroll
                for (int w = 0; w < nt / 64; ++w) qq += L.q_part[w];
                conclude(a, qi, !result_is_safe(key, unordered(L.f_last), a, qq), key);
            }
        }
    }
    if (tid == 0 && m < kp) conclude(a, qi, false, 0.0);
    pad_results(a, qi, tot);
    signal_done(a);
}

// =============================================================================================
// Exact second pass for a query whose first result could not be proven (merge_kernel's step 5), or
// whose candidates did not fit the list-major merge: every selected resident row is scored in fp64, in
// the order of operations of the re-score.  Only rows that reach redo_thr, a lower bound of the k-th
// best score, can belong to the result; each wavefront keeps the k best of those it meets, ordered by
// (score, id), in a small list in LDS.  The workgroup that finishes last cuts the entries of all lists
// and the host's candidates to the k best (radix select on the scores and, where equal scores hold
// the k-th place, on their ids) and rewrites the query's results.  Launched after every merge of the
// device path: the workgroups of the whole call share the flagged queries, and leave at once when
// there are none.  Bound by the bytes of the rows, then by one workgroup's trips over the lists.  (One query
// of 1 M x 768 fp32 rows, nprobe 32, with 300 copies of the best row, whole call with k 10 and 100: 3.2 and
// 183 ms when every entry of the lists was ranked by counting from memory; this: 0.33 and 0.51.)
// =============================================================================================
constexpr int kRedoThreads = 256;
constexpr int kRedoWaves = kRedoThreads / 64;
static_assert(kRedoWaves == kRedoListsPerWg, "the list buffers are sized by kRedoListsPerWg");

// Workgroups of a call at most: four per compute unit of the largest part; each looks at every flag of the call, so one
// per query makes the look quadratic (60,000 queries x 2 lists of 100 fp16 x 64, none flagged, whole call: 16.4 ms,
// 3.5 with this bound; 16,384 queries 1.40, 0.97).
constexpr uint32_t kRedoMaxWgs = 1024;

// The number of flagged queries; `mine` of them are this thread's (tid, tid + 256, ...), numbers `before` and on.
__device__ __forceinline__ uint32_t count_flagged(const uint32_t* flag, int nq, uint32_t* s_count, uint32_t& before, uint32_t& mine) {
    const int tid = threadIdx.x;
    before = 0;
    mine = 0;
    if (nq == 1) return flag[0] != 0 ? 1u : 0u;
    for (int i = tid; i < nq; i += kRedoThreads) mine += flag[i] != 0 ? 1u : 0u;
    if (!__syncthreads_or(mine != 0)) return 0u;
    s_count[tid] = mine;
    __syncthreads();
    uint32_t total = 0;
    for (int t = 0; t < kRedoThreads; ++t) { const uint32_t c = s_count[t]; before += t < tid ? c : 0u; total += c; }
    __syncthreads();
    return total;
}
// the index of flagged query number `want`, by the workgroup together
__device__ __forceinline__ int flagged_query(const uint32_t* flag, int nq, uint32_t want, uint32_t before, uint32_t mine, uint32_t* s_found) {
    if (nq == 1) return 0;
    if (want >= before && want < before + mine) {
        uint32_t seen = before;
        for (int i = threadIdx.x; i < nq; i += kRedoThreads)
            if (flag[i] != 0 && seen++ == want) *s_found = (uint32_t)i;
    }
    __syncthreads();
    const int qi = (int)*s_found;
    __syncthreads();
    return qi;
}

__global__ __launch_bounds__(kRedoThreads) void exact_redo_kernel(RedoArgs a) {
    __shared__ uint32_t s_last, s_n;
    __shared__ __align__(16) uint32_t hist[256];
    __shared__ uint32_t sh[8];
    __shared__ unsigned long long w_key[kRedoWaves][IVF_MAX_K];     // ordered score; 0 = empty
    __shared__ long long w_id[kRedoWaves][IVF_MAX_K];
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    uint32_t flags_before, flags_mine;
    const uint32_t flagged = count_flagged(a.redo_flag, a.nq, hist, flags_before, flags_mine);
    if (flagged == 0) return;
    // this workgroup is number `part` of the `parts` that serve a query: first, first + flagged, ...; of more flagged
    // queries than workgroups it serves several, one after the other and alone
    const uint32_t first = blockIdx.x % flagged, part = blockIdx.x / flagged, parts = (gridDim.x - first + flagged - 1) / flagged;
    const int np = a.nprobe, k = a.k;
#pragma unroll 1
    for (uint32_t number = first; number < flagged; number += gridDim.x) {
        const int qi = flagged_query(a.redo_flag, a.nq, number, flags_before, flags_mine, hist);
        const float* q = a.q + (size_t)qi * a.d;
        const uint32_t* rp = a.slots.rprefix + (size_t)qi * (np + 1);
        const int64_t* s_base = a.slots.base + (size_t)qi * np;
        const uint32_t* s_grow = a.slots.grow + (size_t)qi * np;
        const uint32_t R = rp[np];
        const double thr = a.redo_thr[qi];
        unsigned long long* mk = w_key[wave];
        long long* mi = w_id[wave];
        for (int i = lane; i < k; i += 64) { mk[i] = 0ull; mi[i] = 0; }
        int count = 0;                                   // entries in this wavefront's list (uniform)
        constexpr int lpc = kRescoreLanes;
        constexpr int gpw = 64 / lpc;                    // rows a wavefront scores at a time
        const int sub = lane % lpc;
        const uint32_t my_group = (part * kRedoWaves + (uint32_t)wave) * gpw + (uint32_t)(lane / lpc);
        const uint32_t ngroups = parts * kRedoWaves * gpw;
        const uint32_t rounds = (R + ngroups - 1) / ngroups;
#pragma unroll 1
        for (uint32_t it = 0; it < rounds; ++it) {
            const uint32_t r = it * ngroups + my_group;
            double key = -INFINITY;
            long long id = 0;
            if (r < R) {
                uint32_t lo = 0, hi = (uint32_t)np;            // rp[lo] <= r < rp[hi]
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (rp[mid] <= r) lo = mid; else hi = mid;
                }
                const uint32_t in_slot = r - rp[lo];
                const size_t brow = (size_t)(s_base[lo] + (int64_t)in_slot);
                const double s = rescore_row(a.buf, q, a.d, a.dtype, a.metric, brow, sub);
                key = a.metric == 0 ? s : -s;
                const uint32_t grow = s_grow[lo] + in_slot;
                id = a.ids ? (long long)a.ids[grow] : (long long)grow;
            }
            // the rows of this round that reach the threshold, and the last entry of a full list, go into the
            // list one after the other
            const unsigned long long last_key = count == k ? mk[k - 1] : 0ull;
            uint64_t want = __ballot(sub == 0 && r < R && key >= thr && (unsigned long long)ordered(key) >= last_key);
            while (want) {
                const int src = __ffsll((long long)want) - 1;
                want &= want - 1;
                const unsigned long long nk = ordered(__shfl(key, src));
                const long long nid = __shfl(id, src);
                // position: entries ahead of the new one (larger key, or equal key and smaller id)
                int ahead = 0;
                for (int i = lane; i < count; i += 64) ahead += (mk[i] > nk || (mk[i] == nk && mi[i] < nid)) ? 1 : 0;
#pragma unroll
                for (int m = 32; m >= 1; m >>= 1) ahead += __shfl_xor(ahead, m);
                if (ahead >= k) continue;                      // the list is full of better rows
                const int last = min(count, k - 1);            // entries ahead .. last-1 move down by one
                for (int base = ((last - 1) / 64) * 64; base >= 0 && last > ahead; base -= 64) {
                    const int i = base + lane;
                    const bool mv = i >= ahead && i < last;
                    const unsigned long long tk = mv ? mk[i] : 0ull;
                    const long long ti = mv ? mi[i] : 0;
                    if (mv) { mk[i + 1] = tk; mi[i + 1] = ti; }    // a wavefront's LDS operations complete in order
                }
                if (lane == 0) { mk[ahead] = nk; mi[ahead] = nid; }
                count = min(count + 1, k);
            }
        }
        // every wavefront leaves its k slots (0 = empty) in the list of its workgroup
        {
            const size_t o = ((size_t)blockIdx.x * kRedoWaves + wave) * (size_t)k;
            for (int i = lane; i < k; i += 64) {
                __hip_atomic_store(&a.list_key[o + i], i < count ? mk[i] : 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&a.list_id[o + i], mi[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        wait_for_stores();                               // the lists are in memory before the ticket says so
        __syncthreads();
        if (tid == 0) {
            __threadfence();
            s_last = atomicAdd(&a.redo_ticket[qi], 1u) == parts - 1 ? 1u : 0u;
        }
        __syncthreads();
        if (!s_last) return;                             // (parts > 1: there is no further query)
        __threadfence();
        // the last workgroup: the k best entries of all lists and of the host's candidates, by (score, id)
        const uint32_t per_wg = kRedoWaves * (uint32_t)k, n = parts * per_wg;
        const uint32_t nh = a.host_cand ? min((uint32_t)a.host_count[qi], (uint32_t)a.kprime) : 0u;
        const uint32_t tot = n + nh;
        auto place_of = [&](uint32_t j) -> size_t { return (size_t)(first + j / per_wg * flagged) * per_wg + j % per_wg; };
        auto key_of = [&](uint32_t j) -> uint64_t {
            if (j < n) return __hip_atomic_load(&a.list_key[place_of(j)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return ordered(a.host_cand[(size_t)qi * a.kprime + (j - n)].key);
        };
        auto id_of = [&](uint32_t j) -> long long {
            if (j < n) return __hip_atomic_load(&a.list_id[place_of(j)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return (long long)a.host_cand[(size_t)qi * a.kprime + (j - n)].id;
        };
        // ascending = best first; the all-ones key marks an empty entry
        auto up = [&](uint32_t j) -> uint64_t { return ~key_of(j); };
        uint32_t mine = 0;
        for (uint32_t j = tid; j < tot; j += kRedoThreads) mine += key_of(j) != 0 ? 1u : 0u;
        if (tid == 0) s_n = 0;
        __syncthreads();
        if (mine) atomicAdd(&s_n, mine);
        __syncthreads();
        const uint32_t valid = s_n, kept = min(valid, (uint32_t)k);
        uint64_t mask = 0, prefix = 0, id_edge = ~0ull;
        uint32_t need = valid, group = valid;
        if (valid > (uint32_t)k) {
            block_radix_select<uint64_t>(up, tot, (uint32_t)k, hist, sh, mask, prefix, need, group);
            if (need != group) {
                // equal scores hold the k-th place: of those the `need` smallest ids
                uint64_t im, ip;
                uint32_t in, ig;
                auto tied_id = [&](uint32_t j) -> uint64_t { const uint64_t u = up(j); return u != ~0ull && (u & mask) == prefix ? (uint64_t)id_of(j) : ~0ull; };
                block_radix_select<uint64_t>(tied_id, tot, need, hist, sh, im, ip, in, ig);
                id_edge = ip | ~im;
            }
        }
        __syncthreads();
        if (tid == 0) s_n = 0;
        __syncthreads();
        unsigned long long* o_key = w_key[0];
        long long* o_id = w_id[0];
        // those on the very edge last: with ids that occur more than once there may be more of them than places
        for (int edge = 0; edge < 2; ++edge) {
            for (uint32_t j = tid; j < tot; j += kRedoThreads) {
                const uint64_t u = up(j);
                if (u == ~0ull || (u & mask) > prefix) continue;
                const long long id = id_of(j);
                const bool tied = need != group && (u & mask) == prefix;
                if ((tied && (uint64_t)id > id_edge) || (tied && (uint64_t)id == id_edge) != (edge == 1)) continue;
                const uint32_t pos = atomicAdd(&s_n, 1u);
                if (pos < kept) { o_key[pos] = ~u; o_id[pos] = id; }
            }
            __syncthreads();
        }
        for (uint32_t e = tid; e < kept; e += kRedoThreads) {
            const unsigned long long ek = o_key[e];
            const long long ei = o_id[e];
            uint32_t rank = 0;
            for (uint32_t j = 0; j < kept; ++j) rank += (uint32_t)(o_key[j] > ek || (o_key[j] == ek && (o_id[j] < ei || (o_id[j] == ei && j < e))));
            const double key = unordered((uint64_t)ek);
            a.out_ids[(size_t)qi * k + rank] = (int64_t)ei;
            a.out_dists[(size_t)qi * k + rank] = (float)(a.metric == 0 ? key : -key);
        }
        for (uint32_t i = kept + tid; i < (uint32_t)k; i += kRedoThreads) {
            a.out_ids[(size_t)qi * k + i] = -1;
            a.out_dists[(size_t)qi * k + i] = a.metric == 0 ? -INFINITY : INFINITY;
        }
        __syncthreads();                                 // the lists in LDS are read until here
    }
}

hipError_t launch_redo(const RedoArgs& a, int grid, hipStream_t s) {
    if (a.k > IVF_MAX_K) return hipErrorInvalidValue;
    hipLaunchKernelGGL(exact_redo_kernel, dim3(std::min((uint32_t)grid * (uint32_t)a.nq, kRedoMaxWgs)), dim3(kRedoThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_merge(const MergeArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (a.done && a.nq != 1) return hipErrorInvalidValue;
    const size_t pool = (size_t)kMergeCandCap * sizeof(uint64_t);
    if (a.kprime > 64) IVF_LAUNCH(merge_wide_kernel, dim3(a.nq), dim3(kMergeWideThreads), pool + 2 * kWideLists * sizeof(uint16_t), s, e0, e1, a);
    else if (a.beside) IVF_LAUNCH(merge_kernel<kMergeBesideThreads>, dim3(a.nq), dim3(kMergeBesideThreads), pool, s, e0, e1, a);
    else IVF_LAUNCH(merge_kernel<kMergeThreads>, dim3(a.nq), dim3(kMergeThreads), pool, s, e0, e1, a);
    return hipGetLastError();
}

// =============================================================================================
// Layout build (the contiguous cluster-major region of Sec. "Implementation Details"): input
// rows scattered to their positions, one wavefront per row, 16 bytes per lane when rows allow.
// =============================================================================================
__global__ void scatter_rows_kernel(const unsigned char* src, unsigned char* dst, const int64_t* pos,
                                    int64_t n, size_t row_bytes) {
    const int lane = lane_id();
    int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t i = wave; i < n; i += nwaves) {
        const unsigned char* s = src + (size_t)i * row_bytes;
        unsigned char* d = dst + (size_t)pos[i] * row_bytes;
        if (row_bytes % 16 == 0) {
            for (size_t o = (size_t)lane * 16; o < row_bytes; o += 1024) *(uint4*)(d + o) = *(const uint4*)(s + o);
        } else {
            for (size_t o = lane; o < row_bytes; o += 64) d[o] = s[o];
        }
    }
}

hipError_t launch_scatter_rows(const void* src, void* dst, const int64_t* pos, int64_t n,
                               size_t row_bytes, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 3) / 4;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(scatter_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                       (const unsigned char*)src, (unsigned char*)dst, pos, n, row_bytes);
    return hipGetLastError();
}

// =============================================================================================
// Consolidation of the prefetch buffer (Sec. 4.2 "Cache design"; appendix: the GPU memory is
// consolidated after each batch).  One launch carries out a group of moves that do not disturb
// each other (no destination of the group overlaps a source of the group): the moves are cut
// into chunks of kMoveChunk bytes and every workgroup copies chunks, 16 bytes per lane where the
// addresses allow.  HBM-bound: every byte moved is read once and written once.
// =============================================================================================
constexpr uint32_t kMoveChunk = 64u << 10;

__global__ __launch_bounds__(256) void gather_moves_kernel(unsigned char* buf, const MoveDesc* moves, int n_moves,
                                                           uint32_t n_chunks) {
    for (uint32_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
        int lo = 0, hi = n_moves;                  // moves[lo].chunk0 <= ch < moves[hi].chunk0 (a sentinel past the end)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (moves[mid].chunk0 <= ch) lo = mid; else hi = mid;
        }
        const MoveDesc m = moves[lo];
        const uint64_t o = (uint64_t)(ch - m.chunk0) * kMoveChunk;
        const uint64_t len = min((uint64_t)kMoveChunk, m.bytes - o);
        const unsigned char* src = buf + m.from_byte + o;
        unsigned char* dst = buf + m.to_byte + o;
        if ((((uintptr_t)src | (uintptr_t)dst) & 15u) == 0) {
            const uint32_t vec = (uint32_t)(len / 16);
            // eight loads per lane in flight before the first store
#pragma unroll 1
            for (uint32_t i0 = 0; i0 < vec; i0 += 8 * 256) {
                uint4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t i = i0 + u * 256 + threadIdx.x;
                    v[u] = load_stream16(src + (size_t)min(i, vec - 1) * 16);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t i = i0 + u * 256 + threadIdx.x;
                    if (i < vec) store_stream16(dst + (size_t)i * 16, v[u]);
                }
            }
            for (uint64_t i = (uint64_t)vec * 16 + threadIdx.x; i < len; i += blockDim.x) dst[i] = src[i];
        } else {
            for (uint64_t i = threadIdx.x; i < len; i += blockDim.x) dst[i] = src[i];
        }
    }
}

uint32_t move_chunks(uint64_t bytes) { return (uint32_t)((bytes + kMoveChunk - 1) / kMoveChunk); }

hipError_t launch_gather_moves(void* buf, const MoveDesc* moves_dev, int n_moves, uint32_t n_chunks, int n_cu, hipStream_t s) {
    if (n_moves <= 0 || n_chunks == 0) return hipSuccess;
    const uint32_t grid = std::min<uint32_t>(n_chunks, (uint32_t)n_cu * 8u);
    hipLaunchKernelGGL(gather_moves_kernel, dim3(grid), dim3(256), 0, s, (unsigned char*)buf, moves_dev, n_moves, n_chunks);
    return hipGetLastError();
}

// =============================================================================================
// Prefetched clusters (Sec. 4.1 step 1): one launch reads all lists of a prefetch from pinned host memory and
// writes them to their places in the device buffer, in the order of the plan.  Bound by the link to the
// host: 16 workgroups with 32 KB on its way each reach 57 GB/s, what the copy engine reaches in one piece of 256 MB (8: 44
// for lists of 0.1 MB, 50 for larger ones; 4: 28 to 35).  Kernels beside it that deal their work out evenly wait for
// the units that fetch, with fewer of them no less.  Rows may start at any element: 16-byte stores to aligned places, from
// loads at any address.  (One hipMemcpyAsync per list: 23 GB/s for lists of 390 KB, half of a list's time
// passes before its first byte.)
// =============================================================================================
constexpr uint32_t kFetchWgs = 16;

__global__ __launch_bounds__(256) void fetch_lists_kernel(const unsigned char* lists, unsigned char* buf, const MoveDesc* moves,
                                                          int n_moves, uint32_t n_chunks) {
    constexpr int U = 8;                           // loads of a lane in flight
    for (uint32_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
        int lo = 0, hi = n_moves;                  // moves[lo].chunk0 <= ch < moves[hi].chunk0
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (moves[mid].chunk0 <= ch) lo = mid; else hi = mid;
        }
        const MoveDesc m = moves[lo];
        const uint64_t o = (uint64_t)(ch - m.chunk0) * kMoveChunk;
        const uint32_t len = (uint32_t)min((uint64_t)kMoveChunk, m.bytes - o);
        const unsigned char* src = lists + m.from_byte + o;
        unsigned char* dst = buf + m.to_byte + o;
        // to the first 16-byte boundary of the destination element by element (of 2 bytes), then 16 bytes at a
        // time, then the rest
        const uint32_t head = min((uint32_t)(-(uintptr_t)dst & 15u), len), vec = (len - head) / 16, tail = head + vec * 16;
        const uint32_t e = threadIdx.x * 2;
        if (e < head) *(uint16_t*)(dst + e) = *(const uint16_t*)(src + e);
        if (tail + e < len) *(uint16_t*)(dst + tail + e) = *(const uint16_t*)(src + tail + e);
#pragma unroll 1
        for (uint32_t i0 = 0; i0 < vec; i0 += U * 256) {
            uint4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = load_chunk<true>(src + head + (size_t)min(i0 + u * 256 + threadIdx.x, vec - 1) * 16);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = i0 + u * 256 + threadIdx.x;
                if (i < vec) store_stream16(dst + head + (size_t)i * 16, v[u]);
            }
        }
    }
}

hipError_t launch_fetch_lists(const void* lists_dev, void* buf, const MoveDesc* moves_dev, int n_moves, uint32_t n_chunks, hipStream_t s) {
    if (n_moves <= 0 || n_chunks == 0) return hipSuccess;
    hipLaunchKernelGGL(fetch_lists_kernel, dim3(std::min(n_chunks, kFetchWgs)), dim3(256), 0, s, (const unsigned char*)lists_dev,
                       (unsigned char*)buf, moves_dev, n_moves, n_chunks);
    return hipGetLastError();
}

// =============================================================================================
// Queries handed over in host memory: a few KB that a kernel reads from the pinned buffer itself
// (one dispatch on the search stream) instead of a copy engine transfer set up by the runtime.
// =============================================================================================
__global__ void stage_query_kernel(const float* src, float* dst, size_t n) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

// More than kStageOne floats: four to a load, four loads of a lane in flight, so that the link is busy throughout (an engine
// copy of 256 KB takes 10 us and the next one starts 10 us later).
constexpr size_t kStageOne = 16384;
__global__ __launch_bounds__(256) void stage_many_kernel(const float* src, float* dst, size_t n) {
    constexpr int U = 4;
    const size_t quads = n / 4, stride = (size_t)gridDim.x * 256 * U;
    for (size_t i0 = (size_t)blockIdx.x * 256 * U + threadIdx.x; i0 < quads; i0 += stride) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = ((const float4*)src)[min(i0 + u * 256, quads - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) if (i0 + u * 256 < quads) ((float4*)dst)[i0 + u * 256] = v[u];
    }
    if (blockIdx.x == 0 && threadIdx.x < n % 4) dst[quads * 4 + threadIdx.x] = src[quads * 4 + threadIdx.x];
}

hipError_t launch_stage_query(const float* src_pinned, float* dst, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (n > kStageOne && (((uintptr_t)src_pinned | (uintptr_t)dst) & 15u) == 0) {
        hipLaunchKernelGGL(stage_many_kernel, dim3((unsigned)std::min<size_t>((n / 4 + 1023) / 1024, 64)), dim3(256), 0, s, src_pinned, dst, n);
        return hipGetLastError();
    }
    const size_t blocks = std::min<size_t>((n + 255) / 256, 64);
    hipLaunchKernelGGL(stage_query_kernel, dim3((unsigned)blocks), dim3(256), 0, s, src_pinned, dst, n);
    return hipGetLastError();
}

// =============================================================================================
// Cluster cache bookkeeping (Sec. 4.2 "Cache design"; appendix: hotness h <- h / d, + h_inc when
// the cluster was used in the round).  hot[c] < 0 marks a cluster that is not cached.
// Single precision, one correctly rounded division and one addition per cluster.
// =============================================================================================
// reset: the cache starts over (hotness and use marks are dropped) before the admission
__global__ void cache_admit_kernel(float* hot, uint32_t* used, const int64_t* res_off, int nlist, float h_init, int reset) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nlist) return;
    if (reset) used[c] = 0u;
    float h = reset ? -1.f : hot[c];
    if (res_off[c] < 0) h = -1.f;
    else if (h < 0.f) h = h_init;            // fetched since the last call: cached from now on
    hot[c] = h;
}

__global__ void cache_round_kernel(float* hot, uint32_t* used, int nlist, float decay, float h_inc) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nlist) return;
    float h = hot[c];
    if (h >= 0.f) {
        h = h / decay;
        if (used[c]) h = h + h_inc;
        hot[c] = h;
    }
    used[c] = 0u;
}

hipError_t launch_cache_admit(float* hot, uint32_t* used, const int64_t* res_off, int nlist, float h_init, int reset,
                              hipStream_t s) {
    hipLaunchKernelGGL(cache_admit_kernel, dim3((nlist + 255) / 256), dim3(256), 0, s, hot, used, res_off, nlist, h_init, reset);
    return hipGetLastError();
}
hipError_t launch_cache_round(float* hot, uint32_t* used, int nlist, float decay, float h_inc, hipStream_t s) {
    hipLaunchKernelGGL(cache_round_kernel, dim3((nlist + 255) / 256), dim3(256), 0, s, hot, used, nlist, decay, h_inc);
    return hipGetLastError();
}

}  // namespace ivf
