// Small problems, unprotected: one launch per assignment, one per Lloyd iteration.
//
// Below some ten million multiplications an assignment is not bound by any unit but by its launches
// (norms, matrix kernel, settlement: 17 us for 20 000 x 24 points and 100 centroids, of which the matrix
// kernel computes for two), and an iteration by its seven (33 us at 4096 x 16, K = 8).  Here the
// centroids sit in LDS, a point in the registers of the P lanes that share its centroids, and distances
// are taken in direct-difference form in double (fp64 runs at the fp32 rate on the vector units here):
// nothing has to be prepared, certified or settled afterwards.
#include "ftk_internal.h"
#include "ftk_direct.h"
#include "ftk_mma.h"
#include "ftk_quads.h"
#include "ftk_small.h"

namespace ftk {

constexpr int SM_THREADS = 256;
constexpr int SM_CELLS = 8192;        // most elements of C (LDS)
constexpr int SM_FIT_CELLS = 4096;    // the same where a table of sums lies beside them
constexpr int SM_GRID = 512;
constexpr int SM_FILL = 256;          // workgroups to aim at: more lanes per point than that fills cost time (20000 x 24,
                                      // K = 100: 13.4 us; aiming at 1024: 15.4)
constexpr int SM_LIMB_BITS = 24;

// the update's fixed point (see ftk_update.hip): the same scale and rounding, so the same sums
__device__ __forceinline__ double small_scale(double absmax, int64_t rows)
{
    int L = 11;
    while (((int64_t)1 << L) < rows) ++L;
    if (!(absmax > 0.0) || !(absmax < __builtin_huge_val())) return 1.0;
    return ldexp(1.0, 62 - L - (ilogb(absmax) + 1));
}
__device__ __forceinline__ long long small_fixed(double x, double scale)
{
    constexpr double MAGIC = 6755399441055744.0;  // 1.5 * 2^52
    return __double_as_longlong(fma(x, scale, MAGIC)) - __double_as_longlong(MAGIC);
}

struct SmallArgs {
    const void *X;
    const void *C;       // centroids of this assignment, or (FIT, prev given) those before it
    int64_t N;
    int D, K, p_log2;
    int32_t *labels;     // may be NULL
    void *mindist;       // may be NULL
    // FIT
    const unsigned long long *prev;  // sums the centroids are formed from: [K*D] low, [K*D] high, then counts; or NULL
    unsigned long long *cur, *next;  // this iteration's, and the one to clear for the next
    void *C_out;         // where workgroup 0 leaves the centroids formed from prev
    const double *absmax;
    int64_t scale_rows;
    const double *partials_prev;     // objective of the previous iteration, by workgroup
    double *partials, *inertia_prev;
};

template <typename T>
__device__ __forceinline__ T small_mean(const unsigned long long *sums, int cells, int i, int n, double inv)
{
    const double total = (double)(long long)sums[cells + i] * (double)(1ll << SM_LIMB_BITS) + (double)(long long)sums[i];
    return (T)((total * inv) / (double)n);
}

// NQ quads of features, PT points per thread.
// AHEAD: the first rows are on their way while the centroids are formed (in a fit their means wait for the sums, then for
// divisions), and those of the next round while distances are taken (launch_small_t() tells when).
template <typename T, int NQ, int PT, bool FIT, bool AHEAD>
__global__ __launch_bounds__(SM_THREADS) void small_kernel(SmallArgs a)
{
    constexpr int E = 16 / sizeof(T);              // elements per LDS read
    constexpr int SU = (4 * NQ / E) | 1;           // 16-byte units per row: odd, so that rows spread over the banks
    extern __shared__ __align__(16) unsigned char lds_raw[];
    T *ldsC = reinterpret_cast<T *>(lds_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int D = a.D, K = a.K, cells = K * D;
    unsigned long long *tab = reinterpret_cast<unsigned long long *>(lds_raw + (size_t)K * SU * 16);
    int *cnt = reinterpret_cast<int *>(tab + (FIT ? cells : 0));
    const int P = 1 << a.p_log2, sub = tid & (P - 1);
    const T *X = reinterpret_cast<const T *>(a.X), *C = reinterpret_cast<const T *>(a.C);
    T *C_out = reinterpret_cast<T *>(a.C_out);

    const int per_wg = (SM_THREADS >> a.p_log2) * PT;  // points per workgroup and round
    // element d of point t goes to put(t, d, value, whether the row has it)
    auto read_rows = [&](int64_t p0, auto put) {
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            const int64_t p = p0 + (int64_t)t * (SM_THREADS >> a.p_log2) + (tid >> a.p_log2);
            const T *row = X + (p < a.N ? p : a.N - 1) * D;
            if (D % 4 == 0) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const Quad<T> f = load_quad<T>(row + min(4 * q, D - 4));
#pragma unroll
                    for (int e = 0; e < 4; ++e) put(t, 4 * q + e, f.v[e], 4 * q < D);
                }
            } else {
#pragma unroll
                for (int d = 0; d < 4 * NQ; ++d) put(t, d, row[min(d, D - 1)], d < D);
            }
        }
    };
    T raw[PT][AHEAD ? 4 * NQ : 1];
    auto request = [&](int64_t p0) {
        read_rows(p0, [&](int t, int d, T v, bool) { raw[t][d] = v; });
    };
    if constexpr (AHEAD) request((int64_t)blockIdx.x * per_wg);
    double scale = 1.0;
    if constexpr (FIT) scale = small_scale(*a.absmax, a.scale_rows);
    const double inv = 1.0 / scale;
    const int *prev_cnt = reinterpret_cast<const int *>(a.prev + 2 * (size_t)cells);
    for (int i = tid; i < K * 4 * NQ; i += SM_THREADS) {
        const int k = i / (4 * NQ), d = i - k * 4 * NQ;
        T v = T(0);
        if (d < D) {
            v = C[k * D + d];
            if (FIT && a.prev) {
                const int n = prev_cnt[k];
                if (n > 0) v = small_mean<T>(a.prev, cells, k * D + d, n, inv);  // an empty cluster keeps its centroid
                if (blockIdx.x == 0) C_out[k * D + d] = v;
            }
        }
        ldsC[k * (SU * E) + d] = v;
    }
    if constexpr (FIT) {
        for (int i = tid; i < cells; i += SM_THREADS) tab[i] = 0ull;
        for (int i = tid; i < K; i += SM_THREADS) cnt[i] = 0;
        int *next = reinterpret_cast<int *>(a.next);
        for (int64_t i = (int64_t)blockIdx.x * SM_THREADS + tid; i < 4 * (int64_t)cells + K; i += (int64_t)gridDim.x * SM_THREADS)
            next[i] = 0;
        if (a.partials_prev && blockIdx.x == 0 && tid < 64) {  // every iteration has the same grid
            double s = 0.0;
            for (int i = lane; i < (int)gridDim.x; i += 64) s += a.partials_prev[i];
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
            if (lane == 0) *a.inertia_prev = s;
        }
    }
    __syncthreads();

    double inertia = 0.0;
    for (int64_t p0 = (int64_t)blockIdx.x * per_wg; p0 < a.N; p0 += (int64_t)gridDim.x * per_wg) {
        double x[PT][4 * NQ];
        double best[PT];
        int bj[PT];
        bool live[PT];
        int64_t p[PT];
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            p[t] = p0 + (int64_t)t * (SM_THREADS >> a.p_log2) + (tid >> a.p_log2);
            live[t] = p[t] < a.N;
            if constexpr (AHEAD)
#pragma unroll
                for (int d = 0; d < 4 * NQ; ++d) x[t][d] = d < D ? (double)raw[t][d] : 0.0;
            best[t] = __builtin_huge_val();
            bj[t] = 0x7fffffff;
        }
        if constexpr (AHEAD) {
            if (p0 + (int64_t)gridDim.x * per_wg < a.N) request(p0 + (int64_t)gridDim.x * per_wg);
        } else {
            read_rows(p0, [&](int t, int d, T v, bool there) { x[t][d] = there ? (double)v : 0.0; });
        }
        for (int j = sub; j < K; j += P) {
            const T *c = ldsC + j * (SU * E);
            double d[PT];
#pragma unroll
            for (int t = 0; t < PT; ++t) d[t] = 0.0;
#pragma unroll
            for (int q = 0; q < 4 * NQ / E; ++q) {
                const typename Mma<T>::frag_t f = *reinterpret_cast<const typename Mma<T>::frag_t *>(c + q * E);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const double ce = (double)f[e];
#pragma unroll
                    for (int t = 0; t < PT; ++t) {
                        const double diff = x[t][q * E + e] - ce;
                        d[t] = fma(diff, diff, d[t]);  // in feature order: equal centroids tie exactly
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                const bool better = d[t] < best[t];
                best[t] = better ? d[t] : best[t];
                bj[t] = better ? j : bj[t];
            }
        }
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            for (int m = 1; m < P; m <<= 1) {
                const double od = __shfl_xor(best[t], m, 64);
                const int oj = __shfl_xor(bj[t], m, 64);
                const bool take = od < best[t] || (od == best[t] && oj < bj[t]);
                best[t] = take ? od : best[t];
                bj[t] = take ? oj : bj[t];
            }
            const int lab = bj[t] == 0x7fffffff ? 0 : bj[t];  // no distance was a number
            if (live[t] && sub == 0) {
                if (a.labels) a.labels[p[t]] = lab;
                if (a.mindist) reinterpret_cast<T *>(a.mindist)[p[t]] = (T)best[t];
                if (FIT) {
                    inertia += (double)(T)best[t];
                    atomicAdd(&cnt[lab], 1);
                }
            }
            if constexpr (FIT) {
                if (live[t]) {
#pragma unroll
                    for (int d = 0; d < 4 * NQ; ++d)
                        if ((d & (P - 1)) == sub && d < D)
                            atomicAdd(&tab[lab * D + d], (unsigned long long)small_fixed(x[t][d], scale));
                }
            }
        }
    }
    if constexpr (FIT) {
        __shared__ double sh_in[SM_THREADS / 64];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) inertia += __shfl_xor(inertia, m, 64);
        if (lane == 0) sh_in[tid >> 6] = inertia;
        __syncthreads();
        if (tid == 0) a.partials[blockIdx.x] = (sh_in[0] + sh_in[1]) + (sh_in[2] + sh_in[3]);
        // integer sums: the order of these additions does not matter.  fp32: one limb scaled for all of N;
        // fp64: scaled for this workgroup's rows, so the total needs two
        for (int i = tid; i < cells; i += SM_THREADS) {
            const long long v = (long long)tab[i];
            if (v == 0) continue;
            if (sizeof(T) == 4) {
                atomicAdd(a.cur + i, (unsigned long long)v);
            } else {
                atomicAdd(a.cur + i, (unsigned long long)(v & ((1ll << SM_LIMB_BITS) - 1)));
                atomicAdd(a.cur + cells + i, (unsigned long long)(v >> SM_LIMB_BITS));
            }
        }
        int *cur_cnt = reinterpret_cast<int *>(a.cur + 2 * (size_t)cells);
        for (int i = tid; i < K; i += SM_THREADS)
            if (cnt[i]) atomicAdd(cur_cnt + i, cnt[i]);
    }
}

// What the first iteration needs of a few points, in one workgroup: the largest |x| (as absmax_kernel finds it), a
// cleared table.  4096 x 16: 4.6 us against three launches and the gaps between them.
constexpr int SM_PREPARE = 131072;  // elements
template <typename T>
__global__ __launch_bounds__(1024) void small_prepare_kernel(const T *X, int count, double *absmax, int32_t *table, int words)
{
    __shared__ double sh[16];
    const int tid = threadIdx.x;
    T m = T(0);
    auto add = [&](T x) {
        const T v = fabs(x);
        m = (v > m && v < Mma<T>::huge()) ? v : m;  // NaN and Inf never raise the maximum
    };
    const int quads = count / 4;
#pragma unroll 8
    for (int i = tid; i < quads; i += 1024) {
        const Quad<T> q = load_quad<T>(X + 4 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e) add(q.v[e]);
    }
    if (4 * quads + tid < count) add(X[4 * quads + tid]);
    for (int i = tid; i < words; i += 1024) table[i] = 0;
    double d = (double)m;
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) d = fmax(d, __shfl_xor(d, k, 64));
    if ((tid & 63) == 0) sh[tid >> 6] = d;
    __syncthreads();
    if (tid == 0) {
        for (int i = 1; i < 16; ++i) d = fmax(d, sh[i]);
        *absmax = d;
    }
}

// centroids, counts and objective of the last iteration
template <typename T>
__global__ __launch_bounds__(256) void small_finish_kernel(const unsigned long long *sums, const T *C_prev, T *C_out,
                                                           int32_t *counts, int D, int K, const double *absmax,
                                                           int64_t scale_rows, const double *partials, int n_partials,
                                                           double *inertia)
{
    const int cells = K * D, i = blockIdx.x * 256 + threadIdx.x;
    const int *cnt = reinterpret_cast<const int *>(sums + 2 * (size_t)cells);
    if (i < cells) {
        const int n = cnt[i / D];
        C_out[i] = n > 0 ? small_mean<T>(sums, cells, i, n, 1.0 / small_scale(*absmax, scale_rows)) : C_prev[i];
    }
    if (i < K) counts[i] = cnt[i];
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        double s = 0.0;
        for (int k = threadIdx.x; k < n_partials; k += 64) s += partials[k];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
        if (threadIdx.x == 0) *inertia = s;
    }
}

// ---- host ----------------------------------------------------------------------------------------
static int small_quads(int D) { return D <= 8 ? 2 : (D <= 16 ? 4 : (D <= 24 ? 6 : (D <= 32 ? 8 : (D <= 48 ? 12 : 16)))); }
static int small_points(int nq) { return nq <= 8 ? 2 : 1; }

// Where one launch wins: up to about 5 * 10^7 multiplications (whole calls, before / here: fp32 20000 x 24,
// K = 100 15.6 / 13.9 us; 10^5 x 8, K = 64 14.5 / 10.9; 10^5 x 4, K = 100 15.4 / 15.1; 1000 x 16, K = 32 10.6 / 4.7;
// fp64 20000 x 32, K = 64 13.4 / 12.9; 10^6 x 8, K = 2 43 / 13).  Rows of more than 32 doubles take one point per
// thread, and more centroids or points than a few outweigh the launches: 20000 x 64, K = 8 12.4 / 8.1, K = 32
// 12.7 / 15.8; 10^5 x 45, K = 8 20 / 31.
static bool small_work(ftk_dtype dtype, int64_t N, int D, int K)
{
    const double work = (double)N * K * D;
    if (dtype == FTK_F64 && D > 32) return work <= 2e7 && N <= 32768;
    return work <= 5e7;
}

bool small_assign_fits(ftk_dtype dtype, int64_t N, int D, int K)
{
    return D <= 64 && (int64_t)K * small_quads(D) * 4 <= SM_CELLS && small_work(dtype, N, D, K);
}
// An assignment of longer rows is faster with several lanes a row, see ftk_direct.hip (this kernel / that one): fp32
// 6521 x 57, K = 95 15.8 / 12.2 us, 58896 x 52, K = 12 12.9 / 10.9, but 32803 x 48, K = 17 11.2 / 14.9, where a third
// of its last group of centroids is padding, and 9429 x 39, K = 70 14.0 / 17.4, 13186 x 54, K = 67 17.0 / 20.1,
// 22036 x 48, K = 44 13.8 / 15.9, 17320 x 39, K = 67 19.0 / 22.6, where the last of several rounds of centroids or
// features is nearly empty (one round 6303 x 62, K = 69 13.5 / 12.1, 15822 x 53, K = 46 13.9 / 12.0; no features left
// over 42028 x 51, K = 17 19.8 / 16.4); ragged ones with few centroids 600000 x 10, K = 4 13.7 / 9.2, 600000 x 25
// 49 / 27, but 600000 x 15 14.6 / 15.4; fp64 4278 x 25, K = 91 18.2 / 9.4, 28555 x 19, K = 17 9.4 / 7.9, but
// 185114 x 23, K = 10 17 / 29, 20000 x 20, K = 100 14.3 / 18.9, 60000 x 28, K = 26 11.7 / 13.6 (ragged 60000 x 25,
// K = 26 13.5 / 11.8, x 31 13.1 / 13.9).
bool small_assign_pays(ftk_dtype dtype, int64_t N, int D, int K)
{
    if (!small_assign_fits(dtype, N, D, K)) return false;
    if (dtype == FTK_F32) {
        if (K <= 4 && D > 8 && D < 32 && D != 15 && D % 4 != 0) return false;
        if (D <= 32 || (D % 4 == 0 && K > 8 && 5 * ceil_div(K, 8) * 8 >= 7 * (int64_t)K)) return true;
        const DirectPlan p = cut_direct(dtype, N, D, K);
        const int round = p.kg << p.tc_log2;  // centroids of one
        if (K <= 16 || K <= round) return false;
        const double centroids = (double)ceil_div(K, round) * round / K, features = (double)ceil_div(D / 4, p.lanes) * p.lanes * 4 / D;
        return features >= 1 && (centroids >= 1.42 || centroids * features >= 1.58);
    }
    const double work = (double)N * D * K;
    if (D > 24) return D <= 32 && (D % 4 == 0 || D >= 30) && work >= 2.5e7;
    return D <= 16 || N >= 60000 || work >= (D > 20 ? 1.5e7 : 2.5e7);
}

bool small_fit_pays(ftk_dtype dtype, int64_t N, int D, int K)
{
    return D <= 64 && (int64_t)K * small_quads(D) * 4 <= SM_FIT_CELLS && small_work(dtype, N, D, K);
}

size_t small_fit_bytes(int D, int K)
{
    if (D > 64 || (int64_t)K * small_quads(D) * 4 > SM_FIT_CELLS) return 0;
    return 3 * align_up(((size_t)2 * K * D) * 8 + (size_t)K * 4, 256) + align_up((size_t)K * D * 8, 256);
}

// lanes per point: as many as give every compute unit a workgroup, at most one centroid each
static int small_lanes_log2(int64_t N, int K, int pt, int *grid)
{
    int l = 0;
    while (l < 5 && (2 << l) <= K && ((N << l) / pt) < (int64_t)SM_FILL * SM_THREADS) ++l;
    const int64_t wgs = ceil_div(N, (int64_t)(SM_THREADS >> l) * pt);
    *grid = (int)(wgs < SM_GRID ? wgs : SM_GRID);
    return l;
}

// Rows ahead, us without / with: fp32 20000 x 24, K = 100 13.9 / 13.1, 700000 x 20, K = 3 16.6 / 14.6, fit of
// 4096 x 16, K = 8, ten iterations 139 / 136; 14 doubles and more that are read one by one, 200000 x 15, K = 9
// 12.3 / 9.9, 700000 x 22, K = 3 51 / 36. Longer rows and other doubles pay for the registers with a wave:
// 60000 x 32, K = 26 10.6 / 12.0; fp64 700000 x 9, K = 3 14.7 / 16.0, 700000 x 16, K = 3 19.0 / 21.5, 60000 x 20,
// K = 26 9.7 / 10.3, fit of 20000 x 32, K = 20, five iterations 159 / 206.
template <typename T, bool FIT>
static void launch_small_t(const SmallArgs &a, int grid, hipStream_t st)
{
    const int nq = small_quads(a.D);
    const size_t row = (size_t)((4 * nq * sizeof(T) / 16) | 1) * 16;
    const size_t lds = (size_t)a.K * row + (FIT ? (size_t)a.K * a.D * 8 + (size_t)a.K * 4 : 0);
    const dim3 g((unsigned)grid), b(SM_THREADS);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, b, lds, st, a); };
    constexpr bool F32 = sizeof(T) == 4;
    const bool ahead = F32 || (!FIT && a.D > 13 && a.D % 4 != 0);
    switch (nq) {
    case 2: launch(small_kernel<T, 2, 2, FIT, F32>); break;
    case 4: launch(ahead ? small_kernel<T, 4, 2, FIT, F32 || !FIT> : small_kernel<T, 4, 2, FIT, F32>); break;
    case 6: launch(ahead ? small_kernel<T, 6, 2, FIT, F32 || !FIT> : small_kernel<T, 6, 2, FIT, F32>); break;
    case 8: launch(small_kernel<T, 8, 2, FIT, false>); break;
    case 12: launch(small_kernel<T, 12, 1, FIT, false>); break;
    default: launch(small_kernel<T, 16, 1, FIT, false>); break;
    }
}

ftk_status launch_small_assign(const AssignCall &c, hipStream_t st)
{
    SmallArgs a = {};
    a.X = c.X;
    a.C = c.C;
    a.N = c.N;
    a.D = c.D;
    a.K = c.K;
    a.labels = c.labels;
    a.mindist = c.mindist;
    int grid;
    a.p_log2 = small_lanes_log2(c.N, c.K, small_points(small_quads(c.D)), &grid);
    if (c.dtype == FTK_F32) launch_small_t<float, false>(a, grid, st);
    else launch_small_t<double, false>(a, grid, st);
    FTK_TRY_HIP(hipGetLastError());
    return FTK_OK;
}

// Iteration t adds into table t % 3 and clears the next one; the centroids of iteration t + 1 are formed
// from it by every workgroup for itself, in the launch that uses them.
ftk_status launch_small_fit(ftk_dtype dtype, const void *X, int64_t N, int D, int K, int iters, const void *C_first, void *C_cur,
                            void *C_out, int32_t *labels, int32_t *counts, double *absmax, double *inertia, double *partials,
                            void *scratch, hipStream_t st)
{
    const size_t cells = (size_t)K * D;
    const size_t table = align_up(2 * cells * 8 + (size_t)K * 4, 256);
    char *base = (char *)scratch;
    auto tab = [&](int t) { return reinterpret_cast<unsigned long long *>(base + (size_t)(t % 3) * table); };
    void *C_alt = base + 3 * table;
    SmallArgs a = {};
    a.X = X;
    a.N = N;
    a.D = D;
    a.K = K;
    const int pt = small_points(small_quads(D));
    int grid;
    a.p_log2 = small_lanes_log2(N, K, pt, &grid);
    const int64_t per_wg = (int64_t)(SM_THREADS >> a.p_log2) * pt;
    a.scale_rows = dtype == FTK_F32 ? N : ceil_div(ceil_div(N, per_wg), grid) * per_wg;
    a.absmax = absmax;
    const int words = (int)(4 * cells + K);
    int32_t *const first = reinterpret_cast<int32_t *>(tab(0));
    if (N * D <= SM_PREPARE && words <= SM_PREPARE) {
        if (dtype == FTK_F32)
            hipLaunchKernelGGL(small_prepare_kernel<float>, dim3(1), dim3(1024), 0, st, (const float *)X, (int)(N * D), absmax, first, words);
        else
            hipLaunchKernelGGL(small_prepare_kernel<double>, dim3(1), dim3(1024), 0, st, (const double *)X, (int)(N * D), absmax, first, words);
    } else {
        FTK_TRY(launch_absmax(dtype, X, N * (int64_t)D, absmax, first, words, st));
    }
    void *C_buf[2] = {C_cur, C_alt};
    for (int t = 0; t < iters; ++t) {
        // centroids before the update of iteration t - 1 are in C_buf[(t - 1) & 1]; those after go to the other
        a.C = t <= 1 ? C_first : C_buf[(t - 1) & 1];
        a.C_out = C_buf[t & 1];
        a.prev = t == 0 ? nullptr : tab(t - 1);
        a.cur = tab(t);
        a.next = tab(t + 1);
        a.labels = t == iters - 1 ? labels : nullptr;  // those of the last assignment are what is asked for
        a.partials = partials + (t & 1) * SM_GRID;
        a.partials_prev = t == 0 ? nullptr : partials + ((t - 1) & 1) * SM_GRID;
        a.inertia_prev = t == 0 ? nullptr : inertia + t - 1;
        ProfileMark mark;
        FTK_TRY(profile_begin(mark, st));
        if (dtype == FTK_F32) launch_small_t<float, true>(a, grid, st);
        else launch_small_t<double, true>(a, grid, st);
        FTK_TRY(profile_end(mark, st));
    }
    const dim3 g((unsigned)ceil_div((int64_t)cells > K ? (int64_t)cells : K, 256));
    const int last = iters - 1;
    const void *const C_prev = last == 0 ? C_first : C_buf[last & 1];
    if (dtype == FTK_F32)
        hipLaunchKernelGGL((small_finish_kernel<float>), g, dim3(256), 0, st, tab(last), (const float *)C_prev,
                           (float *)C_out, counts, D, K, absmax, a.scale_rows, partials + (last & 1) * SM_GRID, grid,
                           inertia + last);
    else
        hipLaunchKernelGGL((small_finish_kernel<double>), g, dim3(256), 0, st, tab(last), (const double *)C_prev,
                           (double *)C_out, counts, D, K, absmax, a.scale_rows, partials + (last & 1) * SM_GRID, grid,
                           inertia + last);
    FTK_TRY_HIP(hipGetLastError());
    return FTK_OK;
}

}  // namespace ftk
