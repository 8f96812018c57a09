// Unprotected assignment in one launch: every distance in direct-difference form (Section 3.1.1), in double.
//
// The matrix kernels need norms ahead and a settlement behind, and cut the points into blocks of 128 or 256: three
// launches, and too few workgroups where points are few (14665 x 520, K = 2: 115 of them, 33 us a call; 1278 x 639,
// K = 43: ten). With few centroids they stay below the memory's rate too (426483 x 126, K = 2: 62 us, X read at 3.5
// TB/s).  Here fp64 arithmetic runs on the vector units at the fp32 rate, two instructions a multiplication, and
// nothing has to be prepared, certified or settled: what a call below some 10^8 .. 10^9 multiplications spends on
// launches is more.
//
// L lanes share the features of a row (row-contiguous 16-byte pieces), each of them for R points against KG centroids at
// a time: R + KG loads for 4 R KG differences, so that the vector units and not the caches set the pace.  TC such groups
// take different centroids of the same points, the rest of the workgroup other points.  How L and TC are chosen: see
// cut_direct().
#include <type_traits>

#include "ftk_internal.h"
#include "ftk_direct.h"
#include "ftk_quads.h"

namespace ftk {

constexpr int DR_THREADS = 256;
constexpr int DR_R = 4;  // points of a lane
static int direct_group(int K) { return K <= 2 ? 2 : (K <= 4 ? 4 : 8); }  // centroids of a lane at a time

struct DirectArgs {
    int64_t N;
    int D, K, tc_log2;
    int32_t *labels;
    void *mindist;  // may be NULL
};

template <typename T, int L, int KG>
__global__ __launch_bounds__(DR_THREADS) void direct_kernel(const T *X, const T *C, DirectArgs a)
{
    constexpr int R = DR_R;
    const int tid = threadIdx.x;
    const int sub = tid & (L - 1);
    const int TC = 1 << a.tc_log2, tc = (tid / L) & (TC - 1);
    const int TP = DR_THREADS / L >> a.tc_log2, tp = (tid / L) >> a.tc_log2;
    const int D = a.D, K = a.K, Dq = D & ~3;
    const int64_t first = (int64_t)blockIdx.x * (R * TP);
    const T *const X0 = X + first * D;
    unsigned xo[R];  // rows of the points, from the workgroup's first one
#pragma unroll
    for (int u = 0; u < R; ++u) xo[u] = (unsigned)(min((int64_t)(u * TP + tp), a.N - 1 - first) * D);
    double best[R];
    int bj[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        best[u] = __builtin_huge_val();
        bj[u] = 0x7fffffff;
    }
    for (int k0 = 0; k0 < K; k0 += TC * KG) {
        const int kb = k0 + tc * KG;
        unsigned co[KG];
#pragma unroll
        for (int r = 0; r < KG; ++r) co[r] = (unsigned)min(kb + r, K - 1) * (unsigned)D;
        double d[R][KG];
#pragma unroll
        for (int u = 0; u < R; ++u)
#pragma unroll
            for (int r = 0; r < KG; ++r) d[u][r] = 0.0;
        if (Dq) {  // (the last piece of a row is requested again in place of the one behind it)
            Quad<T> xn[R];
#pragma unroll
            for (int u = 0; u < R; ++u) xn[u] = load_quad<T>(X0 + (xo[u] + (unsigned)min(4 * sub, Dq - 4)));
            for (int f = 4 * sub; f < Dq; f += 4 * L) {
                double x[R][4];
#pragma unroll
                for (int u = 0; u < R; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[u][e] = (double)xn[u].v[e];
                const unsigned fn = (unsigned)min(f + 4 * L, Dq - 4);
#pragma unroll
                for (int u = 0; u < R; ++u) xn[u] = load_quad<T>(X0 + (xo[u] + fn));
#pragma unroll
                for (int r = 0; r < KG; ++r) {
                    const Quad<T> c = load_quad<T>(C + (co[r] + (unsigned)f));
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double ce = (double)c.v[e];
#pragma unroll
                        for (int u = 0; u < R; ++u) {
                            const double t = x[u][e] - ce;
                            d[u][r] = fma(t, t, d[u][r]);  // the same order for every centroid: equal ones tie exactly
                        }
                    }
                }
            }
        }
        for (int f = Dq + sub; f < D; f += L)
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const double x = (double)X0[xo[u] + (unsigned)f];
#pragma unroll
                for (int r = 0; r < KG; ++r) {
                    const double t = x - (double)C[co[r] + (unsigned)f];
                    d[u][r] = fma(t, t, d[u][r]);
                }
            }
#pragma unroll
        for (int u = 0; u < R; ++u)
#pragma unroll
            for (int r = 0; r < KG; ++r) {
                double v = d[u][r];
                if constexpr (L > 1) v = group_sum<L>(v);
                const bool better = v < best[u] && kb + r < K;  // indices increase: the first of equal ones stays
                best[u] = better ? v : best[u];
                bj[u] = better ? kb + r : bj[u];
            }
    }
    // the groups that took other centroids: those of this wave, then those of the others
    auto take = [&](int u, double od, int oj) {
        const bool other = od < best[u] || (od == best[u] && oj < bj[u]);
        best[u] = other ? od : best[u];
        bj[u] = other ? oj : bj[u];
    };
    const int span = L << a.tc_log2;
    for (int m = L; m < span && m < 64; m <<= 1)
#pragma unroll
        for (int u = 0; u < R; ++u) take(u, __shfl_xor(best[u], m, 64), __shfl_xor(bj[u], m, 64));
    if (span > 64) {
        __shared__ double sh_d[DR_THREADS / 64][R];
        __shared__ int sh_j[DR_THREADS / 64][R];
        const int wave = tid >> 6;
        if ((tid & 63) == 0)
#pragma unroll
            for (int u = 0; u < R; ++u) {
                sh_d[wave][u] = best[u];
                sh_j[wave][u] = bj[u];
            }
        __syncthreads();
        const int first_wave = wave & ~(span / 64 - 1);
        for (int w = first_wave; w < first_wave + span / 64; ++w)
#pragma unroll
            for (int u = 0; u < R; ++u) take(u, sh_d[w][u], sh_j[w][u]);
    }
    if ((tid & (span - 1)) == 0)
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int64_t p = first + u * TP + tp;
            if (p < a.N) {
                a.labels[p] = bj[u] == 0x7fffffff ? 0 : bj[u];  // no distance was a number
                if (a.mindist) static_cast<T *>(a.mindist)[p] = (T)best[u];
            }
        }
}

// ---- host ----------------------------------------------------------------------------------------
// Lanes that share a row: enough that they read whole lines of it, few enough that each has several pieces (what the
// lanes of a row have is added up once per centroid).  Groups of lanes on other centroids of the same points: until
// 65536 threads are busy (and while four of them take all centroids of long rows: one read of X); where that does not
// do, more lanes per row.  Of 41 shapes timed with every choice (10^3 .. 10^6 points, 4 .. 1000 features, 2 .. 700
// centroids, both types) this one is near the best: 1286 x 73, K = 110 9.1 / 9.1 us, 1278 x 639, K = 43 15.7 / 14.1,
// 14665 x 520, K = 2 8.9 / 7.2.
// Up to four centroids the rows are all that a call waits for: twice the lanes ask for twice as much of a row at once
// (such lanes / twice as many: 480049 x 60, K = 2 34 / 25, 46418 x 316, K = 3 18.5 / 14.5, fp64 1585025 x 70, K = 2
// 250 / 187, 1592522 x 32, K = 1 114 / 80, fp32 1800000 x 14, K = 1 57 / 25, fp64 x 15, K = 3 170 / 81; four or eight
// lanes: 700000 x 52, K = 1 41 / 30, 44 31 / 28, 36 24 / 25, fp64 700000 x 34, K = 1 47 / 33, 1200000 x 48, K = 4
// 98 / 113), but for fp32 data that the memory-side cache holds anyway (121474 x 108, K = 2 12.2 / 13.4, 54590 x 256
// 11.2 / 13.3).  So do few doubles, whose rows are as long as those of twice as many floats (50000 x 29, K = 8
// 11.3 / 9.5, 4000 x 56, K = 50 11.5 / 9.3), until the vector units set the pace (20000 x 17, K = 40 10.0 / 11.5,
// 20000 x 25, K = 60 12.0 / 15.2).
DirectPlan cut_direct(ftk_dtype dtype, int64_t N, int D, int K)
{
    DirectPlan p = {};
    p.kg = direct_group(K);
    const bool f64 = dtype == FTK_F64;
    const bool twice = f64 ? K <= 4 || (double)N * D * K < (D > 32 ? 2e7 : 1.2e7)
                           : K <= 4 && (D <= 112 ? (double)N * D >= (D < 16 ? 1e7 : 1.6e7) : N < 50000);
    const int four = K > 4 ? 56 : (K > 2 ? 48 : (f64 ? 32 : 42));  // most features of four lanes, twice as many as usual
    if (twice) p.lanes = D <= 8 ? 1 : (D <= 16 ? 2 : (D <= four ? 4 : (D <= 224 ? 8 : 16)));
    else p.lanes = D <= 15 ? 1 : (D <= 32 ? 2 : (D <= 112 ? 4 : (D <= 448 ? 8 : 16)));
    const int64_t groups = ceil_div(K, p.kg), quads = ceil_div(N, DR_R);
    auto threads = [&] { return (quads * p.lanes) << p.tc_log2; };
    while ((1 << p.tc_log2) < groups && (p.lanes << p.tc_log2) < DR_THREADS && (threads() < 65536 || (groups <= 4 && D >= 64))) ++p.tc_log2;
    while (p.lanes < 32 && (f64 ? 8 : 16) * p.lanes <= D && (p.lanes << p.tc_log2) < DR_THREADS && threads() < 40000) p.lanes *= 2;
    return p;
}

// Where one launch of double arithmetic beats the matrix kernels behind their norms and ahead of their refine kernel:
// 1400 random shapes of 500 .. 2 * 10^6 points, 2 .. 1024 features, 2 .. 1000 centroids and up to 10^9
// multiplications timed with both, and 900 again with the matrix kernels' rows by lines (matrix / this, whole calls,
// geometric means of the second lot): fp32 up to 7 * 10^7 multiplications 2.0, with up to 4 centroids 1.4 at any
// size, fp64 1.9 and 1.2; centroids that fill up the last group count like others.  Near the lines, us:
//   fp32  16438 x 672, K = 13 45 / 47; 159477 x 576, K = 3 80 / 75; 35681 x 216, K = 12 31 / 30; 50387 x 128, K = 16 18 / 17; 132339 x 41,
//         K = 9 18 / 25; 33607 x 7, K = 278 20 / 27; 146809 x 124, K = 8 32 / 34; 478244 x 51, K = 5 49 / 41; 641930 x 2, K = 110 53 / 38
//   fp64  393442 x 86, K = 2 70 / 58; 54801 x 136, K = 8 20.6 / 21.3; 333471 x 36, K = 5 33 / 36; 95490 x 56, K = 9 17.6 / 27.6; 2627 x 635,
//         K = 84 69 / 50; 300000 x 100, K = 20 67 / 162
// Rows of up to 64 features fill a few rounds of their lanes, and few groups of centroids a few rounds: where there
// are many points the line lies by what the rounds hold (47873 x 52, K = 22 17.0 / 18.8, 74775 x 36, K = 21
// 15.3 / 22.3, 58280 x 51, K = 15 15.3 / 10.0; 34278 x 20, K = 91 16.4 / 21.2, 69142 x 12, K = 79 17.1 / 22.9,
// 51448 x 31, K = 37 14.7 / 20.9, 26719 x 16, K = 127 15.7 / 13.0; fp64 33958 x 58, K = 20 16.8 / 21.9, 16727 x 58,
// K = 48 16.1 / 22.1, 10630 x 54, K = 77 18.8 / 22.8, 66468 x 38, K = 10 14.4 / 18.3, 50704 x 59, K = 10
// 15.5 / 14.0).
// Two lanes to rows of almost their eight quads ask for too little at once where there are many
// (10^6 x 32, K = 8 47 / 60); rows of two or three features have nothing to share out among many centroids' groups
// (333333 x 2, K = 150 46 / 35, 166666 x 2, K = 600 55 / 70; fp64 277777 x 3, K = 300 66 / 90).
bool direct_pays(ftk_dtype dtype, int64_t N, int D, int K)
{
    const double work = (double)N * D * K;
    if (K <= 4) return work <= (dtype == FTK_F32 ? 1e9 : 4e8);
    const int KG = direct_group(K);
    const double filled = D < 16 ? work : (double)N * D * (ceil_div(K, KG) * KG);
    if (K > 8 && D > (dtype == FTK_F32 ? 8 : 32) && D <= 64 && N >= (dtype == FTK_F64 ? 8000 : (D > 32 ? 30000 : 16000))) {
        const DirectPlan p = cut_direct(dtype, N, D, K);
        const int64_t centroids = (int64_t)KG << p.tc_log2, features = 4 * p.lanes;  // of a round
        const double rounds = (double)ceil_div(K, centroids) * centroids * (ceil_div(D / 4, p.lanes) * features + D % 4);
        if ((double)N * rounds > (dtype == FTK_F32 ? (D > 32 ? 7.2e7 : 7.6e7) : (N < 16000 ? 8.2e7 : 5.1e7))) return false;
    }
    if (dtype == FTK_F32) {
        if (D > 24 && D <= 32 && N > 500000) return false;
        if (K <= 8) return work <= (D < 64 ? 1.5e8 : 1.1e8);
        return filled <= (D < 16 && K > 100 ? 5e7 : 7e7) || (N <= 8000 && work <= 1e8) || (D < 4 && K <= 200 && work <= 2e8);
    }
    if (K <= 8) return filled <= 7e7 || (N <= 8000 && work <= 1.5e8) || (D < 4 && work <= 2.5e8);
    return filled <= 5e7 || (N <= 8000 && work <= 1.5e8) || (D < 4 && K <= 200 && work <= 2.5e8);
}

template <typename T>
static void launch_direct_t(const AssignCall &c, const DirectPlan &p, hipStream_t st)
{
    DirectArgs a = {};
    a.N = c.N;
    a.D = c.D;
    a.K = c.K;
    a.labels = c.labels;
    a.mindist = c.mindist;
    a.tc_log2 = p.tc_log2;
    const int64_t points = (int64_t)DR_R * (DR_THREADS / p.lanes >> p.tc_log2);
    const dim3 grid((unsigned)ceil_div(c.N, points)), block(DR_THREADS);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, st, (const T *)c.X, (const T *)c.C, a); };
#define FTK_LAUNCH_DIRECT(L)                                    \
    case L:                                                     \
        if (p.kg == 2) launch(direct_kernel<T, L, 2>);          \
        else if (p.kg == 4) launch(direct_kernel<T, L, 4>);     \
        else launch(direct_kernel<T, L, 8>);                    \
        break
    switch (p.lanes) {
        FTK_LAUNCH_DIRECT(1);
        FTK_LAUNCH_DIRECT(2);
        FTK_LAUNCH_DIRECT(4);
        FTK_LAUNCH_DIRECT(8);
        FTK_LAUNCH_DIRECT(16);
        FTK_LAUNCH_DIRECT(32);
    }
#undef FTK_LAUNCH_DIRECT
}

ftk_status launch_direct_assign(const AssignCall &c, const DirectPlan &p, hipStream_t st)
{
    if (c.dtype == FTK_F32) launch_direct_t<float>(c, p, st);
    else launch_direct_t<double>(c, p, st);
    FTK_TRY_HIP(hipGetLastError());
    return FTK_OK;
}

}  // namespace ftk
