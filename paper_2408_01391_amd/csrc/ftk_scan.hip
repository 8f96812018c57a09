// Assignment without fault tolerance for fp32 and fp64 data, in three passes:
//
//   scan    the contraction on the 16-bit matrix instructions, both operands split into two bf16 pieces (large
//           calls: rounded to one fp16 piece), fp32 accumulation.  Per point it keeps the best score, its centroid and the second-best
//           score - nothing else;
//   settle  the distance to the named centroid in direct-difference form, in the data's own type
//           (Section 3.1.1; in double where either form may run), and the decision whether the scan could be trusted: where the two best
//           scores are closer than the scan's error bound the point is listed;
//   resolve the listed points: every centroid whose score lies within the bound of the best is
//           evaluated in double; where there are many of those, all centroids on the matrix instructions
//           of the data's type, and what these cannot tell apart in double.
//
// Results are therefore those of the fp32 / fp64 matrix kernels - labels exact up to the documented
// ties, distances direct - while the contraction runs on hardware that does 16 (fp32) or 32 (fp64)
// times as many multiplications a second.
//
// Error of a score.  A value is x = x0 + x1 + r with x0 = bf16(x), x1 = bf16(x - x0), the same for c.  A
// piece rounds to nearest at 8 significant bits: |x1| up to 2^-8 |x|, |r| up to 2^-17 |x|.  Kept are
// x0c0 + x0c1 + x1c0; lost are x1c1, r.c and x.r', by Cauchy-Schwarz at most
//     ||x1|| ||c1|| + ||r_x|| ||c|| + ||x|| ||r_c||.
// That is up to 512 u of ||x|| ||c|| (u = 2^-24) where every feature sits at a midpoint of the rounding.  The
// largest ratios ||c1|| / ||c|| and ||r_c|| / ||c|| are measured by the preparation, which leaves 280 u on data at
// large.  (Norms of the points' pieces measured by the settle pass as well would leave 130 u, but cost it more
// than the points they save: 300007 x 45, K = 333 70.8 us a call against 66, 2^18 x 128, K = 256 103 against 97.)
// An instruction rounds to within 7 u of what it adds up (measured, pinned by a test), at most
// ||x|| ||c|| + ||c||^2 / 2: 21 u per block of 16 features.  Rows of up to 8 features leave half of a block
// empty, which holds the three-piece form (six products; 24 bits in three pieces, what is lost is 2 u) in
// the same three instructions; rows of up to 16 take that form in six, because short rows in many clusters
// have norms far above their distances and the wider band lists too many of them (10^6 x 16 in a box of
// 200, K = 200: a tenth of the points).
//
// All of this is in proportion to ||x|| ||c||, the distances are not: of data far from the origin every
// point would have to be settled (2^18 x 32 at 1000, spread 5, K = 1024: 6.2 ms, against 88 us at the origin).
// Distances do not change when everything moves, so a vector r, the trimmed mean of eight centroid rows, is
// taken off the centroids (in the data's type, before the split) where these rows say that it shortens them:
//     x.c - ||c||^2 / 2 = x.(c - r) - (r.(c - r) + ||c - r||^2 / 2) + a term without c,
// and the start value makes up for it.  The bound is then in proportion to (||x|| + ||r||) ||c - r||.  (Taken off
// the points as well it would be ||x - r|| ||c - r||, but their share of it costs the streaming scan 3 (fp32) to
// 20 % (fp64) on any data, and matters for offsets of more than about 10^4 spreads only.)
//
// One far centroid must not widen the band of all points either (2^18 x 8, K = 1024, one centroid 100 times
// farther out than the others: 3 % of the points listed).  With e(c) = A ||c|| + psi ||c||^2 / 2 the error of the
// score of centroid c, start values are raised by lift ||c||^2, lift > psi / 2: the score of any c is then at most
//     A ||c|| + (psi / 2 - lift) ||c||^2 <= A^2 / (4 lift - 2 psi)
// too low, whatever its norm, and that of the named centroid at most A ||c|| + (psi / 2 + lift) ||c||^2 too high.
//
// Large calls take a cheaper form where their rows allow it, FORM_HALF: one fp16 piece of either operand and one product, a third of the
// matrix work.  Lost are r_x.c and x.r_c, |r| up to 2^-11 |x|: ||r_c|| / ||c|| is measured by the preparation and ||r_x|| by the settle
// pass, some 0.45 2^-11 each, which makes the bound some 25 times wider than that of two bf16 pieces and leaves 1 to 10 %
// of the points for the third pass - with two candidates as a rule, so that it costs a tenth of the scan.  An operand below
// 2^-14 rounds like that value, in the piece and in the instruction (pinned by a test): norms are raised by 2^-14 for every
// feature.  Data whose points lie far from the origin or in groups would list nearly all, so a sample of the rows chooses
// (scan_choose_kernel).
//
// Both operands are multiplied by one power of two taken from the same rows, so that the scores
// sit in the middle of the fp32 exponent range whatever the scale of the data; what falls outside all
// the same (overflow, NaN) is found by the settle pass, and such a point is compared with every centroid.
#include <cmath>
#include <limits>
#include <type_traits>

#include "ftk_internal.h"
#include "ftk_mma.h"
#include "ftk_quads.h"
#include "ftk_scan.h"
#include "ftk_smalld.h"

namespace ftk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
constexpr int SC_THREADS = 256;  // resident scan: four waves of two point tiles
constexpr int SC_PT = 2;
constexpr int SC_POINTS = 256;   // points per workgroup (both scans)
constexpr int SS_THREADS = 512;  // streaming scan: eight waves
constexpr int FRAG_UNITS = 64;   // 16-byte units per fragment: one per lane
constexpr int SCAN_FILL = 512;     // workgroups that fill the chip (resident scan; the streaming one runs one a unit)
constexpr int SETTLE_ROWS_MAX = 512;  // rows of a workgroup
constexpr int settle_rows(size_t element) { return element == 8 ? 2 : 4; }  // rows a group of lanes settles at once
constexpr int SCAN_LISTS = 64;    // lists of points to resolve, a counter in a line of its own each
constexpr int LIST_STRIDE = 32;
constexpr float HALF_RANGE = 6e4f;  // of a norm: no feature leaves the range of fp16
// The rows that decide between the forms come in shares of 32 that a workgroup compares with a tile of centroids:
// fewer for many centroids, where this adds up (150 000 x 128, K = 2085 5 us with four shares, 33000 x 256, K = 8192
// 28).
static int sample_shares(int tiles) { return tiles <= 64 ? 4 : (tiles <= 128 ? 2 : 1); }
// Of them listed, from which on two pieces are taken: 14, 19, 22 percent.  They are faster from 10 percent
// (524288 x 96, K = 800: 11.5 percent 289 us, refused 272), 13 (400000 x 32, K = 2000: 10.5 percent 182, 15 percent
// 234, refused 212), 16 (130003 x 256, K = 1024: 15 percent 262, refused 297) or more than 20 (2^21 x 32, K = 4096:
// 21 percent 1331, refused 1595) on.
static int sample_limit(int shares) { return shares == 4 ? 18 : (shares == 2 ? 12 : 7); }
constexpr float SCAN_FLOOR = 7.9e-31f;  // 2^-100: below it scores (of centroids near 1) may have lost digits to underflow

// how a block of the contraction is laid out
enum ScanForm : int {
    FORM_PAIR = 0,    // 16 features, two pieces: fragments c0, c1 against x0, x1; c1x0 + c0x1 + c0x0
    FORM_OCTET = 1,   // 8 features, three pieces: fragments (c0 | c1), (c2 | c0) against (x0 | x0), (x1 | x1), (x0 | x2)
    FORM_TRIPLE = 2,  // 16 features, three pieces: c0, c1, c2 against x0, x1, x2; the six largest products
    FORM_HALF = 3     // 16 features, one fp16 piece: one product
};
// centroid and point fragments per block
static constexpr int form_frags(int form) { return form == FORM_HALF ? 1 : (form == FORM_TRIPLE ? 3 : 2); }
static constexpr int form_pieces(int form) { return form == FORM_HALF ? 1 : (form == FORM_PAIR ? 2 : 3); }

// Which of two forms a call takes: see scan_choose_kernel.
struct ScanGate {
    const int32_t *refused;  // not 0: two pieces; NULL: no choice
    __device__ __forceinline__ bool half() const { return refused && *refused == 0; }
    template <int FORM>
    __device__ __forceinline__ bool closed() const
    {
        return refused && (*refused != 0) == (FORM == FORM_HALF);
    }
};

struct ScanArgs {
    const void *X;
    const uint4 *image;
    const float *start;
    const double *scale;
    int64_t N;
    int D;
    int tiles;   // tiles that hold centroids
    int tpc;     // tiles per chunk
    int nch;     // chunks
    int cps;     // chunks per split
    int splits;
    int pblocks;
    ScanRecord *rec;
    ScanGate gate;
};

__device__ __forceinline__ void split_pair(const float (&v)[8], uint4 &hi, uint4 &lo)
{
    bf16x8 p0, p1;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p0[e] = (__bf16)v[e];
        p1[e] = (__bf16)(v[e] - (float)p0[e]);  // the difference is exact
    }
    hi = __builtin_bit_cast(uint4, p0);
    lo = __builtin_bit_cast(uint4, p1);
}

__device__ __forceinline__ void split_triple(const float (&v)[8], uint4 &a, uint4 &b, uint4 &c)
{
    bf16x8 p0, p1, p2;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p0[e] = (__bf16)v[e];
        const float r = v[e] - (float)p0[e];
        p1[e] = (__bf16)r;
        p2[e] = (__bf16)(r - (float)p1[e]);
    }
    a = __builtin_bit_cast(uint4, p0);
    b = __builtin_bit_cast(uint4, p1);
    c = __builtin_bit_cast(uint4, p2);
}

__device__ __forceinline__ uint4 round_half(const float (&v)[8])
{
    halfx8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (_Float16)v[e];
    return __builtin_bit_cast(uint4, h);
}

// squared norm of what an fp16 piece leaves of a value (the difference is exact)
__device__ __forceinline__ void add_lost_half(float v, float &n)
{
    const float r = v - (float)(_Float16)v;
    n = fmaf(r, r, n);
}

// squared norms of what two pieces leave of a value: the second piece, and what neither holds
__device__ __forceinline__ void add_lost(float v, float &n1, float &nr)
{
    const float d = v - (float)(__bf16)v;
    const float p = (float)(__bf16)d, r = d - p;
    n1 = fmaf(p, p, n1);
    nr = fmaf(r, r, nr);
}

__device__ __forceinline__ uint4 select_units(bool c, const uint4 &a, const uint4 &b)
{
    return make_uint4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, c ? a.w : b.w);
}

// Four features from `off`, without branches: whole quads by one access clamped into the row, the
// quad that holds the row's end (RAG: D not a multiple of 4) from `tail`, zero beyond.
template <typename T, bool RAG>
struct RowReader {
    const T *row;
    int D, Dq;  // features, and those in whole quads
    T tail[3];
    __device__ __forceinline__ RowReader(const T *r, int d) : row(r), D(d), Dq(d & ~3)
    {
        if constexpr (RAG) {
#pragma unroll
            for (int e = 0; e < 3; ++e) tail[e] = row[min(Dq + e, D - 1)];
        }
    }
    __device__ __forceinline__ Quad<T> request(int off) const { return load_quad<T>(row + min(off, Dq - 4)); }
    __device__ __forceinline__ Quad<T> keep(Quad<T> q, int off) const
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            T v = off < Dq ? q.v[e] : T(0);
            if constexpr (RAG) {
                if (e < 3) v = (off == Dq && Dq + e < D) ? tail[e < 3 ? e : 0] : v;
            }
            q.v[e] = v;
        }
        return q;
    }
};

// the largest of 64 lanes, but for those that are not numbers
template <typename V>
__device__ __forceinline__ V wave_max(V v)
{
    v = fmax(v, dpp_move<0xB1>(v));
    v = fmax(v, dpp_move<0x4E>(v));
    v = fmax(v, dpp_move<0x141>(v));
    v = fmax(v, dpp_move<0x140>(v));
    v = fmax(v, __shfl_xor(v, 16, 64));
    return fmax(v, __shfl_xor(v, 32, 64));
}

// ---- centroids: pieces in fragment order, start values, norms --------------------------------
// One workgroup per tile of 32 centroids; lane l of a fragment supplies row l % 32 and the 8 features
// 16b + 8(l/32) of block b (FORM_OCTET: all 8 features).  Each of them forms the reference r and the scale for
// itself, from the same rows by the same instructions; r stays in LDS (REF_BYTES; longer rows go without).
constexpr int REF_ROWS = 8;
// second image, of fp16 pieces; nb 0: none
struct HalfImage {
    uint4 *image;
    float *start;
    void *ref;  // the reference goes there
    int32_t *rest_count;
    float4 *sample;  // [tiles][32 shares] best score of a tile, the second, the bound of the best
    const void *X;   // the rows are taken from [N] of these
    int64_t N;
    int tiles;       // workgroups of the images; the others take a tile and a share of the sample each
    int shares;
    int nb;
    float lift, tiny;
};
constexpr size_t REF_BYTES = 64 * 1024;
// HALF: the second image too, and the scores of sampled rows (fp64: more registers than 16 waves have)
constexpr int centroid_waves(size_t element, bool half) { return half && element == 8 ? 8 : 16; }
// RAG: rows that are not whole quads (only HALF asks)
template <typename T, int FORM, bool HALF, bool RAG = true>
__global__ __launch_bounds__(64 * centroid_waves(sizeof(T), HALF)) void scan_centroids_kernel(const T *C, int D, int K, int nb, uint4 *image, float *start,
                                                              float4 *tile_stat, double *scale, int32_t *list_count, int lists,
                                                              int has_ref, float *norm, double lift, HalfImage half_args)
{
    const HalfImage half = HALF ? half_args : HalfImage{};
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int nb_all = max(nb, half.nb);
    T *const ref = reinterpret_cast<T *>(lds_raw);  // [16 nb_all]
    // sampling: [waves][4][64] sums of the rows over a wave's blocks
    floatx4 *const part = reinterpret_cast<floatx4 *>(lds_raw + (has_ref ? (size_t)16 * nb_all * sizeof(T) : 0));
    __shared__ float sh_start[32], sh_norm[32];
    __shared__ double sh_n[16][32], sh_rc[16][32];
    __shared__ float sh_n1[16][32], sh_nr[16][32];  // squared norms of the second pieces and of the residuals
    __shared__ float sh_nh[16][32];                 // and of what fp16 pieces leave
    __shared__ T sh_m[16][2];
    __shared__ double sh_s[16][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = (int)blockDim.x >> 6;
    // (beside the images, as few of the chip's units are busy: one workgroup for both took 42 us at K = 357, 1021 fp64
    // features, so 28; 18 and 15 at K = 720, 512 features)
    const bool sampling = HALF && (int)blockIdx.x >= half.tiles;
    const int extra = (int)blockIdx.x - half.tiles, tile = sampling ? extra / half.shares : (int)blockIdx.x;
    const int row = lane & 31, g = lane >> 5;
    const int j = 32 * tile + row;
    const RowReader<T, RAG> reader(C + (size_t)(j < K ? j : 0) * D, D);
    const int share = extra - tile * half.shares;
    const int64_t picked = sampling ? half.N * (2 * (32 * share + row) + 1) / (64 * half.shares) : 0;
    const RowReader<T, RAG> xr(sampling ? static_cast<const T *>(half.X) + picked * D : C, D);
    T m = T(0), whole = T(0);  // largest magnitude of the rows less the reference, and of the rows
    double gain = 0.0, rr = 0.0;  // half the rows' sum of squares less that of what is left of them, and ||r||^2
    for (int d = tid; d < D; d += blockDim.x) {
        T c[REF_ROWS], sum = T(0);
#pragma unroll
        for (int q = 0; q < REF_ROWS; ++q) c[q] = C[(size_t)((int64_t)K * q / REF_ROWS) * D + d];
        // without the smallest and the largest, so that one far centroid does not move it
        T lo = c[0], hi = c[0];
#pragma unroll
        for (int q = 0; q < REF_ROWS; ++q) {
            sum += c[q] * T(1.0 / REF_ROWS);
            lo = c[q] < lo ? c[q] : lo;
            hi = c[q] > hi ? c[q] : hi;
        }
        T r = ((sum - lo * T(1.0 / REF_ROWS)) - hi * T(1.0 / REF_ROWS)) * T((double)REF_ROWS / (REF_ROWS - 2));
        if (!(fabs(r) < Mma<T>::huge())) r = T(0);
        T md = T(0), wd = T(0);
#pragma unroll
        for (int q = 0; q < REF_ROWS; ++q) {
            const T a = fabs(c[q] - r), w = fabs(c[q]);
            md = a > md ? a : md;
            wd = w > wd ? w : wd;
            gain = fma(0.5 * (double)w, (double)w, gain);
            gain = fma(-(double)a, (double)a, gain);
        }
        // (each feature's largest left out of both)
        gain = fma(-0.5 * (double)wd, (double)wd, gain);
        gain = fma((double)md, (double)md, gain);
        rr = fma((double)r, (double)r, rr);
        m = md > m ? md : m;
        whole = wd > whole ? wd : whole;
        if (has_ref) ref[d] = r;
    }
    if (has_ref)
        for (int d = D + tid; d < 16 * nb_all; d += blockDim.x) ref[d] = T(0);
    m = wave_max(m);
    whole = wave_max(whole);
    gain = group_sum<64>(gain);
    if (HALF || blockIdx.x == 0) rr = group_sum<64>(rr);  // (else the only one to use it)
    if (lane == 0) {
        sh_m[wave][0] = m;
        sh_m[wave][1] = whole;
        sh_s[wave][0] = gain;
        sh_s[wave][1] = rr;
    }
    __syncthreads();
    gain = rr = 0.0;
    for (int i = 0; i < nw; ++i) {
        m = sh_m[i][0] > m ? sh_m[i][0] : m;
        whole = sh_m[i][1] > whole ? sh_m[i][1] : whole;
        gain += sh_s[i][0];
        rr += sh_s[i][1];
    }
    // The reference is taken where it halves the squared norms at least: of data about the origin it is
    // a random vector.  The scale: the largest magnitude goes to [1, 2) - that of the rows themselves where
    // they are all the same.
    const bool moved = has_ref && gain > 0.0;
    if (!moved || !(m > T(0))) m = whole;
    int e2 = 0;
    if (m > T(0) && m < Mma<T>::huge()) e2 = ilogb(m);
    constexpr int E2 = sizeof(T) == 4 ? 100 : 1000;
    e2 = e2 > E2 ? E2 : (e2 < -E2 ? -E2 : e2);
    const T s = (T)ldexp(1.0, -e2);
    if (blockIdx.x == 0 && tid == 0) {
        scale[0] = (double)s;
        scale[1] = moved ? sqrt(rr) * (double)s : 0.0;
    }
    if (blockIdx.x == 0) {
        if (tid < lists) list_count[tid * LIST_STRIDE] = 0;
        if (tid < SCAN_LISTS && half.nb) half.rest_count[tid * LIST_STRIDE] = 0;
        if (half.nb)
            for (int d = tid; d < D; d += blockDim.x) static_cast<T *>(half.ref)[d] = moved ? ref[d] : T(0);
    }
    double n = 0.0, rc = 0.0;
    float n1 = 0.f, nr = 0.f, nh = 0.f;
    float sn = 0.f, src = 0.f;
    floatx16 sum;
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[r] = 0.f;
#pragma unroll 2
    for (int b = wave; b < nb_all; b += nw) {
        const int f0 = FORM == FORM_OCTET ? 0 : 16 * b + 8 * g;
        const Quad<T> q0 = reader.request(f0), q1 = reader.request(f0 + 4);
        Quad<T> x0 = {}, x1 = {};
        if (sampling) {
            x0 = xr.request(f0);
            x1 = xr.request(f0 + 4);
        }
        const Quad<T> k0 = reader.keep(q0, f0), k1 = reader.keep(q1, f0 + 4);
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const T r = moved ? ref[f0 + e] : T(0);
            const T w = j < K ? ((e < 4 ? k0.v[e & 3] : k1.v[e & 3]) - r) * s : T(0);
            v[e] = (float)w;
            if (sampling) {  // (their scores carry the error of fp16 pieces)
                sn = fmaf(v[e], v[e], sn);
                src = fmaf(v[e], (float)(r * s), src);
            } else {
                n = fma((double)w, (double)w, n);
                rc = fma((double)w, (double)r, rc);
            }
        }
        if (sampling) {
            x0 = xr.keep(x0, f0);
            x1 = xr.keep(x1, f0 + 4);
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = (float)((e < 4 ? x0.v[e & 3] : x1.v[e & 3]) * s);
            sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, round_half(v)),
                                                         __builtin_bit_cast(halfx8, round_half(x)), sum, 0, 0, 0);
            continue;
        }
        uint4 *dst = image + ((size_t)tile * nb + b) * (form_frags(FORM) * FRAG_UNITS) + lane;
        if constexpr (FORM != FORM_PAIR) {
            uint4 a0, a1, a2;
            split_triple(v, a0, a1, a2);
            if constexpr (FORM == FORM_OCTET) {
                dst[0] = select_units(g != 0, a1, a0);
                dst[FRAG_UNITS] = select_units(g != 0, a0, a2);
            } else {
                dst[0] = a0;
                dst[FRAG_UNITS] = a1;
                dst[2 * FRAG_UNITS] = a2;
            }
        } else {
            if (b < nb) {
                uint4 a0, a1;
                split_pair(v, a0, a1);
                dst[0] = a0;
                dst[FRAG_UNITS] = a1;
#pragma unroll
                for (int e = 0; e < 8; ++e) add_lost(v[e], n1, nr);
            }
            if (b < half.nb) {
                half.image[((size_t)tile * half.nb + b) * FRAG_UNITS + lane] = round_half(v);
#pragma unroll
                for (int e = 0; e < 8; ++e) add_lost_half(v[e], nh);
            }
        }
    }
    if (sampling) {
        n = (double)sn;
        rc = (double)src / (double)s;
    }
    if (FORM != FORM_OCTET) {
        n += __shfl_xor(n, 32, 64);
        rc += __shfl_xor(rc, 32, 64);
    }
    if (FORM == FORM_PAIR) {
        n1 += __shfl_xor(n1, 32, 64);
        nr += __shfl_xor(nr, 32, 64);
        nh += __shfl_xor(nh, 32, 64);
    }
    if (lane < 32) {
        sh_n[wave][lane] = n;
        sh_rc[wave][lane] = rc;
        sh_n1[wave][lane] = n1;
        sh_nr[wave][lane] = nr;
        sh_nh[wave][lane] = nh;
    }
    if (sampling) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            part[(wave * 4 + i) * 64 + lane] = floatx4{sum[4 * i], sum[4 * i + 1], sum[4 * i + 2], sum[4 * i + 3]};
    }
    __syncthreads();
    if (tid < 32) {
        n = rc = 0.0;
        n1 = nr = nh = 0.f;
        for (int i = 0; i < nw; ++i) {
            n += sh_n[i][tid];
            rc += sh_rc[i][tid];
            n1 += sh_n1[i][tid];
            nr += sh_nr[i][tid];
            nh += sh_nh[i][tid];
        }
        // register r of lane group gg reads row 8(r/4) + 4gg + r%4
        const int gg = (tid >> 2) & 1, r = 4 * (tid >> 3) + (tid & 3);
        const float half_start =
            32 * tile + tid < K ? (float)(((double)half.lift - 0.5) * n - rc * (double)s) : -__builtin_huge_valf();
        sh_start[tid] = half_start;
        sh_norm[tid] = sqrtf((float)n);
        if (!sampling) {
            start[tile * 32 + gg * 16 + r] =
                32 * tile + tid < K ? (float)((lift - 0.5) * n - rc * (double)s) : -__builtin_huge_valf();
            if (half.nb) half.start[tile * 32 + gg * 16 + r] = half_start;
            norm[tile * 32 + tid] = sqrtf((float)n);
        }
        // (a NaN row never wins and does not count)
        float f = n > 0.0 ? (float)n : 0.f;
        float q1 = n > 0.0 ? (float)((double)n1 / n) : 0.f, qr = n > 0.0 ? (float)((double)nr / n) : 0.f;
        const float full = sqrtf(f) + half.tiny;
        float qh = half.nb && full > 0.f ? nh / (full * full) : 0.f;
#pragma unroll
        for (int k = 16; k >= 1; k >>= 1) {
            f = fmaxf(f, __shfl_xor(f, k, 64));
            q1 = fmaxf(q1, __shfl_xor(q1, k, 64));
            qr = fmaxf(qr, __shfl_xor(qr, k, 64));
            qh = fmaxf(qh, __shfl_xor(qh, k, 64));
        }
        if (tid == 0 && !sampling) tile_stat[tile] = make_float4(f, q1, qr, qh);
    }
    if (sampling) {
        __syncthreads();
        if (wave > 0) return;
        float m1 = Mma<float>::neg_inf(), m2 = m1;
        int j1 = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            floatx4 v = part[i * 64 + lane];
            for (int w = 1; w < nw; ++w) v += part[(w * 4 + i) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int jj = 8 * i + 4 * g + e;
                const float score = v[e] + sh_start[jj];
                const bool better = score > m1;
                m2 = better ? m1 : (score > m2 ? score : m2);
                m1 = better ? score : m1;
                j1 = better ? jj : j1;
            }
        }
        const float o1 = __shfl_xor(m1, 32, 64), o2 = __shfl_xor(m2, 32, 64);
        const int oj = __shfl_xor(j1, 32, 64);
        const bool mine = m1 >= o1;
        // about the bound of the settle pass, with the named centroid's norm in place of the point's
        const float c = sh_norm[mine ? j1 : oj], r = moved ? (float)(sqrt(rr) * (double)s) : 0.f;
        if (lane < 32)
            half.sample[(size_t)extra * 32 + lane] =
                make_float4(mine ? m1 : o1, fmaxf(fmaxf(m2, o2), mine ? o1 : m1), 0.9f * 0x1p-11f * (c + r) * c, 0.f);
    }
}

// ---- choice of form ---------------------------------------------------------------------------
// One fp16 piece leaves nearly all points of some data to the third pass (data far from the origin or in groups, against
// their spread; a centroid beyond the range of fp16): two pieces scan these.  Rows spread evenly over the whole problem
// tell, whatever their order, before either scan runs; the choice holds for all launches of the problem.
// The sample costs one launch, 4 us, beside what it adds to the preparation (2^21 x 32, K = 4096 2 us; 1021 fp64 features, K = 357
// 11 us).  (A vote of the scan's first workgroups costs none, but all of that scan where all run at
// once: two groups at +-20, spread 1, in 200000 x 32, K = 2400 206 us against 144 by two pieces alone, 150001 x 128 fp64,
// K = 2085 475 / 317; a scan of 32 000 rows ahead 24 to 62 us.)
__global__ __launch_bounds__(1024) void scan_choose_kernel(const float4 *sample, const float4 *tile_stat, int tiles, int rows, int limit,
                                                           int32_t *refused)
{
    __shared__ float sh_m1[1024], sh_m2[1024], sh_bound[1024];
    const int tid = threadIdx.x, i = tid & (rows - 1);  // rows: a power of two
    float m1 = Mma<float>::neg_inf(), m2 = m1, bound = 0.f;
    auto add = [&](float o1, float o2, float ob) {
        const bool mine = m1 >= o1;
        m2 = fmaxf(fmaxf(m2, o2), mine ? o1 : m1);
        m1 = mine ? m1 : o1;
        bound = mine ? bound : ob;
    };
#pragma unroll 4
    for (int64_t k = tid; k < (int64_t)tiles * rows; k += 1024) {
        const float4 v = sample[k];
        add(v.x, v.y, v.z);
    }
    bool far = false;
    for (int t = tid; t < tiles; t += 1024) far = far || !(tile_stat[t].x < 0.99f * HALF_RANGE * HALF_RANGE);
    sh_m1[tid] = m1;
    sh_m2[tid] = m2;
    sh_bound[tid] = bound;
    far = __syncthreads_or(far);
    if (tid < rows)
        for (int k = i + rows; k < 1024; k += rows) add(sh_m1[k], sh_m2[k], sh_bound[k]);
    const int listed = __syncthreads_count(tid < rows && !(m1 - m2 > bound));
    if (tid == 0) *refused = far || listed >= limit;
}

// ---- bookkeeping of the scans -----------------------------------------------------------------
// Tile maximum, runner-up tile maximum and the 16 scores of the best tile of one lane: two scores
// share a v_max3; the copy of the scores is skipped unless some lane of the wave found a better tile, and runs as moves
// under the lane mask: a v_mov_b64 takes the issue time of one v_cndmask_b32 and moves two scores (2^20 x 8, K = 1024
// 152 us a call with selects, 140 with moves; 2^21 x 32, K = 4096 850 / 785; 300007 x 45, K = 333 69.7 / 67.7).
struct ScanBest {
    float m1, m2;
    int t1;
    floatx16 s;
};

__device__ __forceinline__ void scan_best_init(ScanBest &b)
{
    b.m1 = b.m2 = Mma<float>::neg_inf();
    b.t1 = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) b.s[r] = Mma<float>::neg_inf();
}

__device__ __forceinline__ void scan_best_add(ScanBest &b, const floatx16 &acc, int T)
{
    float tm = max2f(acc[0], acc[1]);
#pragma unroll
    for (int r = 2; r < 16; r += 2) tm = max3f(tm, acc[r], acc[r + 1]);
    const bool c = tm > b.m1;
    b.m2 = __builtin_amdgcn_fmed3f(b.m1, b.m2, tm);
    b.m1 = max2f(b.m1, tm);
    if (c) {
        asm volatile("");  // (keeps the branch: the compiler would turn it into selects)
        b.t1 = T;
#pragma unroll
        for (int r = 0; r < 16; ++r) b.s[r] = acc[r];
    }
}

// best score, its centroid and the second best of a point (both lanes of the pair get them)
__device__ __forceinline__ void scan_best_finish(const ScanBest &b, int g, float &m1, int &j1, float &m2)
{
    int r1 = 0;
#pragma unroll
    for (int r = 15; r >= 0; --r) r1 = b.s[r] == b.m1 ? r : r1;
    float sec = b.m2;
#pragma unroll
    for (int r = 0; r < 16; ++r) sec = (r != r1 && b.s[r] > sec) ? b.s[r] : sec;
    const int j = 32 * b.t1 + 8 * (r1 >> 2) + 4 * g + (r1 & 3);
    const float om1 = __shfl_xor(b.m1, 32, 64), osec = __shfl_xor(sec, 32, 64);
    const int oj = __shfl_xor(j, 32, 64);
    const bool mine = b.m1 > om1 || (b.m1 == om1 && j < oj);
    m1 = mine ? b.m1 : om1;
    j1 = mine ? j : oj;
    m2 = mine ? (sec > om1 ? sec : om1) : (osec > b.m1 ? osec : b.m1);
    if (!(b.m1 == b.m1) || !(om1 == om1)) m2 = __builtin_huge_valf();  // NaN scores: not to be trusted
}

// ---- settle -----------------------------------------------------------------------------------
// L lanes share a row (row-contiguous 16-byte loads) and take ROWS of them at once: the pass is a
// chain of latencies - record, then the centroid's row - that only requests in flight can hide.
// A workgroup hands its listed points over with one atomic, to one of 64 lists: atomics on one word
// follow one another at about 10 ns (2^21 x 32, K = 4096: 9 000 workgroups with something to list).
struct SettleArgs {
    ScanRecord *rec;
    int splits;
    const float4 *tile_stat;
    int tiles;
    const double *scale;
    int64_t N;
    int D, K;
    float psi, lost;    // rounding of a score; what is lost of ||x|| ||c|| whatever the centroids
    float lift;         // by which multiple of ||c||^2 the scores were raised
    const float *norm;  // ||c||
    float sums;         // rounding of a sum of squares over a row, halved
    float slack, tiny;  // of the measured norms: their own rounding, and what underflow takes from them
    int32_t *labels;
    ScanListed *list;  // (point, score a candidate needs), or NULL: the points alone go to wl
    int32_t *wl, *list_count;
    int lists, list_cap;
    int32_t *tickets;   // [N/32 + 1] cleared here for the pass that follows
    // scans on fp16 pieces: their numbers where the gate chooses them
    ScanGate gate;
    int half_splits;
    float half_psi, half_lift, half_tiny;
    const void *ref;    // [D] the reference r
};

enum SettleKind : int {
    SETTLE_PLAIN = 0,   // distances in the data's type
    SETTLE_DOUBLE = 1,  // in double, added up in the order of group_sqdist(): whatever passes a point goes through, and so
                        // whichever form scanned it (batches of a step take the one that is faster for their size),
                        // its distance has the same bits; fp32 2^21 x 32, K = 4096 859 / 860 us a call, 60000 x 1024
                        // 343 / 344
    SETTLE_HALF = 2     // the same, and the records may come from fp16 pieces
};
// lanes of a row
constexpr int settle_lanes(int D) { return D <= 12 ? 2 : (D <= 24 ? 4 : (D <= 128 ? 8 : (D <= 512 ? 16 : 64))); }

// of a row: squared norms of x, of x - r and of what an fp16 piece leaves of x; its record and ||c||
struct SettleSums {
    float x2, y2, xr2, m1, m2, cn;
    int32_t j;
};
template <typename T, int L, int ROWS>
struct SettleShared {
    static constexpr int N = 256 / L * ROWS;  // rows of a block
    float max[4][4];
    int n, base;
    SettleSums sums[N];
    T dist[N];
};

// Block `block` of N rows.  own: their records where the workgroup that scanned the points settles them itself, else
// NULL; half: the records come from fp16 pieces; again: a block after another one.
template <typename T, int L, int ROWS, int KIND>
__device__ __forceinline__ void settle_block(const T *X, const T *C, T *mindist, const SettleArgs &a, const int64_t block,
                                             const ScanRecord *own, const bool half, const bool again,
                                             SettleShared<T, L, ROWS> &sh)
{
    constexpr bool HALF = KIND == SETTLE_HALF;
    using Acc = std::conditional_t<KIND == SETTLE_PLAIN, T, double>;
    const int splits = own ? 1 : (half ? a.half_splits : a.splits);
    const float psi = half ? a.half_psi : a.psi, lift = half ? a.half_lift : a.lift, tiny = half ? a.half_tiny : a.tiny;
    constexpr int RPB = 256 / L;  // rows side by side
    constexpr int Q = HALF ? 4 : 3;
    const int tid = threadIdx.x, lane = tid & 63;
    const int sub = tid & (L - 1), grp = tid / L;
    const int Dq = a.D & ~3;
    const int64_t first = block * (ROWS * RPB);
    int at[ROWS];  // of the rows, from the first one
    float m1[ROWS], m2[ROWS];
    int j[ROWS];
    const T *c[ROWS];
    const T *const X0 = X + first * a.D;
    const ScanRecord *rec = own ? own : a.rec + first;
    Quad<T> xv[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        at[u] = (int)min((int64_t)(u * RPB + grp), a.N - 1 - first);
        const ScanRecord r = rec[at[u]];
        m1[u] = r.m1;
        m2[u] = r.m2;
        j[u] = r.j1;
    }
    // the first piece of every row travels with the records
#pragma unroll
    for (int u = 0; u < ROWS; ++u) xv[u] = load_quad<T>(X0 + (unsigned)(at[u] * a.D + min(4 * sub, Dq - 4)));
    if (tid == 0) sh.n = 0;
    const int64_t i0 = block * 256 + tid;
    if (i0 * 32 < a.N) a.tickets[i0] = 0;
    float cm[Q] = {};
    for (int i = again ? a.tiles : tid; i < a.tiles; i += 256) {
        const float4 t = a.tile_stat[i];
        cm[0] = fmaxf(cm[0], t.x);
        cm[1] = fmaxf(cm[1], t.y);
        cm[2] = fmaxf(cm[2], t.z);
        if constexpr (HALF) cm[3] = fmaxf(cm[3], t.w);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        cm[q] = wave_max(cm[q]);
        if (lane == 0 && !again) sh.max[tid >> 6][q] = cm[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) cm[q] = fmaxf(fmaxf(sh.max[0][q], sh.max[1][q]), fmaxf(sh.max[2][q], sh.max[3][q]));
    const float cmax = 1.000001f * sqrtf(cm[0]) + tiny;
    // a score of centroid c is off by at most A ||c|| + psi ||c||^2 / 2, A = lost ||x|| + psi (||x|| + ||r||); ||x1||
    // <= 2^-8 ||x|| (fp16 pieces: lost ||x|| is ||r_x|| + max(||r_c|| / ||c||) ||x||, the first measured below)
    const float lost = half ? 1.001f * a.slack * sqrtf(cm[Q - 1])
                            : a.lost + 1.001f * a.slack * (0x1p-8f * sqrtf(cm[1]) + sqrtf(cm[2]));
    const T s = (T)a.scale[0];
    const float ref = 1.000001f * (float)a.scale[1] + tiny;  // ||r||
    const float under = (float)((T)(a.D + 16) * std::numeric_limits<T>::min() * s * s);
    for (int k = 1; k < splits; ++k) {
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const ScanRecord o = rec[(int64_t)k * a.N + at[u]];
            const bool mine = m1[u] >= o.m1;
            m2[u] = fmaxf(fmaxf(m2[u], o.m2), mine ? o.m1 : m1[u]);
            m1[u] = mine ? m1[u] : o.m1;
            j[u] = mine ? j[u] : o.j1;
        }
    }
    Acc d[ROWS];
    float xn[ROWS], yn[ROWS], cn[ROWS], xr[ROWS];  // of x and of x - r, of c, of what an fp16 piece leaves of x
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        j[u] = (unsigned)j[u] < (unsigned)a.K ? j[u] : 0;  // padding rows, when no score was a number
        c[u] = C + (size_t)j[u] * a.D;
        cn[u] = a.norm[j[u]];
        if (sub == 0) {
            SettleSums &q = sh.sums[u * RPB + grp];
            q.m1 = m1[u];
            q.m2 = m2[u];
            q.j = j[u];
        }
        d[u] = Acc(0);
        xn[u] = yn[u] = xr[u] = 0.f;
    }
    const T *const ref_row = (const T *)a.ref;
    auto add = [&](int u, T xe, T ce, T re) {
        const Acc t = (Acc)xe - (Acc)ce;
        d[u] = fma(t, t, d[u]);
        const float w = (float)(xe * s);
        xn[u] = fmaf(w, w, xn[u]);
        if constexpr (HALF) {
            const float y = (float)((xe - re) * s);
            yn[u] = fmaf(y, y, yn[u]);
            add_lost_half(w, xr[u]);
        }
    };
    for (int f = 4 * sub; f < Dq;) {
        Quad<T> cv[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) cv[u] = load_quad<T>(c[u] + f);
        Quad<T> rv = {};
        if constexpr (HALF) rv = load_quad<T>(ref_row + f);
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) add(u, xv[u].v[e], cv[u].v[e], rv.v[e]);
        f += 4 * L;
        if (f < Dq)
#pragma unroll
            for (int u = 0; u < ROWS; ++u) xv[u] = load_quad<T>(X0 + (unsigned)(at[u] * a.D + f));
    }
    for (int f = Dq + sub; f < a.D; f += L)
#pragma unroll
        for (int u = 0; u < ROWS; ++u) add(u, X0[(unsigned)(at[u] * a.D + f)], c[u][f], HALF ? ref_row[f] : T(0));
    // a row's bound is some hundred instructions: a thread takes one instead of its L lanes the same one
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const T dist = (T)group_sum<L>(d[u]);
        const float x2 = group_sum<L>(xn[u]);
        float y2 = 0.f, xr2 = 0.f;
        if constexpr (HALF) {
            y2 = group_sum<L>(yn[u]);
            if (half) xr2 = group_sum<L>(xr[u]);
        }
        if (sub == 0) {
            SettleSums &q = sh.sums[u * RPB + grp];
            q.x2 = x2;
            q.y2 = y2;
            q.xr2 = xr2;
            q.cn = cn[u];
            sh.dist[u * RPB + grp] = dist;
        }
    }
    __syncthreads();
    // whether score bounds say who is nearest; the score a candidate needs
    auto bound = [&](const SettleSums &q, T dist, float &thr) {
        const float norm = a.slack * sqrtf(q.x2) + tiny;
        float A = lost * norm + psi * (norm + ref);
        const float B = lift - 0.5f * psi;
        if constexpr (HALF) A += half ? 1.001f * a.slack * sqrtf(q.xr2) : 0.f;
        const float c1 = 1.000001f * q.cn + tiny, t = fminf(A / (2.f * B), cmax);  // the norm most too low
        // How much too low the score of any centroid is, at most, and how much too high that of the named one.
        const float low = 1.00001f * ((A - B * t) * t + (A + psi * cmax) * tiny) + SCAN_FLOOR;
        const float high = 1.00001f * (A + (lift + 0.5f * psi) * c1) * c1;
        float least = q.m1 - high;
        if constexpr (HALF) {
            // Its true score is also known from the distance, (||x - r||^2 - ||x - c||^2) / 2, to within the rounding
            // of these sums: of fp16 pieces that halves the bound (2^21 x 32, K = 4096: 68 000 points listed against
            // 105 000). The distance comes from differences that carry no scale: `under` is what underflow may have
            // taken from it, infinite (a distance out of range: d2) where these sums say nothing.
            const float d2 = (float)(dist * s * s);
            least = fmaxf(least, 0.5f * (q.y2 - d2) - a.sums * (q.y2 + d2) - under);
        }
        least -= low;
        // No score means anything where one may have left the fp32 range (||c||^2 or a product infinite, also on
        // the way to a sum that is not): a threshold that is not a number makes every centroid a candidate.
        const bool sound = (norm + ref + cmax) * cmax < 1e38f && (!half || fmaxf(norm, cmax) < HALF_RANGE);
        thr = sound ? least : __builtin_nanf("");
        return sound && least > q.m2;
    };
    // results and the list leave in whole lines
    int mine[(RPB * ROWS + 255) / 256];
    float thr[(RPB * ROWS + 255) / 256];
#pragma unroll
    for (int k = 0; k < (RPB * ROWS + 255) / 256; ++k) {
        const int i = k * 256 + tid;
        const int64_t p = first + i;
        mine[k] = -1;
        if (i < RPB * ROWS && p < a.N) {
            const SettleSums q = sh.sums[i];
            const T dist = sh.dist[i];
            a.labels[p] = q.j;
            if (mindist) mindist[p] = dist;
            if (!bound(q, dist, thr[k])) mine[k] = atomicAdd(&sh.n, 1);
        }
    }
    __syncthreads();
    if (sh.n == 0) return;
    const int which = (int)(block % a.lists);
    if (tid == 0) sh.base = atomicAdd(a.list_count + which * LIST_STRIDE, sh.n);
    __syncthreads();
    const int64_t slot0 = (int64_t)which * a.list_cap + sh.base;
#pragma unroll
    for (int k = 0; k < (RPB * ROWS + 255) / 256; ++k) {
        if (mine[k] < 0) continue;
        const int i = k * 256 + tid;
        if (a.list)
            a.list[slot0 + mine[k]] = ScanListed{(int32_t)(first + i), thr[k]};
        else
            a.wl[slot0 + mine[k]] = (int32_t)(first + i);
    }
}

template <typename T, int L, int KIND>
__global__ __launch_bounds__(256, 4) void scan_settle_kernel(const T *X, const T *C, T *mindist, SettleArgs a)
{
    __shared__ SettleShared<T, L, settle_rows(sizeof(T))> sh;
    settle_block<T, L, settle_rows(sizeof(T)), KIND>(X, C, mindist, a, blockIdx.x, nullptr,
                                                     KIND == SETTLE_HALF && a.gate.half(), false, sh);
}

// The points of a scan's workgroup, settled by it where no other one shares them: their records stay in LDS, and its
// requests travel while other workgroups multiply; a pass of its own waits for them with nothing else to do, after a
// launch and a read of what the scan has just written.  Passes apart / as one, whole calls, us:
//   2 lanes a row  2^20 x 8, K = 1024 136.9 / 130.1; 10^6 x 12, K = 700 150 / 140; fp64 2^20 x 6, K = 300 80 / 72
//   4              1.5 * 10^6 x 16, K = 300 116 / 106; 700000 x 24, K = 1000 120 / 109; fp64 500000 x 20, K = 1000 121 / 115
//   8              2^21 x 32, K = 4096 762 / 733; 971508 x 27, K = 781 153 / 153.  Two pieces alone, where half_pays() is not
//                  met (fewer workgroups a unit, fewer centroids): 1864205 x 29, K = 89 133 / 162; 749932 x 29, K = 417 106 / 112
//   33 features or more: 10^6 x 40, K = 700 178 / 186; 10^6 x 33, K = 50 87 / 91; 300000 x 96, K = 2000 206 / 209
struct SettleOwn {
    const void *C;   // NULL: scan_settle_kernel follows
    void *mindist;
    SettleArgs s;
};
constexpr int OWN_D = 32;  // features of a row, at most
// Rows a group of lanes settles at once, within the registers of the scan: eight lanes, four rows of fp32 spill 128
// bytes of the fp16 form (2^21 x 32, K = 4096 758 us against 750), four lanes do better with them (700000 x 24,
// K = 1000 112, 118).
constexpr int own_rows(size_t element, int lanes) { return element == 4 && lanes == 4 ? 4 : 2; }
template <typename T, int L>
struct OwnShared {
    ScanRecord rec[SC_POINTS];
    SettleShared<T, L, own_rows(sizeof(T), L)> sh;
};
template <typename T, int L, int KIND>
__device__ __forceinline__ void settle_own(const void *X, const SettleOwn &o, int pb, const bool half, OwnShared<T, L> &sh)
{
    constexpr int ROWS = own_rows(sizeof(T), L), N = 256 / L * ROWS, BLOCKS = SC_POINTS / N;
    for (int i = 0; i < BLOCKS; ++i) {
        const int64_t block = (int64_t)pb * BLOCKS + i;
        if (block * N >= o.s.N) break;
        if (i) __syncthreads();
        settle_block<T, L, ROWS, KIND>((const T *)X, (const T *)o.C, (T *)o.mindist, o.s, block, sh.rec + i * N, half, i > 0, sh.sh);
    }
}

// ---- scan of rows of up to 128 features ---------------------------------------------------------
// A wave keeps the pieces of its 2 x 32 points in registers for the whole sweep; the centroid image
// passes through LDS in chunks of 16 or 32 KB, the next chunk copied (global memory to LDS, no
// registers) while the current one is multiplied.  Fragments are stored lane by lane, so the copy is
// linear and the reads are free of bank conflicts.  Rows of up to 32 features are settled here too (SettleOwn); longer
// ones are not: at 128 features 228 registers, two workgroups of four waves per compute unit that wait at their own
// barriers.
// waves of a SIMD whose registers suffice
constexpr int resident_waves(int nb, int form, bool wide, bool ragged)
{
    if (form != FORM_HALF) return nb <= 4 ? 3 : 2;
    return wide ? (nb <= 2 ? 4 : (nb <= 4 ? 3 : 2)) : (nb <= 3 ? 4 : (nb <= 6 || !ragged ? 3 : 2));
}
// GATED: part of a call that chooses its form (the check alone, ahead of all other requests, is 1 us of 38 at 300007 x 45).
template <typename T, int NB, int FORM, bool RAG, bool GATED>
__global__ __launch_bounds__(SC_THREADS, resident_waves(NB, FORM, sizeof(T) == 8, RAG)) void scan_resident_kernel(ScanArgs a, SettleOwn own)
{
    if (GATED && a.gate.closed<FORM>()) return;
    constexpr int FR = form_frags(FORM);
    constexpr int TU = NB * FR * FRAG_UNITS;  // units per tile
    extern __shared__ __align__(16) uint4 lds4[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5;
    const int pb = (int)blockIdx.x / a.splits, split = (int)blockIdx.x % a.splits;
    const int ch0 = split * a.cps, ch1 = min(ch0 + a.cps, a.nch);
    const int cu = a.tpc * TU + ((a.tpc + 1) / 2) * 16;  // units of a chunk buffer: fragments, then start values
    const int64_t p0 = (int64_t)pb * SC_POINTS + wave * (SC_PT * 32);

    auto stage = [&](int ch, uint4 *buf) {
        const int tile0 = ch * a.tpc;
        const uint4 *src = a.image + (size_t)tile0 * TU;
        const int n = a.tpc * TU / FRAG_UNITS;
        for (int i = wave; i < n; i += SC_THREADS / 64) to_lds16(src + i * FRAG_UNITS + lane, buf + i * FRAG_UNITS);
        // start values, two tiles a time (the array is padded by one tile)
        const float *sv = a.start + tile0 * 32;
        float *dst = reinterpret_cast<float *>(buf + a.tpc * TU);
        for (int i = wave; 2 * i < a.tpc; i += SC_THREADS / 64) to_lds4(sv + i * 64 + lane, dst + i * 64);
    };
    stage(ch0, lds4);

    const T s = (T)a.scale[0];
    const T *X = reinterpret_cast<const T *>(a.X);
    constexpr int NP = form_pieces(FORM);
    uint4 b[SC_PT][NB][NP];
#pragma unroll
    for (int pt = 0; pt < SC_PT; ++pt) {
        int64_t p = p0 + pt * 32 + col;
        if (p >= a.N) p = a.N - 1;
        const RowReader<T, RAG> row(X + p * a.D, a.D);
        // all of a row's loads in flight together, unless that takes more registers than there are
        constexpr int BATCH = sizeof(T) == 8 && NB > 4 ? NB / 2 : NB;
        auto off = [&](int u) { return FORM == FORM_OCTET ? 4 * u : 16 * (u >> 1) + 8 * g + 4 * (u & 1); };
        Quad<T> q[2 * BATCH];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (k % BATCH == 0) {
                if (k) asm volatile("" ::: "memory");
#pragma unroll
                for (int u = 0; u < 2 * BATCH; ++u) q[u] = row.request(off(2 * k + u));
            }
            float v[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const Quad<T> w = row.keep(q[2 * (k % BATCH) + h], off(2 * k + h));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * h + e] = (float)(w.v[e] * s);
            }
            if constexpr (FORM == FORM_HALF) {
                b[pt][k][0] = round_half(v);
            } else if constexpr (FORM != FORM_PAIR) {
                uint4 x0, x1, x2;
                split_triple(v, x0, x1, x2);
                b[pt][k][0] = x0;
                b[pt][k][1] = x1;
                b[pt][k][2] = FORM == FORM_TRIPLE ? x2 : select_units(g != 0, x2, x0);
            } else {
                split_pair(v, b[pt][k][0], b[pt][k][1]);
            }
        }
    }
    ScanBest best[SC_PT];
#pragma unroll
    for (int pt = 0; pt < SC_PT; ++pt) scan_best_init(best[pt]);
    wait_loads<0>();
    __syncthreads();

    int cur = 0;
    for (int ch = ch0; ch < ch1; ++ch) {
        uint4 *buf = lds4 + cur * cu;
        if (ch + 1 < ch1) stage(ch + 1, lds4 + (cur ^ 1) * cu);
        const int nt = min(a.tpc, a.tiles - ch * a.tpc);
        const float *hv = reinterpret_cast<const float *>(buf + a.tpc * TU) + g * 16;
        for (int t = 0; t < nt; ++t) {
            const uint4 *f = buf + t * TU + lane;
            floatx16 acc[SC_PT];
            {
                floatx16 ci;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const floatx4 h = *reinterpret_cast<const floatx4 *>(hv + t * 32 + 4 * i);
#pragma unroll
                    for (int e = 0; e < 4; ++e) ci[4 * i + e] = h[e];
                }
#pragma unroll
                for (int pt = 0; pt < SC_PT; ++pt) acc[pt] = ci;
            }
            // the fragments of block k + 1 are requested before the instructions of block k are issued
            uint4 n[FR];
#pragma unroll
            for (int i = 0; i < FR; ++i) n[i] = f[i * FRAG_UNITS];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                bf16x8 af[FR];
#pragma unroll
                for (int i = 0; i < FR; ++i) af[i] = __builtin_bit_cast(bf16x8, n[i]);
                if (k + 1 < NB) {
#pragma unroll
                    for (int i = 0; i < FR; ++i) n[i] = f[((k + 1) * FR + i) * FRAG_UNITS];
                }
                if constexpr (FORM == FORM_HALF) {
#pragma unroll
                    for (int pt = 0; pt < SC_PT; ++pt)
                        acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                            __builtin_bit_cast(halfx8, af[0]), __builtin_bit_cast(halfx8, b[pt][k][0]), acc[pt], 0, 0, 0);
                    continue;
                }
                // (centroid, point) fragments of the products, smallest first; the chains of the two
                // point tiles interleave
                constexpr int NM = FORM == FORM_TRIPLE ? 6 : 3;
                constexpr int PROD[6][2] = {{FORM == FORM_TRIPLE ? 2 : 1, FORM == FORM_OCTET ? 2 : 0},
                                            {FORM == FORM_TRIPLE ? 1 : 0, 1}, {0, FORM == FORM_TRIPLE ? 2 : 0},
                                            {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
                for (int i = 0; i < NM; ++i)
#pragma unroll
                    for (int pt = 0; pt < SC_PT; ++pt)
                        acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            af[PROD[i][0] % FR], __builtin_bit_cast(bf16x8, b[pt][k][PROD[i][1] % NP]), acc[pt], 0, 0, 0);
            }
            // keep that order through instruction scheduling, which would sink every read to its use
            // (at four blocks the second pair of fragments does not fit the registers of three waves)
            if constexpr (NB != 4 && FORM != FORM_TRIPLE && FORM != FORM_HALF) {
                __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
                for (int k = 0; k + 1 < NB; ++k) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 3 * SC_PT, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 3 * SC_PT, 0);
            }
#pragma unroll
            for (int pt = 0; pt < SC_PT; ++pt) scan_best_add(best[pt], acc[pt], ch * a.tpc + t);
        }
        wait_loads<0>();  // the next chunk has arrived
        __syncthreads();
        cur ^= 1;
    }
#pragma unroll
    for (int pt = 0; pt < SC_PT; ++pt) {
        float m1, m2;
        int j1;
        scan_best_finish(best[pt], g, m1, j1, m2);
        const int64_t p = p0 + pt * 32 + col;
        if (NB <= 2 && own.C) {
            // the chunks are done with: every wave has passed the barrier behind the last one
            ScanRecord *const rec = reinterpret_cast<ScanRecord *>(lds4) + (wave * SC_PT + pt) * 32 + col;
            if (g == 0) *rec = ScanRecord{m1, m2, j1, 0};
        } else if (g == 0 && p < a.N) {
            a.rec[(int64_t)split * a.N + p] = ScanRecord{m1, m2, j1, 0};
        }
    }
    if constexpr (NB <= 2) {
        if (!own.C) return;
        __syncthreads();
        constexpr int KIND = GATED ? SETTLE_HALF : SETTLE_PLAIN;
        auto settle = [&](auto lanes) {
            constexpr int L = decltype(lanes)::value;
            settle_own<T, L, KIND>(a.X, own, pb, FORM == FORM_HALF, *reinterpret_cast<OwnShared<T, L> *>(lds4));
        };
        // an octet's rows go to two lanes, a triple's to two or four, those of two blocks to four or, of calls that
        // choose their form, eight: settles_own()
        if constexpr (FORM == FORM_OCTET) {
            settle(std::integral_constant<int, 2>{});
        } else if constexpr (FORM == FORM_TRIPLE) {
            if (settle_lanes(a.D) == 2) settle(std::integral_constant<int, 2>{});
            else settle(std::integral_constant<int, 4>{});
        } else {
            if (!GATED || settle_lanes(a.D) == 4) settle(std::integral_constant<int, 4>{});
            else settle(std::integral_constant<int, 8>{});
        }
    }
}

// ---- scan of longer rows --------------------------------------------------------------------------
// A workgroup multiplies 256 points by 64 * CT centroids, 32 features at a time through LDS (double buffered, up to
// 128 KB): the centroid fragments are copied from the image, the rows of X are split on the way - requested two
// stages ahead, split and stored one stage ahead.  Wave w takes point tiles 2(w%4) .. +1 and the centroid tiles of
// half w/4.  The workgroups that share a block of points run side by side on one XCD, so that X comes from memory
// once whatever K.
template <typename T, int CT, bool RAG, bool GATED>
__global__ __launch_bounds__(SS_THREADS, 2) void scan_stream_kernel(ScanArgs a)
{
    if (GATED && a.gate.closed<FORM_PAIR>()) return;
    constexpr int TPC = 2 * CT;  // centroid tiles per workgroup
    constexpr int AU = TPC * 4 * FRAG_UNITS, BU = 8 * 4 * FRAG_UNITS;  // units per stage: centroids, points
    extern __shared__ __align__(16) uint4 lds4[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5;
    // consecutive workgroups go to consecutive XCDs: those of one XCD that follow each other share points
    const int xcd = (int)blockIdx.x & 7, slot = (int)blockIdx.x >> 3;
    const int ch = slot % a.nch;
    const int pb = (slot / a.nch) * 8 + xcd;
    if (pb >= a.pblocks) return;
    const int D = a.D;
    const int ns = (D + 31) >> 5;
    const int nb = 2 * ns;  // blocks per tile of the image
    const int wp = wave & 3, wc = wave >> 2;

    // The features this thread brings in: four of each of four rows; eight lanes take a row's 32, whole lines of
    // memory.  (16 features of one row a lane, 64 places a request, whole calls: 500000 x 130, K = 64 149 us against
    // 130, 131072 x 512, K = 100 139 / 131, 100000 x 301, K = 300 153 / 144, 9000 x 640, K = 1000 116 / 107; fp64
    // 40000 x 900, K = 310 339 / 257.)
    const int q8 = lane & 7, r8 = lane >> 3;
    const T *X = reinterpret_cast<const T *>(a.X);
    auto reader = [&](int i) {
        return RowReader<T, RAG>(X + min((int64_t)pb * SC_POINTS + wave * 32 + 8 * i + r8, a.N - 1) * D, D);
    };
    const RowReader<T, RAG> rows[4] = {reader(0), reader(1), reader(2), reader(3)};
    const T s = (T)a.scale[0];
    Quad<T> xq[4];
    auto request = [&](int st) {
#pragma unroll
        for (int i = 0; i < 4; ++i) xq[i] = rows[i].request(32 * st + 4 * q8);
    };
    auto stage_centroids = [&](int st, uint4 *buf) {
        if (TPC == 8 || wave < TPC) {
            const uint4 *src = a.image + (((size_t)(ch * TPC + wave)) * nb + 2 * st) * (2 * FRAG_UNITS) + lane;
#pragma unroll
            for (int i = 0; i < 4; ++i) to_lds16(src + i * FRAG_UNITS, buf + (wave * 4 + i) * FRAG_UNITS);
        }
    };
    auto store = [&](int st, uint4 *buf) {
        uint2 *const dst = reinterpret_cast<uint2 *>(buf + AU + (wave * 4 + 2 * (q8 >> 2)) * FRAG_UNITS + (q8 >> 1 & 1) * 32 + r8) + (q8 & 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const Quad<T> w = rows[i].keep(xq[i], 32 * st + 4 * q8);
            bf16x4 hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = (float)(w.v[e] * s);
                hi[e] = (__bf16)v;
                lo[e] = (__bf16)(v - (float)hi[e]);  // the difference is exact
            }
            dst[16 * i] = __builtin_bit_cast(uint2, hi);
            dst[16 * i + 2 * FRAG_UNITS] = __builtin_bit_cast(uint2, lo);
        }
    };

    floatx16 acc[CT][SC_PT];
    const int tile0 = ch * TPC + wc * CT;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const float *hv = a.start + (tile0 + c) * 32 + g * 16;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float h = hv[r];
#pragma unroll
            for (int pt = 0; pt < SC_PT; ++pt) acc[c][pt][r] = h;
        }
    }
    request(0);
    stage_centroids(0, lds4);
    store(0, lds4);
    request(min(1, ns - 1));
    wait_loads<0>();
    __syncthreads();
    for (int st = 0; st < ns; ++st) {
        const uint4 *buf = lds4 + (st & 1) * (AU + BU);
        uint4 *nxt = lds4 + ((st + 1) & 1) * (AU + BU);
        // (the last stage repeats itself into the buffer nobody reads: no branch in the loop)
        stage_centroids(min(st + 1, ns - 1), nxt);
        const uint4 *af = buf + (wc * CT) * 4 * FRAG_UNITS + lane;
        const uint4 *bf = buf + AU + (wp * 2) * 4 * FRAG_UNITS + lane;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            bf16x8 x0[SC_PT], x1[SC_PT];
#pragma unroll
            for (int pt = 0; pt < SC_PT; ++pt) {
                x0[pt] = __builtin_bit_cast(bf16x8, bf[(pt * 4 + 2 * k) * FRAG_UNITS]);
                x1[pt] = __builtin_bit_cast(bf16x8, bf[(pt * 4 + 2 * k + 1) * FRAG_UNITS]);
            }
            uint4 n0 = af[(2 * k) * FRAG_UNITS], n1 = af[(2 * k + 1) * FRAG_UNITS];
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const bf16x8 a0 = __builtin_bit_cast(bf16x8, n0);
                const bf16x8 a1 = __builtin_bit_cast(bf16x8, n1);
                if (c + 1 < CT) {
                    n0 = af[((c + 1) * 4 + 2 * k) * FRAG_UNITS];
                    n1 = af[((c + 1) * 4 + 2 * k + 1) * FRAG_UNITS];
                }
#pragma unroll
                for (int pt = 0; pt < SC_PT; ++pt)
                    acc[c][pt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, x0[pt], acc[c][pt], 0, 0, 0);
#pragma unroll
                for (int pt = 0; pt < SC_PT; ++pt)
                    acc[c][pt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, x1[pt], acc[c][pt], 0, 0, 0);
#pragma unroll
                for (int pt = 0; pt < SC_PT; ++pt)
                    acc[c][pt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, x0[pt], acc[c][pt], 0, 0, 0);
            }
        }
        store(min(st + 1, ns - 1), nxt);
        // fp32: reads two fragments ahead of the matrix instructions, the split after them - the rows requested
        // at the end of the last stage are then there, and the other wave of the SIMD fills its time.  (Spread
        // between the second block's instructions it waited for the rows: 60000 x 1024, K = 1024 461 us a call
        // against 437.)  fp64 rows take the registers the read-ahead needs: left to the compiler, 295 against 274
        // at 10^5 x 256, K = 1024.
        if constexpr (sizeof(T) == 4) {
            __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
            for (int i = 0; i < 2 * CT; ++i) {
                if (i + 1 == CT) __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
                else if (i + 1 < 2 * CT) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 3 * SC_PT, 0);
            }
        }
        request(min(st + 2, ns - 1));
        wait_loads<sizeof(T) == 4 ? 4 : 8>();  // the centroids have arrived; the rows requested above travel on
        __syncthreads();
    }
    // the records of the two centroid halves meet in LDS
    float *xm1 = reinterpret_cast<float *>(lds4), *xm2 = xm1 + SC_POINTS;
    int *xj = reinterpret_cast<int *>(xm2 + SC_POINTS);
    float m1[SC_PT], m2[SC_PT];
    int j1[SC_PT];
#pragma unroll
    for (int pt = 0; pt < SC_PT; ++pt) {
        ScanBest best;
        scan_best_init(best);
#pragma unroll
        for (int c = 0; c < CT; ++c) scan_best_add(best, acc[c][pt], tile0 + c);
        scan_best_finish(best, g, m1[pt], j1[pt], m2[pt]);
        if (wc == 1 && g == 0) {
            const int i = (wp * 2 + pt) * 32 + col;
            xm1[i] = m1[pt];
            xm2[i] = m2[pt];
            xj[i] = j1[pt];
        }
    }
    __syncthreads();
    if (wc == 0 && g == 0) {
#pragma unroll
        for (int pt = 0; pt < SC_PT; ++pt) {
            const int i = (wp * 2 + pt) * 32 + col;
            const float o1 = xm1[i], o2 = xm2[i];
            const bool mine = m1[pt] >= o1;
            const float hi = mine ? m1[pt] : o1, lo = mine ? o1 : m1[pt];
            const float sec = fmaxf(fmaxf(m2[pt], o2), lo);
            const int64_t p = (int64_t)pb * SC_POINTS + i;
            if (p < a.N)
                a.rec[(int64_t)ch * a.N + p] = ScanRecord{hi, sec, mine ? j1[pt] : xj[i], 0};
        }
    }
}

// ---- scan on fp16 pieces of rows of 129 .. 1024 features ---------------------------------------------
// One piece is a third of the matrix work, and the streaming scan does not follow: it reads and splits X once per 256
// centroids, a stage at a time between barriers (60000 x 1024, K = 1024: 230-260 us so shaped, 70 us of them matrix
// instructions).  Here a workgroup rounds the rows of 32 PT points once, into LDS (up to 128 KB), and sweeps all
// centroids without a barrier: each of its eight waves multiplies every eighth pair of centroid tiles, the
// image's fragments straight from L2 with RING blocks of 16 features in flight.  Two tiles at a time halve the LDS
// reads of an instruction, which would be its bound (a fragment of 1 KB per 32 cycles and SIMD), and all 64 (128)
// points that LDS holds share a read of the image (64 bytes a clock from L2: 2 MB per 64 points of 1024 features).
// The chain of a tile is long, so its 16 scores are compared one by one: three registers a point.
constexpr int SP_THREADS = 512, SP_WAVES = SP_THREADS / 64, SP_CT = 2;
constexpr int sp_ring(int pt) { return pt == 2 ? 8 : 4; }
template <typename T, int PT, bool RAG>
__global__ __launch_bounds__(SP_THREADS, 2) void scan_points_kernel(ScanArgs a, int nb)
{
    if (a.gate.closed<FORM_HALF>()) return;
    constexpr int P = 32 * PT, CT = SP_CT, RING = sp_ring(PT);
    extern __shared__ __align__(16) uint4 lds4[];  // [nb][PT][64] fragments; then the waves' records
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5;
    const int64_t p0 = (int64_t)blockIdx.x * P;
    const T *X = reinterpret_cast<const T *>(a.X);
    const T s = (T)a.scale[0];
    {
        // Wave w rounds point tile w % PT, every (8 / PT)th group of BATCH blocks.  Eight lanes take 32 features of a
        // row, whole lines of memory, and eight rows at a time: with a lane to a row a request names 64 places, one
        // after the other (whole calls 60000 x 1024, K = 1024 325 / 320 us, 131072 x 512, K = 1000 287 / 279,
        // 150000 x 200, K = 700 154 / 154).
        constexpr int BATCH = sizeof(T) == 4 ? 8 : 4;
        const int pt = wave % PT, q8 = lane & 7, r8 = lane >> 3;
        auto reader = [&](int i) { return RowReader<T, RAG>(X + min(p0 + pt * 32 + 8 * i + r8, a.N - 1) * a.D, a.D); };
        const RowReader<T, RAG> rows[4] = {reader(0), reader(1), reader(2), reader(3)};
        uint2 *const to = reinterpret_cast<uint2 *>(lds4 + pt * FRAG_UNITS + (q8 >> 1 & 1) * 32 + r8) + (q8 & 1);
        for (int b0 = wave / PT * BATCH; b0 < nb; b0 += SP_WAVES / PT * BATCH) {
            Quad<T> q[BATCH / 2][4];
#pragma unroll
            for (int k = 0; k < BATCH / 2; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) q[k][i] = rows[i].request(16 * (b0 + 2 * k) + 4 * q8);
#pragma unroll
            for (int k = 0; k < BATCH / 2; ++k) {
                const int b = b0 + 2 * k + (q8 >> 2);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const Quad<T> w = rows[i].keep(q[k][i], 16 * (b0 + 2 * k) + 4 * q8);
                    halfx4 h;
#pragma unroll
                    for (int e = 0; e < 4; ++e) h[e] = (_Float16)(float)(w.v[e] * s);
                    if (b < nb) to[2 * (b * PT * FRAG_UNITS + 8 * i)] = __builtin_bit_cast(uint2, h);
                }
            }
        }
    }
    float m1[PT], m2[PT];
    int j1[PT];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
        m1[pt] = m2[pt] = Mma<float>::neg_inf();
        j1[pt] = 0;
    }
    __syncthreads();
    const int pairs = (a.tiles + CT - 1) / CT;
    const size_t tile_units = (size_t)nb * FRAG_UNITS;
    auto fragments = [&](int t) { return a.image + (size_t)min(t, pairs - 1) * CT * tile_units + lane; };
    uint4 ring[RING][CT];
    const uint4 *f = fragments(wave);
#pragma unroll
    for (int u = 0; u < RING; ++u)
#pragma unroll
        for (int c = 0; c < CT; ++c) ring[u][c] = f[c * tile_units + u * FRAG_UNITS];
    floatx16 ci[CT];
    auto request_start = [&](int t) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const float *hv = a.start + (min(t, pairs - 1) * CT + c) * 32 + g * 16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const floatx4 h = *reinterpret_cast<const floatx4 *>(hv + 4 * i);
#pragma unroll
                for (int e = 0; e < 4; ++e) ci[c][4 * i + e] = h[e];
            }
        }
    };
    request_start(wave);
    const uint4 *xf = lds4 + lane;
    uint4 xn[PT];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) xn[pt] = xf[pt * FRAG_UNITS];
    for (int t = wave; t < pairs; t += SP_WAVES) {
        floatx16 acc[CT][PT];
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) acc[c][pt] = ci[c];
        const uint4 *const next = fragments(t + SP_WAVES);
        for (int b = 0; b < nb; b += RING) {
            f = b + RING < nb ? f + RING * FRAG_UNITS : next;
#pragma unroll
            for (int u = 0; u < RING; ++u) {
                halfx8 ah[CT], xh[PT];
#pragma unroll
                for (int c = 0; c < CT; ++c) ah[c] = __builtin_bit_cast(halfx8, ring[u][c]);
#pragma unroll
                for (int pt = 0; pt < PT; ++pt) xh[pt] = __builtin_bit_cast(halfx8, xn[pt]);
#pragma unroll
                for (int c = 0; c < CT; ++c) ring[u][c] = f[c * tile_units + u * FRAG_UNITS];
                const int bn = b + u + 1 < nb ? b + u + 1 : 0;
#pragma unroll
                for (int pt = 0; pt < PT; ++pt) xn[pt] = xf[(bn * PT + pt) * FRAG_UNITS];
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt)
                        acc[c][pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[c], xh[pt], acc[c][pt], 0, 0, 0);
            }
            // requests stay ahead of the instructions (left alone they all gather at the end of the loop)
#pragma unroll
            for (int u = 0; u < RING; ++u) {
                __builtin_amdgcn_sched_group_barrier(0x020, CT, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, PT, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, CT * PT, 0);
            }
        }
        request_start(t + SP_WAVES);
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = 32 * (t * CT + c) + 8 * (r >> 2) + (r & 3);
#pragma unroll
                for (int pt = 0; pt < PT; ++pt) {
                    const float v = acc[c][pt][r];
                    j1[pt] = v > m1[pt] ? j : j1[pt];
                    m2[pt] = __builtin_amdgcn_fmed3f(m1[pt], m2[pt], v);
                    m1[pt] = max2f(m1[pt], v);
                }
            }
    }
    __syncthreads();  // the fragments are done with
    float *xm1 = reinterpret_cast<float *>(lds4), *xm2 = xm1 + SP_WAVES * P;
    int *xj = reinterpret_cast<int *>(xm2 + SP_WAVES * P);
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
        const int j = j1[pt] + 4 * g;
        const float o1 = __shfl_xor(m1[pt], 32, 64), o2 = __shfl_xor(m2[pt], 32, 64);
        const int oj = __shfl_xor(j, 32, 64);
        const bool mine = m1[pt] > o1 || (m1[pt] == o1 && j < oj);
        if (g == 0) {
            const int i = wave * P + pt * 32 + col;
            xm1[i] = mine ? m1[pt] : o1;
            xm2[i] = fmaxf(fmaxf(m2[pt], o2), mine ? o1 : m1[pt]);
            xj[i] = mine ? j : oj;
        }
    }
    __syncthreads();
    if (tid < P) {
        float b1 = xm1[tid], b2 = xm2[tid];
        int j = xj[tid];
        for (int w = 1; w < SP_WAVES; ++w) {
            const float o1 = xm1[w * P + tid];
            const bool mine = b1 >= o1;
            b2 = fmaxf(fmaxf(b2, xm2[w * P + tid]), mine ? o1 : b1);
            j = mine ? j : xj[w * P + tid];
            b1 = mine ? b1 : o1;
        }
        const int64_t p = p0 + tid;
        if (p < a.N) a.rec[p] = ScanRecord{b1, b2, j, 0};
    }
}

// ---- resolve the listed points --------------------------------------------------------------------
// A workgroup repeats the scan for 32 listed points at a time, now noting every centroid whose score
// comes within the bound of the best, and evaluates those in direct-difference form in double, lowest
// index on equal distance.  A point with more of them than are noted (or none: scores that are not
// numbers) meets every centroid: see native_sweep(), then in double.  Listed points are few and scattered, so what counts is the
// time of one group: eight waves share its sweep, the points' fragments sit in LDS, the centroids'
// come straight from the image (L2), eight blocks in flight.  That read is what a group waits for (60000 x
// 1024, K = 1024: 4 MB at 64 bytes a clock, 120 us), so `splits` workgroups share the centroids of one
// group where the records leave room for their results; the last of them to finish combines these.
struct ResolveArgs {
    const uint4 *image;
    const float *start;
    const double *scale;
    ScanRecord *rec;
    int64_t N;
    int D, K, tiles, splits;
    int nb;             // blocks of a row, 0 where the fragments of 32 points do not fit LDS
    int side;           // workgroups that run side by side
    int32_t *labels;
    const ScanListed *list;
    const int32_t *list_count;
    int list_cap;
    int32_t *tickets;
    ftk_ft_stats *stats;
    ScanGate gate;
    // Lists of points that the third pass of a scan on fp16 pieces leaves; FORM_HALF writes them, the other form then
    // settles these instead of its own
    ScanListed *rest;
    int32_t *rest_count;
    int rest_cap;
};

// result of one workgroup for one point, in the place of its scan record
struct ResolveSlot {
    double d;
    int32_t j;  // -1: no candidate, -2: more than are noted
    int32_t unused;
};
static_assert(sizeof(ResolveSlot) == sizeof(ScanRecord), "layout");

// What differences of fp64 data are multiplied by before they are squared: the scale of the operands where squares of the
// data as they are would leave the range, so that distances can be compared at any scale; else 1 (fp32 data: always).
template <typename T>
struct SquareScale {
    double s;
    __device__ __forceinline__ explicit SquareScale(double scale)
        : s(sizeof(T) == 8 && (scale > 0x1p300 || scale < 0x1p-300) ? scale : 1.0)
    {
    }
    __device__ __forceinline__ double diff(T x, T c) const
    {
        if constexpr (sizeof(T) == 8) return (x - c) * s;
        else return (double)x - (double)c;
    }
    __device__ __forceinline__ T result(double d) const  // the distance itself
    {
        if constexpr (sizeof(T) == 8) return d / s / s;
        else return (T)d;
    }
};

// direct-difference distance in double by the L lanes of a group (every lane gets it)
template <typename T, int L>
__device__ __forceinline__ double group_sqdist(const T *x, const T *c, int D, int sub, const SquareScale<T> &q)
{
    const int Dq = D & ~3;
    double d = 0.0;
#pragma unroll 2
    for (int f = 4 * sub; f < Dq; f += 4 * L) {
        const Quad<T> xv = load_quad<T>(x + f), cv = load_quad<T>(c + f);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double t = q.diff(xv.v[e], cv.v[e]);
            d = fma(t, t, d);
        }
    }
    for (int f = Dq + sub; f < D; f += L) {
        const double t = q.diff(x[f], c[f]);
        d = fma(t, t, d);
    }
    return group_sum<L>(d);
}

// the same for P points against R centroids, whose elements are read once
template <typename T, int L, int P, int R>
__device__ __forceinline__ void group_sqdists(const T *const (&x)[P], const T *const (&c)[R], int D, int sub, const SquareScale<T> &q,
                                              double (&d)[P][R])
{
    const int Dq = D & ~3;
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
        for (int r = 0; r < R; ++r) d[i][r] = 0.0;
#pragma unroll 2
    for (int f = 4 * sub; f < Dq; f += 4 * L) {
        Quad<T> xv[P], cv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) cv[r] = load_quad<T>(c[r] + f);
#pragma unroll
        for (int i = 0; i < P; ++i) xv[i] = load_quad<T>(x[i] + f);
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double t = q.diff(xv[i].v[e], cv[r].v[e]);
                    d[i][r] = fma(t, t, d[i][r]);
                }
    }
    for (int f = Dq + sub; f < D; f += L)
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double t = q.diff(x[i][f], c[r][f]);
                d[i][r] = fma(t, t, d[i][r]);
            }
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
        for (int r = 0; r < R; ++r) d[i][r] = group_sum<L>(d[i][r]);
}


constexpr int RS_THREADS = 512, RS_WAVES = RS_THREADS / 64, RS_CAP = 8;

// ---- points with more candidates than are noted -----------------------------------------------------
// Data in several groups far from each other, or with one feature that dominates, leave a point every
// centroid of its group within the bound.  The bound of the data's own type may still tell them apart (fp64:
// nearly always), so up to 32 such points meet all centroids on the fp32 / fp64 matrix instructions first:
// best score, its centroid and the runner-up as the matrix kernels find them, from fragments read straight from
// memory (L2).  Two groups at +-1000, spread 5, K = 1024, every point listed with some 500 candidates, a call with
// all of them compared in double / here: fp64 2^18 x 32 6291 / 1040 us, 60000 x 512 15592 / 2508; fp32 2^18 x 32
// 6155 / 1254.  (The matrix kernels alone take 346, 1133 and 271 us of such data; of data in one piece 346, 1139
// and 188 us against 91, 315 and 93.)
// Wave w takes pairs of centroid tiles; what it finds goes to sh.*[w].
template <typename T>
struct NativeShared {
    T m1[RS_WAVES][32], m2[RS_WAVES][32];
    int j1[RS_WAVES][32];
    double cmax2[RS_WAVES], xn[32];
};

// E elements of a row from feature d0 by one access clamped into the row: those below d0 belong to another
// lane's fragment and count as zero here, and so does all of a fragment beyond D
template <typename T>
__device__ __forceinline__ typename Mma<T>::frag_t native_frag(const T *row, int d0, int D)
{
    constexpr int E = Mma<T>::E;
    const int off = min(d0, D - E);
    typename Mma<T>::frag_t f;
    if constexpr (sizeof(T) == 4) f = *reinterpret_cast<const float4e *>(row + off);
    else f = *reinterpret_cast<const double2e *>(row + off);
#pragma unroll
    for (int e = 0; e < E; ++e) f[e] = off + e >= d0 ? f[e] : T(0);
    return f;
}

template <typename T>
__device__ __forceinline__ void native_sweep(const T *X, const T *C, int D, int K, const int32_t *points, const int *left,
                                             int nleft, NativeShared<T> &sh)
{
    using M = Mma<T>;
    constexpr int E = M::E, TM = M::TM, NT = 32 / M::TN, CT = 2;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane % TM, g = lane / TM;
    const int nq = (D + 7) >> 3;
    const T *x[NT];
    T m1[NT], m2[NT];
    int j1[NT];
    double xn[NT], cmax2 = 0.0;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        x[nt] = X + (int64_t)points[left[min(nt * M::TN + row, nleft - 1)]] * D;
        m1[nt] = m2[nt] = M::neg_inf();
        j1[nt] = 0;
    }
    for (int j0 = wave * CT * TM; j0 < K; j0 += RS_WAVES * CT * TM) {
        const T *c[CT];
        typename M::acc_t acc[CT][NT];
        double cn[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            c[ct] = C + (size_t)min(j0 + ct * TM + row, K - 1) * D;
            cn[ct] = 0.0;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < M::R; ++r) acc[ct][nt][r] = T(0);
        }
        typename M::frag_t xf[NT], cf[CT], xg[NT], cg[CT];
        auto request = [&](int q) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) xg[nt] = native_frag<T>(x[nt], 8 * q + E * g, D);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) cg[ct] = native_frag<T>(c[ct], 8 * q + E * g, D);
        };
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) xn[nt] = 0.0;
        request(0);
        for (int q = 0; q < nq; ++q) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) xf[nt] = xg[nt];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) cf[ct] = cg[ct];
            request(min(q + 1, nq - 1));
#pragma unroll
            for (int e = 0; e < E; ++e) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[ct][nt] = M::mma(cf[ct][e], xf[nt][e], acc[ct][nt]);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) cn[ct] = fma((double)cf[ct][e], (double)cf[ct][e], cn[ct]);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) xn[nt] = fma((double)xf[nt][e], (double)xf[nt][e], xn[nt]);
            }
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
            for (int k = TM; k < 64; k <<= 1) cn[ct] += __shfl_xor(cn[ct], k, 64);
            cmax2 = cn[ct] > cmax2 ? cn[ct] : cmax2;  // (rows beyond K repeat the last one)
#pragma unroll
            for (int r = 0; r < M::R; ++r) {
                const T h = (T)(0.5 * __shfl(cn[ct], M::row(r, g), 64));
                const int j = j0 + ct * TM + M::row(r, g);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const T v = j < K ? acc[ct][nt][r] - h : M::neg_inf();
                    const bool better = v > m1[nt];  // (a score that is not a number counts for nothing)
                    const T low = better ? m1[nt] : v;
                    m2[nt] = low > m2[nt] ? low : m2[nt];
                    m1[nt] = better ? v : m1[nt];
                    j1[nt] = better ? j : j1[nt];
                }
            }
        }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
        for (int k = TM; k < 64; k <<= 1) {
            const T o1 = __shfl_xor(m1[nt], k, 64), o2 = __shfl_xor(m2[nt], k, 64);
            const int oj = __shfl_xor(j1[nt], k, 64);
            const bool other = o1 > m1[nt];
            const T low = other ? m1[nt] : o1;
            m2[nt] = o2 > m2[nt] ? o2 : m2[nt];
            m2[nt] = low > m2[nt] ? low : m2[nt];
            m1[nt] = other ? o1 : m1[nt];
            j1[nt] = other ? oj : j1[nt];
            xn[nt] += __shfl_xor(xn[nt], k, 64);
        }
        if (g == 0) {
            sh.m1[wave][nt * M::TN + row] = m1[nt];
            sh.m2[wave][nt * M::TN + row] = m2[nt];
            sh.j1[wave][nt * M::TN + row] = j1[nt];
            if (wave == 0) sh.xn[nt * M::TN + row] = xn[nt];
        }
    }
#pragma unroll
    for (int k = 1; k < TM; k <<= 1) {
        const double o = __shfl_xor(cmax2, k, 64);
        cmax2 = o > cmax2 ? o : cmax2;
    }
    if (lane == 0) sh.cmax2[wave] = cmax2;
}

// the centroid of point i, or -1 where its scores do not tell (a NaN or an infinity among them: the bound does not hold)
template <typename T>
__device__ __forceinline__ int native_verdict(const NativeShared<T> &sh, int i, int D)
{
    T m1 = sh.m1[0][i], m2 = sh.m2[0][i];
    int j1 = sh.j1[0][i];
    double cmax2 = sh.cmax2[0];
    for (int w = 1; w < RS_WAVES; ++w) {
        const T o1 = sh.m1[w][i], o2 = sh.m2[w][i];
        const bool other = o1 > m1;
        const T low = other ? m1 : o1;
        m2 = o2 > m2 ? o2 : m2;
        m2 = low > m2 ? low : m2;
        m1 = other ? o1 : m1;
        j1 = other ? sh.j1[w][i] : j1;
        cmax2 = sh.cmax2[w] > cmax2 ? sh.cmax2[w] : cmax2;
    }
    // the band of the matrix kernels (see ftk_assign_generic.hip): D products and the sum's start, each rounded
    const double big = sqrt(sh.xn[i] * cmax2) + 0.5 * cmax2;
    const double band = 2.0 * (double)(((D + 7) & ~7) + 4) * Mma<T>::kEps * big;
    // (what underflow takes from the products is below the band)
    const bool sound = big < 0.25 * (sizeof(T) == 4 ? 3e38 : 1e308) && big > (sizeof(T) == 4 ? 0x1p-96 : 0x1p-960);
    return sound && (double)m1 - (double)m2 > band ? j1 : -1;
}

// GATED: in a call that chooses its form
template <typename T, int FORM, int L, bool GATED>
__global__ __launch_bounds__(RS_THREADS, FORM == FORM_HALF ? 4 : 2) void scan_resolve_kernel(const T *X, const T *C, T *mindist, ResolveArgs a)
{
    constexpr int NP = form_pieces(FORM), FR = form_frags(FORM);
    constexpr int GROUPS = RS_THREADS / L;
    extern __shared__ __align__(16) uint4 lds4[];  // [nb][NP][64] fragments of the 32 points
    __shared__ int32_t sh_p[32];
    __shared__ float sh_thr[32];
    __shared__ int sh_cnt[32];
    __shared__ int32_t sh_j[32][RS_CAP];
    __shared__ double sh_d[32][RS_CAP];
    __shared__ double sh_bd[4][RS_WAVES];
    __shared__ int sh_bj[4][RS_WAVES];
    __shared__ int sh_left[32], sh_nleft;  // points that no list of candidates settled
    __shared__ NativeShared<T> sh_native;
    __shared__ double sh_bd32[32];
    __shared__ int32_t sh_code[32];
    __shared__ int sh_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5;
    const int sub = tid & (L - 1), grp = tid / L;
    const bool rest = GATED && FORM != FORM_HALF && a.gate.half();
    if (FORM == FORM_HALF && a.gate.closed<FORM>()) return;
    const ScanListed *const list = rest ? a.rest : a.list;
    const int32_t *const list_count = rest ? a.rest_count : a.list_count;
    const int list_cap = rest ? a.rest_cap : a.list_cap;
    const T s = (T)a.scale[0];
    const SquareScale<T> sq(a.scale[0]);
    __shared__ int sh_pre[SCAN_LISTS + 1];  // listed points before each list
    __shared__ int32_t sh_job[32 * RS_CAP];
    __shared__ int sh_jobs;
    if (wave == 0) {
        int v = list_count[lane * LIST_STRIDE];
#pragma unroll
        for (int k = 1; k < 64; k <<= 1) {
            const int o = __shfl_up(v, k, 64);
            v += lane >= k ? o : 0;
        }
        sh_pre[lane + 1] = v;
        if (lane == 0) sh_pre[0] = 0;
    }
    __syncthreads();
    const int n = sh_pre[SCAN_LISTS];
    // workgroups per group: no more than run side by side
    const int nb = rest ? 0 : a.nb;  // (what is left over meets all centroids)
    const int S = rest ? 1 : max(1, min(a.splits, a.side / max(1, (n + 31) / 32)));
    const int split = (int)blockIdx.x % S, per = (a.tiles + S - 1) / S;
    const int tile_end = min(a.tiles, (split + 1) * per);
    auto listed_point = [&](int i) {  // the i-th of all lists
        int q = 0;
#pragma unroll
        for (int k = SCAN_LISTS / 2; k >= 1; k >>= 1) q += sh_pre[q + k] <= i ? k : 0;
        return list[(int64_t)q * list_cap + (i - sh_pre[q])];
    };
    if (a.stats && !rest && blockIdx.x == 0 && tid == 0 && n > 0) atomicAdd((unsigned long long *)&a.stats->refined, (unsigned long long)n);
    if ((int)blockIdx.x / S >= (int)gridDim.x / S) return;  // a remainder of the grid
    // points per group: 32, or fewer of the rows that meet all centroids right away, while that leaves workgroups idle
    const int per_group = nb ? 32 : max(1, min(32, (n + a.side - 1) / a.side));
    for (int64_t at = (int64_t)((int)blockIdx.x / S) * per_group; at < n; at += (int64_t)((int)gridDim.x / S) * per_group) {
        const int first = (int)at, np = min(per_group, n - first);
        __syncthreads();  // the previous group is written out
        if (tid < 32) {
            const ScanListed e = listed_point(first + min(tid, np - 1));
            sh_p[tid] = e.point;
            sh_thr[tid] = e.thr;
            sh_cnt[tid] = nb ? 0 : RS_CAP + 1;  // rows too long for that: all centroids
        }
        __syncthreads();
        const RowReader<T, true> row(X + (int64_t)sh_p[col] * a.D, a.D);
#pragma unroll(FORM == FORM_HALF ? 4 : 2)
        for (int b = wave; b < nb; b += RS_THREADS / 64) {
            const int f0 = FORM == FORM_OCTET ? 0 : 16 * b + 8 * g;
            const Quad<T> q0 = row.keep(row.request(f0), f0), q1 = row.keep(row.request(f0 + 4), f0 + 4);
            float v[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = (float)(q0.v[e] * s);
                v[4 + e] = (float)(q1.v[e] * s);
            }
            uint4 *dst = lds4 + b * NP * FRAG_UNITS + lane;
            if constexpr (FORM == FORM_HALF) {
                dst[0] = round_half(v);
            } else if constexpr (FORM != FORM_PAIR) {
                uint4 x0, x1, x2;
                split_triple(v, x0, x1, x2);
                dst[0] = x0;
                dst[FRAG_UNITS] = x1;
                dst[2 * FRAG_UNITS] = FORM == FORM_TRIPLE ? x2 : select_units(g != 0, x2, x0);
            } else {
                uint4 x0, x1;
                split_pair(v, x0, x1);
                dst[0] = x0;
                dst[FRAG_UNITS] = x1;
            }
        }
        __syncthreads();
        const float thr = sh_thr[col];
        // this wave's tiles, block by block, `RING` blocks and the next tile's start values in flight
        const int t0 = split * per + wave;
        const int total = t0 < tile_end ? ((tile_end - t0 - 1) / (RS_THREADS / 64) + 1) * nb : 0;
        constexpr int RING = FORM == FORM_HALF ? 8 : 4;
        uint4 ring[RING][FR];
        int lt = t0, lb = 0;  // tile and block of the next request
        auto request = [&](uint4 (&r)[FR]) {
            const uint4 *f = a.image + ((size_t)min(lt, a.tiles - 1) * a.nb + lb) * (FR * FRAG_UNITS) + lane;
#pragma unroll
            for (int i = 0; i < FR; ++i) r[i] = f[i * FRAG_UNITS];
            if (++lb == a.nb) {
                lb = 0;
                lt += RS_THREADS / 64;
            }
        };
        floatx16 ci, acc;
        auto request_start = [&](int t) {
            const float *hv = a.start + min(t, a.tiles - 1) * 32 + g * 16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const floatx4 h = *reinterpret_cast<const floatx4 *>(hv + 4 * i);
#pragma unroll
                for (int e = 0; e < 4; ++e) ci[4 * i + e] = h[e];
            }
        };
        request_start(t0);
#pragma unroll
        for (int u = 0; u < RING; ++u) request(ring[u]);
        int t = t0, b = 0;
        for (int i = 0; i < total; i += RING) {
#pragma unroll
            for (int u = 0; u < RING; ++u) {
                if (i + u >= total) break;
                if (b == 0) {
                    acc = ci;
                    request_start(t + RS_THREADS / 64);
                }
                const uint4 *q = lds4 + b * NP * FRAG_UNITS + lane;
                if constexpr (FORM == FORM_HALF) {
                    const halfx8 a0 = __builtin_bit_cast(halfx8, ring[u][0]);
                    request(ring[u]);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, __builtin_bit_cast(halfx8, q[0]), acc, 0, 0, 0);
                } else {
                    const bf16x8 a0 = __builtin_bit_cast(bf16x8, ring[u][0]);
                    const bf16x8 a1 = __builtin_bit_cast(bf16x8, ring[u][1]);
                    const bf16x8 a2 = __builtin_bit_cast(bf16x8, ring[u][FR - 1]);
                    request(ring[u]);
                    const bf16x8 x0 = __builtin_bit_cast(bf16x8, q[0]);
                    const bf16x8 x1 = __builtin_bit_cast(bf16x8, q[FRAG_UNITS]);
                    const bf16x8 x2 = __builtin_bit_cast(bf16x8, q[(NP - 1) * FRAG_UNITS]);
                    if constexpr (FORM == FORM_TRIPLE) {
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, x0, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, x1, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, x2, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, x0, acc, 0, 0, 0);
                    } else {
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, FORM == FORM_OCTET ? x2 : x0, acc, 0, 0, 0);
                    }
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, x1, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, x0, acc, 0, 0, 0);
                }
                if (++b < a.nb) continue;
                float tm = fmaxf(acc[0], acc[1]);
#pragma unroll
                for (int r = 2; r < 16; r += 2) tm = max3f(tm, acc[r], acc[r + 1]);
                if (__any(tm >= thr)) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int j = 32 * t + 8 * (r >> 2) + 4 * g + (r & 3);
                        if (acc[r] >= thr && j < a.K) {
                            const int at = atomicAdd(&sh_cnt[col], 1);
                            if (at < RS_CAP) sh_j[col][at] = j;
                        }
                    }
                }
                b = 0;
                t += RS_THREADS / 64;
            }
        }
        __syncthreads();
        if (tid < 64) {  // the candidates as one list of jobs
            const int m = tid < np ? sh_cnt[tid] : 0;
            const int mm = m <= RS_CAP ? m : 0;
            int v = mm;
#pragma unroll
            for (int k = 1; k < 32; k <<= 1) {
                const int o = __shfl_up(v, k, 64);
                v += lane >= k ? o : 0;
            }
            for (int i = 0; i < mm; ++i) sh_job[v - mm + i] = tid * RS_CAP + i;
            if (tid == 31) sh_jobs = v;
        }
        __syncthreads();
        for (int q = grp; q < sh_jobs; q += GROUPS) {
            const int k = sh_job[q] / RS_CAP, at = sh_job[q] % RS_CAP;
            const double d = group_sqdist<T, L>(X + (int64_t)sh_p[k] * a.D, C + (size_t)sh_j[k][at] * a.D, a.D, sub, sq);
            if (sub == 0) sh_d[k][at] = d;
        }
        __syncthreads();
        if (tid < np) {
            const int m = sh_cnt[tid];
            double d = __builtin_huge_val();
            int j = m > RS_CAP ? -2 : -1;
            if (m <= RS_CAP)
                for (int i = 0; i < m; ++i) {
                    const double di = sh_d[tid][i];
                    const int ji = sh_j[tid][i];
                    const bool better = j < 0 || di < d || (di == d && ji < j);
                    d = better ? di : d;
                    j = better ? ji : j;
                }
            if (S > 1) {
                ResolveSlot *slot = reinterpret_cast<ResolveSlot *>(a.rec + (int64_t)split * a.N + sh_p[tid]);
                // written and read past the caches that other XCDs do not see: a device-wide fence
                // here would write back a whole L2
                __hip_atomic_store(&slot->d, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&slot->j, j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            sh_bd32[tid] = d;
            sh_code[tid] = j;
        }
        if (S > 1) {
            __builtin_amdgcn_s_waitcnt(0);  // the slots are written
            __syncthreads();
            if (tid == 0) sh_last = atomicAdd(&a.tickets[first / 32], 1) == S - 1;
            __syncthreads();
            if (!sh_last) continue;
            if (tid < np) {
                double d = __builtin_huge_val();
                int j = -1;
                for (int i = 0; i < S; ++i) {
                    ResolveSlot *slot = reinterpret_cast<ResolveSlot *>(a.rec + (int64_t)i * a.N + sh_p[tid]);
                    const double di = __hip_atomic_load(&slot->d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const int ji = __hip_atomic_load(&slot->j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (ji == -2 || j == -2) {
                        j = -2;
                    } else if (ji >= 0 && (j < 0 || di < d || (di == d && ji < j))) {
                        d = di;
                        j = ji;
                    }
                }
                sh_bd32[tid] = d;
                sh_code[tid] = j;
            }
        }
        if (tid < np && sh_code[tid] >= 0) {
            a.labels[sh_p[tid]] = sh_code[tid];
            if (mindist) mindist[sh_p[tid]] = sq.result(sh_bd32[tid]);
        }
        if constexpr (FORM == FORM_HALF) {  // without what follows: half the registers, two workgroups a compute unit
            if (tid < np && sh_code[tid] < 0) {
                const int which = first / 32 % SCAN_LISTS;
                const int slot = atomicAdd(a.rest_count + which * LIST_STRIDE, 1);
                a.rest[(int64_t)which * a.rest_cap + slot] = ScanListed{sh_p[tid], __builtin_nanf("")};
            }
            continue;
        }
        __syncthreads();
        auto collect = [&] {
            if (tid < 64) {
                const bool open = tid < np && sh_code[tid] < 0;
                const unsigned long long m = __ballot(open);
                if (open) sh_left[__popcll(m & ((1ull << tid) - 1ull))] = tid;
                if (tid == 0) sh_nleft = __popcll(m);
            }
            __syncthreads();
        };
        collect();
        // A few points meet all centroids faster below: one, or of rows beyond 1152 features up to eight (7382 x 2419,
        // K = 289, 7 points a group 580 us a call against 592; 20000 x 2000, K = 256, 14 points 853 against 664).
        // Of long fp32 rows the matrix instructions can tell little more than the scan: their band is
        // 3 (D + 4) u of the norms squared, the scan's some (560 + 4 D) u.
        if (const int nleft = sh_nleft; nleft > (a.nb ? 1 : 8) && (sizeof(T) == 8 || a.D <= 256)) {
            native_sweep<T>(X, C, a.D, a.K, sh_p, sh_left, nleft, sh_native);
            __syncthreads();
            if (tid < nleft) {
                const int j = native_verdict<T>(sh_native, tid, a.D);
                if (j >= 0) a.labels[sh_p[sh_left[tid]]] = j;
                sh_code[sh_left[tid]] = j;
            }
            __syncthreads();
            if (mindist)
                for (int q = grp; q < nleft; q += GROUPS) {
                    const int k = sh_left[q], j = sh_code[k];
                    if (j < 0) continue;
                    const double d = group_sqdist<T, L>(X + (int64_t)sh_p[k] * a.D, C + (size_t)j * a.D, a.D, sub, sq);
                    if (sub == 0) mindist[sh_p[k]] = sq.result(d);
                }
            __syncthreads();
            collect();
        }
        // what is left: every centroid in double, up to four points at a time
        auto compare_all = [&](auto count, auto rows, int k0) {
            constexpr int P = decltype(count)::value, R = decltype(rows)::value;  // R centroids at once: loads in flight
            const T *x[P];
            double best[P];
            int bj[P];
#pragma unroll
            for (int i = 0; i < P; ++i) {
                x[i] = X + (int64_t)sh_p[sh_left[min(k0 + i, sh_nleft - 1)]] * a.D;
                best[i] = __builtin_huge_val();
                bj[i] = 0x7fffffff;
            }
            for (int j0 = grp; j0 < a.K; j0 += R * GROUPS) {
                const T *c[R];
#pragma unroll
                for (int r = 0; r < R; ++r) c[r] = C + (size_t)min(j0 + r * GROUPS, a.K - 1) * a.D;
                double d[P][R];
                group_sqdists<T, L, P, R>(x, c, a.D, sub, sq, d);
#pragma unroll
                for (int i = 0; i < P; ++i)
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int j = j0 + r * GROUPS;
                        if (j < a.K && d[i][r] < best[i]) {  // j increases: the first of equal ones stays
                            best[i] = d[i][r];
                            bj[i] = j;
                        }
                    }
            }
            __syncthreads();  // the results of the points before these have been read
#pragma unroll
            for (int i = 0; i < P; ++i) {
#pragma unroll
                for (int q = 32; q >= L; q >>= 1) {
                    const double od = __shfl_xor(best[i], q, 64);
                    const int oj = __shfl_xor(bj[i], q, 64);
                    const bool take = od < best[i] || (od == best[i] && oj < bj[i]);
                    best[i] = take ? od : best[i];
                    bj[i] = take ? oj : bj[i];
                }
                if (lane == 0) {
                    sh_bd[i][wave] = best[i];
                    sh_bj[i][wave] = bj[i];
                }
            }
            __syncthreads();
            if (tid < P && k0 + tid < sh_nleft) {
                double d = sh_bd[tid][0];
                int j = sh_bj[tid][0];
                for (int w = 1; w < RS_WAVES; ++w)
                    if (sh_bd[tid][w] < d || (sh_bd[tid][w] == d && sh_bj[tid][w] < j)) {
                        d = sh_bd[tid][w];
                        j = sh_bj[tid][w];
                    }
                const int32_t p = sh_p[sh_left[k0 + tid]];
                a.labels[p] = j == 0x7fffffff ? 0 : j;
                if (mindist) mindist[p] = sq.result(d);
            }
        };
        for (int k0 = 0; k0 < sh_nleft; k0 += 4) {
            if (sh_nleft - k0 == 1) compare_all(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{}, k0);
            else compare_all(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{}, k0);
        }
    }
}

// ---- listed points of a scan on fp16 pieces, rows of up to 128 features -------------------------------
// These are some percent of all points, most with two candidates, so their sweep is shaped like the scan itself: fragments
// in registers.  (By scan_resolve_kernel, 32 points a group and a chain of latencies
// each: 160 us for the 68 000 points of 2^21 x 32, K = 4096.)  The four waves of a workgroup share 64 points
// and take every fourth tile, its fragments straight from L2 while those before are multiplied (256 points of their own
// each took 123 us, one workgroup per compute unit; the image in chunks through LDS 86 us; so 69).  A lane notes the centroids
// whose score reaches its point's threshold; then L lanes at a time evaluate them in double.  A point with
// more of them than are noted goes on to scan_resolve_kernel, to meet all centroids.
struct RecheckArgs {
    const ScanListed *list;
    const int32_t *list_count;
    int list_cap;
    ScanListed *rest;
    int32_t *rest_count;
    int rest_cap;
    int K;
    int32_t *labels;
    ftk_ft_stats *stats;
};
constexpr int RC_CAP = 6, RC_POINTS = SC_PT * 32;

template <typename T, int NB, bool RAG, int L>
__global__ __launch_bounds__(SC_THREADS, (NB <= 2 ? 4 : (NB <= 4 ? 3 : 2)))
void scan_recheck_kernel(const T *X, const T *C, T *mindist, ScanArgs a, RecheckArgs r)
{
    if (a.gate.closed<FORM_HALF>()) return;
    constexpr int TU = NB * FRAG_UNITS;
    constexpr int GROUPS = SC_THREADS / L;
    __shared__ int sh_pre[SCAN_LISTS + 1];
    __shared__ int32_t sh_p[RC_POINTS];
    __shared__ float sh_thr[RC_POINTS];
    __shared__ int sh_cnt[RC_POINTS];
    __shared__ int32_t sh_j[RC_POINTS][RC_CAP];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5;
    const int sub = tid & (L - 1), grp = tid / L;
    if (wave == 0) {
        int v = r.list_count[lane * LIST_STRIDE];
#pragma unroll
        for (int k = 1; k < 64; k <<= 1) {
            const int o = __shfl_up(v, k, 64);
            v += lane >= k ? o : 0;
        }
        sh_pre[lane + 1] = v;
        if (lane == 0) sh_pre[0] = 0;
    }
    __syncthreads();
    const int n = sh_pre[SCAN_LISTS];
    if (r.stats && blockIdx.x == 0 && tid == 0 && n > 0) atomicAdd((unsigned long long *)&r.stats->refined, (unsigned long long)n);
    const T s = (T)a.scale[0];
    const SquareScale<T> sq(a.scale[0]);
    for (int64_t first = (int64_t)blockIdx.x * RC_POINTS; first < n; first += (int64_t)gridDim.x * RC_POINTS) {
        __syncthreads();  // the points before these are done
        if (tid < RC_POINTS) {
            const int64_t i = first + tid < n ? first + tid : n - 1;
            int q = 0;
#pragma unroll
            for (int k = SCAN_LISTS / 2; k >= 1; k >>= 1) q += sh_pre[q + k] <= i ? k : 0;
            const ScanListed e = r.list[(int64_t)q * r.list_cap + (i - sh_pre[q])];
            sh_p[tid] = e.point;
            sh_thr[tid] = first + tid < n ? e.thr : __builtin_huge_valf();
            sh_cnt[tid] = 0;
        }
        __syncthreads();
        uint4 b[SC_PT][NB];
        float thr[SC_PT];
#pragma unroll
        for (int pt = 0; pt < SC_PT; ++pt) {
            const int i = pt * 32 + col;
            thr[pt] = sh_thr[i];
            const RowReader<T, RAG> row(X + (int64_t)sh_p[i] * a.D, a.D);
            Quad<T> q[2 * NB];
#pragma unroll
            for (int u = 0; u < 2 * NB; ++u) q[u] = row.request(16 * (u >> 1) + 8 * g + 4 * (u & 1));
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                float v[8];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const Quad<T> w = row.keep(q[2 * k + h], 16 * k + 8 * g + 4 * h);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[4 * h + e] = (float)(w.v[e] * s);
                }
                b[pt][k] = round_half(v);
            }
        }
        // this wave's tiles, fragments and start values of the next one requested ahead
        uint4 f[NB];
        floatx4 h[4];
        auto request = [&](int t) {
            const uint4 *src = a.image + (size_t)min(t, a.tiles - 1) * TU + lane;
#pragma unroll
            for (int k = 0; k < NB; ++k) f[k] = src[k * FRAG_UNITS];
            const float *hv = a.start + min(t, a.tiles - 1) * 32 + g * 16;
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = *reinterpret_cast<const floatx4 *>(hv + 4 * i);
        };
        request(wave);
        for (int t = wave; t < a.tiles; t += SC_THREADS / 64) {
            floatx16 acc[SC_PT];
            halfx8 af[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) af[k] = __builtin_bit_cast(halfx8, f[k]);
#pragma unroll
            for (int i = 0; i < 16; ++i)
#pragma unroll
                for (int pt = 0; pt < SC_PT; ++pt) acc[pt][i] = h[i / 4][i % 4];
            request(t + SC_THREADS / 64);
#pragma unroll
            for (int k = 0; k < NB; ++k)
#pragma unroll
                for (int pt = 0; pt < SC_PT; ++pt)
                    acc[pt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[k], __builtin_bit_cast(halfx8, b[pt][k]), acc[pt], 0, 0, 0);
#pragma unroll
            for (int pt = 0; pt < SC_PT; ++pt) {
                float tm = fmaxf(acc[pt][0], acc[pt][1]);
#pragma unroll
                for (int i = 2; i < 16; i += 2) tm = max3f(tm, acc[pt][i], acc[pt][i + 1]);
                if (__any(tm >= thr[pt])) {
                    const int at = pt * 32 + col;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int j = 32 * t + 8 * (i >> 2) + 4 * g + (i & 3);
                        if (acc[pt][i] >= thr[pt] && j < r.K) {
                            const int slot = atomicAdd(&sh_cnt[at], 1);
                            if (slot < RC_CAP) sh_j[at][slot] = j;
                        }
                    }
                }
            }
        }
        __syncthreads();
        const int np = (int)(n - first < RC_POINTS ? n - first : RC_POINTS);
        for (int i = grp; i < np; i += GROUPS) {
            const int m = sh_cnt[i], p = sh_p[i];
            if (m < 1 || m > RC_CAP) {
                if (sub == 0) {
                    const int which = (int)((first / RC_POINTS) % SCAN_LISTS);
                    const int slot = atomicAdd(r.rest_count + which * LIST_STRIDE, 1);
                    r.rest[(int64_t)which * r.rest_cap + slot] = ScanListed{p, __builtin_nanf("")};
                }
                continue;
            }
            const T *const x[1] = {X + (int64_t)p * a.D};
            double best = __builtin_huge_val();
            int bj = -1;
            for (int k = 0; k < m; k += 2) {
                const int j0 = sh_j[i][k], j1 = sh_j[i][min(k + 1, m - 1)];
                const T *const c[2] = {C + (size_t)j0 * a.D, C + (size_t)j1 * a.D};
                double d[1][2];
                group_sqdists<T, L, 1, 2>(x, c, a.D, sub, sq, d);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int j = q ? j1 : j0;
                    const bool better = bj < 0 || d[0][q] < best || (d[0][q] == best && j < bj);
                    best = better ? d[0][q] : best;
                    bj = better ? j : bj;
                }
            }
            if (sub == 0) {
                r.labels[p] = bj;
                if (mindist) mindist[p] = sq.result(best);
            }
        }
    }
}

// ---- host ----------------------------------------------------------------------------------------
static int resident_blocks(int D)
{
    const int nb = (int)ceil_div(D, 16);
    return nb <= 4 ? nb : (nb <= 6 ? 6 : 8);
}

// From how many centroids on the scan beats the fp32 / fp64 matrix kernels.  They read X once, keep it in
// registers and settle in place; the scan reads it twice in four launches but multiplies 16 (32) times as fast, so
// what counts is the matrix work, and how it lies on the chip:
//   few points (up to 36 000): neither fills it.  A matrix kernel's time is one workgroup's sweep over K, the scan
//                cuts the sweep up; long rows make the sweep longer, so the line falls with D.
//   around 60 000: the matrix kernels fill it once, the scan's launches show, and the line is highest.
//   from 110 000 (450 000) on: both fill it; launches do not count, and the line is where the matrix work
//                exceeds the second read of X.
// fp64 falls lower than fp32 as its matrix instructions are half as fast.  Measured on 2487 calls (15 widths of 4 ..
// 1024, 14 counts of 8 .. 2048, 7 numbers of points of 300 .. 10^6, blobs and uniform data), matrix kernel / scan, just
// below and on the line, us:
//   fp32  D = 128  N = 1500 K = 64 20.2 / 23.7, 96 26.3 / 24.4; N = 60000 K = 128 28.8 / 34.5, 256 47.2 / 38.6;
//                  N = 200000 K = 64 50.3 / 57.5, 96 71.0 / 61.2
//         D = 16   N = 20000 K = 512 31.5 / 23.6; N = 60000 K = 256 21.8 / 21.9, 512 31.6 / 25.1; N = 10^6 K = 64 43.5 / 51.5, 96 69.0 / 56.4
//         D = 4    N = 60000 K = 512 22.8 / 28.4, 1024 33.4 / 32.2; N = 10^6 K = 256 61.1 / 62.2, 512 96.1 / 88.0
//   fp64  D = 32   N = 20000 K = 192 21.2 / 22.0, 384 33.4 / 23.1; N = 60000 K = 128 22.3 / 23.2, 256 34.5 / 27.3; N = 200000 K = 64 34.0 / 37.6,
//                  96 47.1 / 38.7
// Rows beyond 128 features again with the matrix kernels that read them by lines (3000 .. 10^6 points, 132 .. 1600
// features, 8 .. 224 centroids, some 2300 calls):
//   fp32  N = 20000 D = 256 K = 48 32 / 39, 66 52 / 43; D = 512 K = 48 62 / 58; N = 60000 D = 132 K = 80 36 / 45; D = 320 K = 50 55 / 54, 80
//         73 / 64; D = 1024 K = 50 155 / 133; N = 200000 D = 256 K = 64 89 / 97, 80 141 / 112; D = 1000 K = 64 392 / 400; N = 500000
//         D = 256 K = 50 199 / 224, 80 276 / 257
//   fp64  N = 20000 D = 256 K = 100 54 / 53, 130 71 / 54; D = 1024 K = 115 176 / 140; N = 60000 D = 256 K = 80 70 / 75, 115 92 / 76;
//         N = 200000 D = 320 K = 50 184 / 233, 100 316 / 253; N = 500000 D = 256 K = 66 451 / 420, 100 553 / 425
static int scan_from(ftk_dtype dtype, int64_t N, int D)
{
    static const int from[2][5][9] = {
        // D < 8, 8, .. 16, .. 48, .. 128, .. 160, .. 384, .. 1024, beyond
        {{768, 512, 256, 160, 96, 48, 48, 48, 48},       // fp32: N < 9 000
         {768, 512, 320, 176, 160, 80, 65, 48, 48},      //       N < 36 000
         {1024, 640, 448, 256, 224, 113, 80, 48, 65},    //       N < 110 000
         {768, 640, 160, 96, 96, 96, 65, 65, 96},        //       N < 450 000
         {384, 384, 96, 72, 72, 96, 65, 65, 96}},        //       more
        {{512, 512, 384, 160, 160, 144, 144, 144, 144},  // fp64
         {512, 512, 384, 288, 272, 129, 112, 129, 129},
         {512, 512, 320, 192, 224, 112, 96, 96, 113},
         {96, 96, 96, 96, 96, 81, 81, 65, 96},
         {48, 48, 48, 72, 80, 81, 81, 81, 96}}};
    const int beyond[] = {160, 384, 1024};
    int d = D < 8 ? 0 : (D == 8 ? 1 : (D <= 16 ? 2 : (D <= 48 ? 3 : (D <= 128 ? 4 : 5))));
    for (int w : beyond) d += D > w;
    const int n = N < 9000 ? 0 : (N < 36000 ? 1 : (N < 110000 ? 2 : (N < 450000 ? 3 : 4)));
    int k = from[dtype == FTK_F32 ? 0 : 1][n][d];
    // fp32 rows that are not whole 16-byte pieces: lines by precision, not by speed.  They were drawn against matrix
    // kernels that read such rows element by element; by pieces those are the faster ones again for few centroids
    // (200000 x 131, K = 32 44 / 74, 60000 x 337, K = 20 47 / 59, 350000 x 27, K = 32 25 / 39), level from 80 or so
    // of long rows (200000 x 131, K = 80 90 / 91), 48 of short ones.  But these calls return distances in
    // direct-difference form, and the matrix kernels' are of the expanded one.
    if (dtype == FTK_F32 && D % 4 != 0) {
        if (D >= 96) k = 8;
        else if (n >= 3) k = d == 0 ? 192 : (d == 2 ? 96 : (N >= 300000 ? 32 : 48));
        else if (n == 2 && d == 3) k = 192;
    }
    return k;
}

static bool scan_pays(ftk_dtype dtype, int64_t N, int D, int K)
{
    if (D < 4 || K < 8) return false;
    // the streaming scan leaves a record per point and 256 centroids: no more than four times the bytes of X
    if (D > 128 && ceil_div(K, 256) * (int64_t)sizeof(ScanRecord) > 4 * (int64_t)D * (dtype == FTK_F32 ? 4 : 8)) return false;
    return K >= scan_from(dtype, N, D);
}

// Where the scan on fp16 pieces runs first.  It has a third of the matrix work, a sample of the rows ahead, a settle pass that measures
// more of each row (fp64: in instructions of half the rate) and some percent of the points in the third pass; four more launches, of
// which two return at once.  Two pieces / one, whole calls, us, blobs, near the line:
//   fp32  D <= 128  65536 x 48, K = 4800 117 / 111; 600000 x 48, K = 544 142 / 128; 65536 x 96, K = 2400 117 / 106; 524288 x 96, K = 512
//                   192 / 165; 300000 x 80, K = 640 143 / 129; 100000 x 72, K = 2100 156 / 131; 800000 x 37, K = 512 168 / 150; 130000 x 40,
//                   K = 2900 132 / 115; 60000 x 128, K = 2000 129 / 122; 450000 x 64, K = 544 132 / 116; 1600000 x 20, K = 512 199 / 168
//         longer    400000 x 160, K = 256 195 / 235; 200000 x 192, K = 330 181 / 166; 65536 x 512, K = 360 138 / 137; 40000 x 512, K = 600
//                   139 / 138; 131072 x 256, K = 512 155 / 146; 33000 x 1024, K = 360 212 / 181; 60000 x 200, K = 1024 132 / 107
//   fp64  D <= 128  600000 x 128, K = 528 451 / 474; 700000 x 96, K = 600 381 / 392; 1000000 x 64, K = 630 365 / 365; 1600000 x 32, K = 800
//                   384 / 362; 500000 x 48, K = 1700 283 / 238; 300000 x 80, K = 1700 305 / 271; 70000 x 128, K = 4500 324 / 271
//         longer    200000 x 130, K = 512 210 / 231; 131072 x 256, K = 360 212 / 211; 40000 x 512, K = 600 193 / 194; 33000 x 1024, K = 360 334 / 277
// Data that the sample refuses pay the sample and the launches that return: 200000 x 32, K = 2400 145 / 163; 130000 x 256, K = 1024
// 300 / 304; fp64 150001 x 128, K = 2085 318 / 347.
static bool half_pays(ftk_dtype dtype, int64_t N, int D, int K)
{
    const double work = (double)N * D * K;
    if (D <= 16 || D > 1024 || N < 32768) return false;
    if (D <= 128) return K >= (dtype == FTK_F32 ? 512 : 640) && N >= 60000 && work >= (dtype == FTK_F32 ? 1.5e10 : 4e10);
    return K >= 320 && work >= (dtype == FTK_F32 || D >= 192 ? 1.2e10 : 3e10);
}

ScanPlan plan_scan(ftk_dtype dtype, int64_t N, int D, int K)
{
    return scan_pays(dtype, N, D, K) ? cut_scan(dtype, N, D, K) : ScanPlan{};
}

// A launch handles points whose records fit SCAN_RECORDS; more points follow in further launches.  Without that the
// records of the streaming scan grow with N K (2^21 x 256, K = 16384: 2.1 GB) and so does its grid, beyond the 2^32
// threads of a launch.  16 thousand workgroups at least stay in a launch.
constexpr int64_t SCAN_RECORDS = (int64_t)1 << 22;  // 64 MB
constexpr int64_t SCAN_BATCH_STEP = 2048;           // points: whole rounds of the streaming scan's XCD order

static ScanPlan cut_launch(ftk_dtype dtype, int64_t N, int D, int K, bool half = false)
{
    ScanPlan p = {};
    p.ok = true;
    p.batch = N;
    p.form = half ? FORM_HALF : (D <= 8 ? FORM_OCTET : (D <= 16 ? FORM_TRIPLE : FORM_PAIR));
    p.stream = D > 128;
    p.tiles = (int)ceil_div(K, 32);
    p.pblocks = ceil_div(N, SC_POINTS);
    if (p.stream && half) {
        p.ct = D <= 512 ? 4 : 2;  // point tiles of a workgroup: 128 KB of fragments at most
        p.nb = (int)ceil_div(D, 16 * sp_ring(p.ct)) * sp_ring(p.ct);
        p.pblocks = ceil_div(N, 32 * p.ct);
        p.tpc = SP_CT;
        p.nch = (int)ceil_div(p.tiles, SP_CT);
        p.cps = p.nch;
        p.splits = 1;
    } else if (p.stream) {
        p.nb = 2 * (int)ceil_div(D, 32);
        // whole chunks of up to eight tiles; smaller ones while the chip is not filled
        int nch = (int)ceil_div(p.tiles, 8);
        const int most = (int)ceil_div(p.tiles, 2);
        while (nch < most && p.pblocks * nch < SCAN_FILL / 2) ++nch;
        p.ct = (int)ceil_div(p.tiles, 2 * nch);
        p.tpc = 2 * p.ct;
        p.nch = (int)ceil_div(p.tiles, p.tpc);
        p.splits = p.nch;
        p.cps = 1;
    } else {
        p.nb = resident_blocks(D);
        const int chunk = p.nb <= 4 ? 16 * 1024 : 32 * 1024;
        int tpc = chunk / (p.nb * form_frags(p.form) * FRAG_UNITS * 16);
        if (tpc > p.tiles) tpc = p.tiles;
        p.tpc = tpc;
        p.nch = (int)ceil_div(p.tiles, tpc);
        // workgroups share a block of points while the chip is not filled
        int splits = (int)ceil_div(SCAN_FILL, p.pblocks);
        if (splits > p.nch) splits = p.nch;
        p.cps = (int)ceil_div(p.nch, splits);
        p.splits = (int)ceil_div(p.nch, p.cps);
    }
    p.tiles_pad = p.nch * p.tpc;
    // 32 points' fragments fit in LDS.  Of longer rows fp64 points go straight to the fp64 matrix instructions, which
    // tell what the scan cannot; those of fp32 can little more on such rows, and refine_kernel takes fewer points
    // better (all centroids in double; uniform data of 7382 x 2419, K = 289: fp64 580 us against 1668 by
    // refine_kernel and 691 by the fp64 matrix kernel, fp32 2000 x 1300, K = 4000 13.5 ms against 0.9).
    p.resolve = p.nb <= 72 || dtype == FTK_F64;
    return p;
}

// the cut of the fp16 form for the points of a launch
static ScanPlan cut_half(const ScanPlan &p, ftk_dtype dtype, int64_t N, int D, int K)
{
    ScanPlan h = cut_launch(dtype, N, D, K, true);
    // the records of a launch are reserved for the other form's split
    if (!p.stream && h.splits > p.splits) {
        h.cps = (int)ceil_div(h.nch, p.splits);
        h.splits = (int)ceil_div(h.nch, h.cps);
    }
    return h;
}

ScanPlan cut_scan(ftk_dtype dtype, int64_t N, int D, int K)
{
    ScanPlan p = cut_launch(dtype, N, D, K);
    const int64_t most = SCAN_RECORDS / p.splits / SCAN_BATCH_STEP * SCAN_BATCH_STEP;
    const int64_t batch_max = most > SCAN_BATCH_STEP ? most : SCAN_BATCH_STEP;
    const int64_t splits = p.splits;
    if (N > batch_max) {  // launches of equal size
        const int64_t n = ceil_div(N, batch_max);
        p = cut_launch(dtype, ceil_div(ceil_div(N, n), SCAN_BATCH_STEP) * SCAN_BATCH_STEP, D, K);
    }
    p.half = p.either = p.form == FORM_PAIR && half_pays(dtype, p.batch, D, K);
    if (p.half) {
        const ScanPlan h = cut_half(p, dtype, p.batch, D, K);
        p.half_nb = h.nb;
        // the preparation writes both images for every tile of its grid, which is padded for the larger chunks
        p.half_tiles = p.stream ? p.tiles + 8 : (h.tiles_pad > p.tiles_pad ? h.tiles_pad : p.tiles_pad);
    }
    // What the points or any part of them may need: fewer points may be shared by more workgroups than the whole,
    // but splits <= SCAN_FILL / pblocks + 1 wherever there is more than the whole's.
    const int64_t fill = (int64_t)SCAN_FILL * SC_POINTS;
    p.rec_reserve = splits * (N < batch_max ? N : batch_max);
    if (p.rec_reserve < fill + (N < fill ? N : fill) + SC_POINTS) p.rec_reserve = fill + (N < fill ? N : fill) + SC_POINTS;
    if (p.rec_reserve > (int64_t)p.tiles * N) p.rec_reserve = (int64_t)p.tiles * N;
    return p;
}

// Tiles that the preparation of a call writes; `last`: the cut of its last launch, whose chunks may be smaller.
static int prepared_tiles(const ScanPlan &p, const ScanPlan &last)
{
    const int tiles = p.tiles_pad > last.tiles_pad ? p.tiles_pad : last.tiles_pad;
    return p.half && tiles < p.half_tiles ? p.half_tiles : tiles;
}

ScanPlan cut_part(const ScanPlan &whole, ftk_dtype dtype, int64_t n, int D, int K)
{
    ScanPlan p = cut_scan(dtype, n, D, K);
    p.half = p.half && whole.half;
    p.either = whole.either;
    return p;
}

static ScanPlan cut_last(const ScanPlan &p, ftk_dtype dtype, int64_t N, int D, int K)
{
    const int64_t rest = N % p.batch;
    return rest ? cut_part(p, dtype, rest, D, K) : p;
}

void scan_padded_rows(ftk_dtype dtype, int64_t N, int D, int K, int64_t *planned, int64_t *reserved)
{
    const ScanPlan whole = cut_scan(dtype, N, D, K);
    const ScanBuffers b = carve_scan((void *)256, whole, N, D);  // (offsets alone)
    const size_t tile = FRAG_UNITS * 16;
    size_t room = ((char *)b.start - (char *)b.image) / ((size_t)whole.nb * form_frags(whole.form) * tile);
    if (whole.half) {
        const size_t h = ((char *)b.half_start - (char *)b.half_image) / ((size_t)whole.half_nb * tile);
        room = h < room ? h : room;
    }
    int most = 0;
    for (int64_t n = N; n >= 1; n /= 2) {  // the points, and batches of them
        const ScanPlan p = cut_part(whole, dtype, n, D, K);
        const int t = prepared_tiles(p, cut_last(p, dtype, n, D, K));
        most = t > most ? t : most;
    }
    *planned = 32 * (int64_t)most;
    *reserved = 32 * (int64_t)room;
}

ScanBuffers carve_scan(void *base, const ScanPlan &p, int64_t N, int D)
{
    ScanBuffers b = {};
    if (!p.ok) return b;
    char *q = (char *)base;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        void *r = q ? (void *)(q + off) : nullptr;
        off += align_up(bytes, 256);
        return r;
    };
    // whole chunks of whatever size a batch is cut into: at most eight tiles (stream), tpc (resident)
    const size_t tiles = p.stream ? (size_t)p.tiles + 8 : (size_t)(p.half && p.half_tiles > p.tiles_pad ? p.half_tiles : p.tiles_pad);
    b.image = (uint4 *)take(tiles * p.nb * form_frags(p.form) * FRAG_UNITS * 16);
    b.start = (float *)take((tiles + 1) * 32 * 4);  // copied two tiles a time
    b.tile_stat = (float4 *)take(tiles * sizeof(float4));
    b.norm = (float *)take(tiles * 32 * 4);
    b.scale = (double *)take(16);
    b.rec = (ScanRecord *)take((size_t)p.rec_reserve * sizeof(ScanRecord));
    b.list_count = (int32_t *)take(((size_t)(p.half ? 2 * SCAN_LISTS : SCAN_LISTS) * LIST_STRIDE + 1) * 4);
    const size_t points = N < SCAN_RECORDS ? N : SCAN_RECORDS;  // of a launch
    b.list = (ScanListed *)take((points + SCAN_LISTS * SETTLE_ROWS_MAX) * sizeof(ScanListed));
    b.tickets = (int32_t *)take((points / 32 + 1) * 4);
    if (p.half) {
        b.half_image = (uint4 *)take((size_t)p.half_tiles * p.half_nb * FRAG_UNITS * 16);
        b.half_start = (float *)take(((size_t)p.half_tiles + 1) * 32 * 4);
        b.ref = take((size_t)D * 8);
        b.sample = (float4 *)take((size_t)p.tiles * sample_shares(p.tiles) * 32 * sizeof(float4));
        b.rest = (ScanListed *)take((points + SCAN_LISTS * SC_POINTS) * sizeof(ScanListed));
    }
    b.bytes = off;
    return b;
}

template <typename T, int NB, int FORM>
static void launch_resident(const ScanArgs &a, const ScanPlan &p, const SettleOwn &own, hipStream_t st)
{
    const dim3 grid((unsigned)(p.pblocks * p.splits)), block(SC_THREADS);
    size_t lds = 2 * ((size_t)p.tpc * NB * form_frags(FORM) * FRAG_UNITS + (size_t)((p.tpc + 1) / 2) * 16) * 16;
    if (own.C && lds < sizeof(OwnShared<T, 2>)) lds = sizeof(OwnShared<T, 2>);  // that of fewest lanes is the largest
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, lds, st, a, own); };
    const bool ragged = a.D % 4 != 0;
    if constexpr (FORM == FORM_PAIR || FORM == FORM_HALF) {
        if (a.gate.refused) {
            if (ragged) launch(scan_resident_kernel<T, NB, FORM, true, true>);
            else launch(scan_resident_kernel<T, NB, FORM, false, true>);
            return;
        }
    }
    if constexpr (FORM != FORM_HALF) {
        if (ragged) launch(scan_resident_kernel<T, NB, FORM, true, false>);
        else launch(scan_resident_kernel<T, NB, FORM, false, false>);
    }
}

template <typename T, int CT>
static void launch_stream(const ScanArgs &a, const ScanPlan &p, hipStream_t st)
{
    const dim3 grid((unsigned)(ceil_div(p.pblocks, 8) * 8 * p.nch)), block(SS_THREADS);
    const size_t lds = 2 * (size_t)(2 * CT + 8) * 4 * FRAG_UNITS * 16;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, lds, st, a); };
    if (a.gate.refused) {
        if (a.D % 4) launch(scan_stream_kernel<T, CT, true, true>);
        else launch(scan_stream_kernel<T, CT, false, true>);
    } else {
        if (a.D % 4) launch(scan_stream_kernel<T, CT, true, false>);
        else launch(scan_stream_kernel<T, CT, false, false>);
    }
}

template <typename T, int PT>
static void launch_points(const ScanArgs &a, const ScanPlan &p, hipStream_t st)
{
    const dim3 grid((unsigned)p.pblocks), block(SP_THREADS);
    const size_t frags = (size_t)p.nb * PT * FRAG_UNITS * 16, records = (size_t)SP_WAVES * 32 * PT * 12;
    const size_t lds = frags > records ? frags : records;
    if (a.D % 4)
        hipLaunchKernelGGL((scan_points_kernel<T, PT, true>), grid, block, lds, st, a, p.nb);
    else
        hipLaunchKernelGGL((scan_points_kernel<T, PT, false>), grid, block, lds, st, a, p.nb);
}

// the scan in form p.form of a call that `a` describes but for the cut
template <typename T>
static void launch_scan_form(ScanArgs a, const ScanPlan &p, const SettleOwn &own, hipStream_t st)
{
    a.tiles = p.tiles;
    a.tpc = p.tpc;
    a.nch = p.nch;
    a.cps = p.cps;
    a.splits = p.splits;
    a.pblocks = (int)p.pblocks;
    if (p.stream) {
        if (p.form == FORM_HALF) {
            if (p.ct == 4) launch_points<T, 4>(a, p, st);
            else launch_points<T, 2>(a, p, st);
            return;
        }
        switch (p.ct) {
        case 1: launch_stream<T, 1>(a, p, st); break;
        case 2: launch_stream<T, 2>(a, p, st); break;
        case 3: launch_stream<T, 3>(a, p, st); break;
        default: launch_stream<T, 4>(a, p, st); break;
        }
    } else if (p.form == FORM_OCTET) {
        launch_resident<T, 1, FORM_OCTET>(a, p, own, st);
    } else if (p.form == FORM_TRIPLE) {
        launch_resident<T, 1, FORM_TRIPLE>(a, p, own, st);
    } else {
#define FTK_LAUNCH_RESIDENT(NB)                                                   \
    case NB:                                                                      \
        if (p.form == FORM_HALF) launch_resident<T, NB, FORM_HALF>(a, p, own, st);     \
        else launch_resident<T, NB, FORM_PAIR>(a, p, own, st);                         \
        break
        switch (p.nb) {
            FTK_LAUNCH_RESIDENT(2);
            FTK_LAUNCH_RESIDENT(3);
            FTK_LAUNCH_RESIDENT(4);
            FTK_LAUNCH_RESIDENT(6);
            FTK_LAUNCH_RESIDENT(8);
        }
#undef FTK_LAUNCH_RESIDENT
    }
}

// L lanes per row in both passes
template <typename T, int L>
static void launch_recheck(const AssignCall &c, const ScanPlan &h, const ScanArgs &a, const RecheckArgs &r, hipStream_t st)
{
    const int64_t groups = ceil_div(c.N, RC_POINTS);
    const dim3 grid((unsigned)(groups < 2048 ? groups : 2048)), block(SC_THREADS);
#define FTK_LAUNCH_RECHECK(NB)                                                                                            \
    case NB:                                                                                                              \
        if (a.D % 4)                                                                                                      \
            hipLaunchKernelGGL((scan_recheck_kernel<T, NB, true, L>), grid, block, 0, st, (const T *)c.X, (const T *)c.C,   \
                               (T *)c.mindist, a, r);                                                                     \
        else                                                                                                              \
            hipLaunchKernelGGL((scan_recheck_kernel<T, NB, false, L>), grid, block, 0, st,  (const T *)c.X,              \
                               (const T *)c.C, (T *)c.mindist, a, r);                                                     \
        break
    if constexpr (L == 4) {
        switch (h.nb) {
            FTK_LAUNCH_RECHECK(2);
        }
    } else {
        switch (h.nb) {
            FTK_LAUNCH_RECHECK(2);
            FTK_LAUNCH_RECHECK(3);
            FTK_LAUNCH_RECHECK(4);
            FTK_LAUNCH_RECHECK(6);
            FTK_LAUNCH_RECHECK(8);
        }
    }
#undef FTK_LAUNCH_RECHECK
}

template <typename T, int L>
static void launch_settle(const AssignCall &c, const ScanPlan &p, const SettleArgs &s, bool own, ResolveArgs r,
                          const ScanBuffers &b, const ScanPlan &ph, const ScanArgs &ah, hipStream_t st)
{
    const int rows = 256 / L * settle_rows(sizeof(T));
    static_assert(256 / L * settle_rows(sizeof(T)) <= SETTLE_ROWS_MAX, "list capacity");
    r.list_cap = s.list_cap;
    const dim3 sg((unsigned)ceil_div(c.N, rows)), sb(256);
    const bool half = L >= 4 && p.half;
    auto settle = [&](auto kernel) { hipLaunchKernelGGL(kernel, sg, sb, 0, st, (const T *)c.X, (const T *)c.C, (T *)c.mindist, s); };
    if (own) {
        // the scan's workgroups have done it
    } else if constexpr (L >= 4) {
        if (half) settle(scan_settle_kernel<T, L, SETTLE_HALF>);
        else if (sizeof(T) == 4 && p.either) settle(scan_settle_kernel<T, L, SETTLE_DOUBLE>);
        else settle(scan_settle_kernel<T, L, SETTLE_PLAIN>);
    } else {
        settle(scan_settle_kernel<T, L, SETTLE_PLAIN>);
    }
    if (!p.resolve) return;
    if (half) {
        r.rest = b.rest;
        r.rest_count = b.list_count + SCAN_LISTS * LIST_STRIDE;
        r.rest_cap = (int)ceil_div(ceil_div(c.N, RC_POINTS), SCAN_LISTS) * RC_POINTS;
    }
    if constexpr (L == 4 || L == 8) {
        if (half) {
            RecheckArgs q = {};
            q.list = b.list;
            q.list_count = b.list_count;
            q.list_cap = s.list_cap;
            q.rest = r.rest;
            q.rest_count = r.rest_count;
            q.rest_cap = r.rest_cap;
            q.K = c.K;
            q.labels = c.labels;
            q.stats = c.stats;
            ScanArgs whole = ah;
            whole.tiles = ph.tiles;
            launch_recheck<T, L>(c, ph, whole, q, st);
        }
    }
    const int64_t groups = ceil_div(c.N, 32);
    // any share of a group among 1 .. splits workgroups divides the grid's work: see the kernel
    const int64_t most = r.nb ? groups * r.splits : c.N;
    const dim3 grid((unsigned)(most < 1024 ? most : 1024)), block(RS_THREADS);
#define FTK_LAUNCH_RESOLVE(F, G)                                                                                     \
    hipLaunchKernelGGL((scan_resolve_kernel<T, F, L, G>), grid, block,                                               \
                       (size_t)r.nb * form_pieces(F) * FRAG_UNITS * 16, st, (const T *)c.X, (const T *)c.C,          \
                       (T *)c.mindist, r)
    if constexpr (L <= 2) {
        if (p.form == FORM_OCTET) FTK_LAUNCH_RESOLVE(FORM_OCTET, false);
        else FTK_LAUNCH_RESOLVE(FORM_TRIPLE, false);
    } else {
        if constexpr (L > 8) {
            if (half) {
                const ResolveArgs own = r;
                r.image = b.half_image;
                r.start = b.half_start;
                r.nb = p.half_nb;
                r.side = 512;
                FTK_LAUNCH_RESOLVE(FORM_HALF, true);
                r = own;
            }
        }
        if (L == 4 && p.form == FORM_TRIPLE) {
            if constexpr (L == 4) FTK_LAUNCH_RESOLVE(FORM_TRIPLE, false);
        } else if (half) {
            FTK_LAUNCH_RESOLVE(FORM_PAIR, true);
        } else {
            FTK_LAUNCH_RESOLVE(FORM_PAIR, false);
        }
    }
#undef FTK_LAUNCH_RESOLVE
}

// Where the workgroups of the scan settle their points themselves: see SettleOwn for where the lines lie.  Of two pieces
// alone in fp32 only the sums in the data's type are built; a part of a call that chooses its form takes those in double.
static bool settles_own(const ScanPlan &p, const ScanPlan &ph, ftk_dtype dtype, int D)
{
    if (D > OWN_D || p.splits != 1 || (!p.half && settle_lanes(D) > 4)) return false;
    return p.half ? ph.splits == 1 : !(dtype == FTK_F32 && p.either);
}

// tiles: those of the image to prepare (0: they are); whole: the problem that c is a part of
template <typename T>
static ftk_status launch_scan_t(const AssignCall &c, const ScanPlan &p, const ScanBuffers &b, const Workspace &w, int tiles,
                                const AssignCall &whole, hipStream_t st)
{
    const int most = centroid_waves(sizeof(T), p.half), waves = p.nb < most ? p.nb : most;
    const dim3 cg((unsigned)(tiles + (p.half ? sample_shares(p.tiles) * p.tiles : 0))), cb((unsigned)(64 * waves));
    // a contiguous list where refine_kernel takes it over
    int32_t *const counts = p.resolve ? b.list_count : w.wl_count;
    const int lists = p.resolve ? SCAN_LISTS : 1;
    // rounding of a score: instructions (1.01: pieces add up to more than the value); 4 u for the start value, the
    // comparison and the bound itself; 2 u for the rounding of the two operands
    const double u = Mma<float>::kEps;
    const double psi = ((p.form == FORM_TRIPLE ? 42.0 : 21.0) * 1.01 * p.nb + 6.0) * u;
    // half of what A comes to for ||x|| = 1 makes the two parts of the bound smallest where ||c|| = 1 as well
    const double lift = 0.5 * ((p.form == FORM_PAIR ? 280.0 : 2.0) * u + psi) + 0.5 * psi;
    // the same for one fp16 piece: what is left of x is at most 2^-11 of it, of c some 0.4 of that; operands below
    // 2^-14 count as that in the rounding of an instruction, and round to within 2^-11 of it
    const double half_psi = (7.0 * 1.01 * p.half_nb + 6.0) * u;
    HalfImage half = {};
    if (p.half) {
        half.rest_count = b.list_count + SCAN_LISTS * LIST_STRIDE;
        half.sample = b.sample;
        half.X = whole.X;
        half.N = whole.N;
        half.tiles = tiles;
        half.shares = sample_shares(p.tiles);
        half.image = b.half_image;
        half.ref = b.ref;
        half.start = b.half_start;
        half.nb = p.half_nb;
        half.lift = (float)(0.5 * (0.8 * 0x1p-11 + half_psi) + 0.5 * half_psi);
        half.tiny = (float)(std::sqrt(16.0 * p.half_nb) * 0x1p-14);
    }
    const size_t ref_bytes = (size_t)(p.half && p.half_nb > p.nb ? p.half_nb : p.nb) * 16 * sizeof(T);
    const bool has_ref = ref_bytes <= REF_BYTES;
    const size_t sums = p.half ? (size_t)waves * 1024 * sizeof(float) : 0;
#define FTK_LAUNCH_CENTROIDS(...)                                                                                     \
    hipLaunchKernelGGL((scan_centroids_kernel<T, __VA_ARGS__>), cg, cb, (has_ref ? ref_bytes : 0) + sums, st, (const T *)c.C, c.D, c.K, p.nb, \
                       b.image, b.start, b.tile_stat, b.scale, counts, lists, (int)has_ref, b.norm, lift, half)
    int32_t *const refused = b.list_count + 2 * SCAN_LISTS * LIST_STRIDE;
    const int zeros = (lists - 1) * LIST_STRIDE + 1 + (p.half ? SCAN_LISTS * LIST_STRIDE : 0);
    if (tiles == 0) FTK_TRY(launch_zero_ints(counts, zeros, st));  // the preparation does that
    else if (p.form == FORM_OCTET) FTK_LAUNCH_CENTROIDS(FORM_OCTET, false);
    else if (p.form == FORM_TRIPLE) FTK_LAUNCH_CENTROIDS(FORM_TRIPLE, false);
    else if (p.half && c.D % 4) FTK_LAUNCH_CENTROIDS(FORM_PAIR, true, true);
    else if (p.half) FTK_LAUNCH_CENTROIDS(FORM_PAIR, true, false);
    else FTK_LAUNCH_CENTROIDS(FORM_PAIR, false);
#undef FTK_LAUNCH_CENTROIDS
    if (tiles && p.half)
        hipLaunchKernelGGL(scan_choose_kernel, dim3(1), dim3(1024), 0, st, b.sample, b.tile_stat, p.tiles, 32 * half.shares,
                           sample_limit(half.shares), refused);
    ScanArgs a = {};
    a.X = c.X;
    a.image = b.image;
    a.start = b.start;
    a.scale = b.scale;
    a.N = c.N;
    a.D = c.D;
    a.rec = b.rec;
    ScanArgs ah = a;  // fp16 pieces
    ah.image = b.half_image;
    ah.start = b.half_start;
    const ScanPlan ph = p.half ? cut_half(p, c.dtype, c.N, c.D, c.K) : ScanPlan{};
    if (p.half) a.gate = ah.gate = ScanGate{refused};
    SettleArgs s = {};
    s.rec = b.rec;
    s.splits = p.splits;
    s.tile_stat = b.tile_stat;
    s.tiles = p.tiles_pad;
    s.scale = b.scale;
    s.N = c.N;
    s.D = c.D;
    s.K = c.K;
    s.psi = (float)psi;
    s.lift = (float)lift;
    s.norm = b.norm;
    s.lost = (float)(p.form == FORM_PAIR ? 128.0 * u : 2.0 * u);  // ||r_x|| <= 2^-17 ||x||; three pieces hold 24 bits
    s.slack = (float)(1.0001 + c.D * u);
    s.ref = b.ref;
    s.tiny = (float)(std::sqrt((double)c.D) * 0x1p-73);  // squares below 2^-149 are lost
    s.labels = c.labels;
    s.tickets = b.tickets;
    s.list = p.resolve ? b.list : nullptr;
    s.wl = w.wl;
    s.list_count = counts;
    s.lists = lists;
    s.gate = a.gate;
    s.half_splits = ph.splits;
    s.half_psi = (float)half_psi;
    s.half_lift = half.lift;
    s.half_tiny = half.tiny;
    ResolveArgs r = {};
    r.gate = a.gate;
    r.image = b.image;
    r.start = b.start;
    r.scale = b.scale;
    r.rec = b.rec;
    r.N = c.N;
    r.D = c.D;
    r.K = c.K;
    r.nb = p.nb <= 72 ? p.nb : 0;
    r.tiles = p.tiles;
    r.splits = r.nb ? (p.splits < 16 ? p.splits : 16) : 1;
    r.side = p.nb > 40 ? 256 : 512;  // the fragments of 32 points: one workgroup per compute unit beyond 80 KB
    r.labels = c.labels;
    r.list = b.list;
    r.list_count = b.list_count;
    r.tickets = b.tickets;
    r.stats = c.stats;
    const int lanes = settle_lanes(c.D);
    // a lane adds up its share, a tree of six the lanes'; 10 u for the differences, their squares and the scale
    s.sums = 0.5f * (float)((c.D / lanes + 4 + 6 + 10) * u);
    SettleOwn own = {};
    if (settles_own(p, ph, c.dtype, c.D)) {
        own.C = c.C;
        own.mindist = c.mindist;
    }
    const int rows = 256 / lanes * (own.C ? own_rows(sizeof(T), lanes) : settle_rows(sizeof(T)));
    s.list_cap = (int)ceil_div(ceil_div(c.N, rows), s.lists) * rows;
    own.s = s;
    if (p.half) launch_scan_form<T>(ah, ph, own, st);
    launch_scan_form<T>(a, p, own, st);
    auto settle = [&](auto l) { launch_settle<T, decltype(l)::value>(c, p, s, own.C != nullptr, r, b, ph, ah, st); };
    switch (lanes) {
    case 2: settle(std::integral_constant<int, 2>{}); break;
    case 4: settle(std::integral_constant<int, 4>{}); break;
    case 8: settle(std::integral_constant<int, 8>{}); break;
    case 16: settle(std::integral_constant<int, 16>{}); break;
    default: settle(std::integral_constant<int, 64>{}); break;
    }
    FTK_TRY_HIP(hipGetLastError());
    return p.resolve ? FTK_OK : launch_refine(c, w, 0, st);
}

ftk_status launch_scan_assign(const AssignCall &c, const ScanPlan &p, const ScanBuffers &b, const Workspace &w,
                              const AssignCall &whole, hipStream_t st)
{
    const size_t esz = c.dtype == FTK_F32 ? 4 : 8;
    const ScanPlan last = cut_last(p, c.dtype, c.N, c.D, c.K);
    int tiles = prepared_tiles(p, last);
    for (int64_t r0 = 0; r0 < c.N; r0 += p.batch) {
        AssignCall part = c;
        part.N = c.N - r0 < p.batch ? c.N - r0 : p.batch;
        part.X = (const char *)c.X + (size_t)r0 * c.D * esz;
        part.labels = c.labels + r0;
        if (c.mindist) part.mindist = (char *)c.mindist + (size_t)r0 * esz;
        const ScanPlan &cut = part.N < p.batch ? last : p;
        FTK_TRY(c.dtype == FTK_F32 ? launch_scan_t<float>(part, cut, b, w, tiles, whole, st)
                                   : launch_scan_t<double>(part, cut, b, w, tiles, whole, st));
        tiles = 0;
    }
    return FTK_OK;
}

}  // namespace ftk
