// Correlation search evaluated through row spectra: the same scores S(d) over the same
// full window and template as the direct sums of register_core.h, for every offset, at a
// cost that no longer grows with the square of the window side.
//
// With the template T = [R, W-R) x [R, H-R) (tw x th), r' = ref - mean_T(ref) and the
// frame f, write b_y(x) = r'(R + x, R + y) for x < tw (0 up to P) and a_r(u) = f(u, r)
// for u < W (0 up to P), P >= W a power of two.  Then
//
//   S(dx, dy) = sum_y sum_x b_y(x) a_{y + R + dy}(x + R + dx)
//             = (1/P) sum_k Z_{R+dy}(k) e^{+2 pi i k (R + dx) / P},
//   Z_j(k)    = sum_y A_{y + j}(k) conj(B_y(k)),
//
// with A_r, B_y the length-P DFTs of the rows (no wrap-around: x + R + dx <= W - 1 < P).
// The rows are real, so only k = 0 .. P/2 is formed (Z at P - k is the conjugate).
// Four steps: row spectra (one P/2-point complex FFT per row of packed real values,
// Stockham radix-16 passes in registers), the contraction Z over template rows (itself by
// transforms along y, block by block), the inverse at the 2R+1 lags needed, and the
// argmax.  The scores carry rounding of order 1e-14 relative to the largest, so the
// offsets are taken from exact direct sums: a +-1 window around the spectral argmax, kept
// when its maximum is not on an inner border of it and its exact peak exceeds every
// spectral score outside the window by more than a bound on the spectral error, and
// otherwise the full direct search for that frame.  The results (integer and sub-pixel
// offsets, peak, flags) are therefore those of the direct search.
#include <algorithm>
#include <string>
#include <type_traits>

#include "common.h"
#include "fftreg.h"
#include "register_core.h"
#include "register_plan.h"

namespace rd {

void register_mean_final(const double *mean_parts, int32_t nparts, double count, double *mean, hipStream_t s);
int32_t register_small_scores(const RegPlan &p, const float *ref, const float *frames, int32_t W, int32_t H, int32_t N,
                              int32_t R, int32_t Rmax, const int32_t *centers, int32_t tx0, int32_t ty0, int32_t tw,
                              int32_t th, const double *mean, double *partial, int32_t skip, hipStream_t s);
void register_scores(const RegPlan &p, const float *ref, const float *frames, int32_t W, int32_t H, int32_t N,
                     int32_t R, int32_t Rmax, const int32_t *centers, const int32_t *map, int32_t tx0, int32_t ty0,
                     int32_t tw, int32_t th, const double *mean, double *partial, double *sc, reduce_offset_t *out,
                     hipStream_t s, const WindowMove &mv);

constexpr int FFT_THREADS = 256;
constexpr int32_t FFT_P_MAX = 8192;    // longest rows: P/2 = 4096 complex values in LDS (64 KB)
constexpr int COL_L = 256;             // rows per block of the contraction (transform length along y)
constexpr int COL_KC = 16;             // spectrum columns per contraction workgroup
constexpr int COL_LAGS = 144;          // most lags per pass: a block then adds at least 113 template rows
constexpr size_t FFT_FALLBACK_BYTES = size_t(256) << 20;

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// two roundings per component
__device__ __forceinline__ double2 cmulf(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}

// The first n_parts workgroups: the sums of the template's mean (register_mean's parts); the
// others: tw[t] = exp(-2 pi i t / P), t in [0, P).
__global__ __launch_bounds__(MEAN_THREADS) void spec_prepare(const float *__restrict__ ref, int32_t W, int32_t tx0,
                                                             int32_t ty0, int32_t tw_, int32_t th, int32_t n_parts,
                                                             double *__restrict__ part, double2 *__restrict__ tw,
                                                             int32_t P)
{
    __shared__ double scratch[MEAN_THREADS / 64];
    if ((int32_t)blockIdx.x < n_parts) {
        const double s = tmpl_part_sum(ref, W, tx0, ty0, tw_, th, blockIdx.x, scratch);
        if (threadIdx.x == 0) part[blockIdx.x] = s;
        return;
    }
    const int32_t t = (blockIdx.x - n_parts) * MEAN_THREADS + threadIdx.x;
    if (t >= P) return;
    double s, c;
    sincospi(-2.0 * (double)t / (double)P, &s, &c);
    tw[t] = make_double2(c, s);
}

// 4-point transform of v[0], v[S], v[2 S], v[3 S] in place (INV: conjugate kernel)
template <bool INV, int S>
__device__ __forceinline__ void dft4(double2 *v)
{
    const double2 a = cadd(v[0], v[2 * S]), b = csub(v[0], v[2 * S]);
    const double2 c = cadd(v[S], v[3 * S]), d = csub(v[S], v[3 * S]);
    const double2 e = INV ? make_double2(-d.y, d.x) : make_double2(d.y, -d.x);  // -+ i d
    v[0] = cadd(a, c);
    v[S] = cadd(b, e);
    v[2 * S] = csub(a, c);
    v[3 * S] = csub(b, e);
}

// W16^e for the exponents that the register transforms need
__device__ __forceinline__ double2 w16(int e)
{
    constexpr double C = 0.92387953251128675613, Sn = 0.38268343236508977173, H = 0.70710678118654752440;
    constexpr double wr[10] = {1, C, H, Sn, 0, -Sn, -H, -C, -1, -C}, wi[10] = {0, -Sn, -H, -C, -1, -C, -H, -Sn, 0, Sn};
    return make_double2(wr[e], wi[e]);
}

// 2-, 4- or 8-point transform of v[0], v[S], ..., v[(X - 1) S] in place, natural order
template <int X, int S>
__device__ __forceinline__ void dft_small(double2 *v)
{
    if constexpr (X == 2) {
        const double2 a = v[0];
        v[0] = cadd(a, v[S]);
        v[S] = csub(a, v[S]);
    } else if constexpr (X == 4) {
        dft4<false, S>(v);
    } else {
        static_assert(X == 8, "radix");
        constexpr double H = 0.70710678118654752440;
        dft4<false, 2 * S>(v);          // even inputs: terms k at v[2 k S]
        dft4<false, 2 * S>(v + S);      // odd inputs
        double2 e[4], o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            e[k] = v[2 * k * S];
            o[k] = v[(2 * k + 1) * S];
        }
        o[1] = make_double2(H * (o[1].x + o[1].y), H * (o[1].y - o[1].x));   // W8
        o[2] = make_double2(o[2].y, -o[2].x);                                // -i
        o[3] = make_double2(H * (o[3].y - o[3].x), -H * (o[3].x + o[3].y));  // W8^3
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k * S] = cadd(e[k], o[k]);
            v[(k + 4) * S] = csub(e[k], o[k]);
        }
    }
}

// 16-point transform in registers, natural order in and out
template <bool INV>
__device__ __forceinline__ void dft16(double2 (&v)[16])
{
    constexpr double H = 0.70710678118654752440;
#pragma unroll
    for (int i = 0; i < 4; ++i) dft4<INV, 4>(v + i);  // v[i + 4 k] = term k of the inputs i, i + 4, ...
    // W16^(i k)
#pragma unroll
    for (int i = 1; i < 4; ++i)
#pragma unroll
        for (int k = 1; k < 4; ++k) {
            const int e = i * k;
            double2 &z = v[i + 4 * k];
            if (e == 4)
                z = INV ? make_double2(-z.y, z.x) : make_double2(z.y, -z.x);
            else if (e == 2)
                z = INV ? make_double2(H * (z.x - z.y), H * (z.x + z.y)) : make_double2(H * (z.x + z.y), H * (z.y - z.x));
            else if (e == 6)
                z = INV ? make_double2(-H * (z.x + z.y), H * (z.x - z.y))
                        : make_double2(H * (z.y - z.x), -H * (z.x + z.y));
            else
                z = cmulf(z, make_double2(w16(e).x, INV ? -w16(e).y : w16(e).y));
        }
#pragma unroll
    for (int k = 0; k < 4; ++k) dft4<INV, 1>(v + 4 * k);  // v[4 k + m] = output k + 4 m
    // output c = k + 4 m sits in v[4 k + m]: transpose the 4 x 4
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int m = k + 1; m < 4; ++m) {
            const double2 x = v[4 * k + m];
            v[4 * k + m] = v[4 * m + k];
            v[4 * m + k] = x;
        }
}

// ---- row spectra -------------------------------------------------------------------------
// Rows of batch b: row r (r < nrows) holds x(u) = base[(b + (b >= skip)) * batch + r * pitch + u] - sub for
// u < ncols, 0 for ncols <= u < P; rows nrows <= r < rows_out are zero.  Output: the
// half spectrum X(k), k = 0 .. P/2, at spec + b * spec_batch + r * PS, and the sum of
// squares of each row at rowsq[b * rows_out + r].  A row of P real values is packed as
// z(n) = x(2n) + i x(2n+1), transformed over N2 = P/2 points, and unpacked:
//   X(k) = E(k) - i w^k O(k),  E = (Z(k) + conj Z(N2-k)) / 2,  O = (Z(k) - conj Z(N2-k)) / 2,
// w = exp(-2 pi i / P).
//
// A thread holds 16 of a row's values, so a row takes N2 / 16 threads and a workgroup of
// 256 takes 4096 / N2 rows.  Stockham passes of radix 16 in registers: the first takes the
// values as they are loaded, so N2 points pass through LDS twice (16 x 16 x N2/256; once for
// N2 <= 256) and a third time for the partners of the unpacking.  Radix-4 passes moved a row
// of 4096 through LDS seven times and read 18 thousand twiddles for it, which bound the
// kernel at half the copy rate (3.45 ms for 16 frames of 6144x6160 and their template, 9.4 GB
// moved, now 2.02, at the copy rate); here the
// second pass's twiddles come from a table of 256 in LDS, the last one's are products of
// four table values.  LDS index i sits at i + i / 16: a
// pass's stores are 16 values apart from lane to lane, which would fall on one bank.
struct RowSrc {
    const float *base;
    int64_t batch, pitch;
    int32_t ncols, nrows;
    const double *sub;  // device scalar subtracted from every value, or NULL
    int32_t skip;       // batch b reads from b + 1 on from this one
};

constexpr int FFT_V = 16;                                   // values per thread
constexpr int FFT_POINTS = FFT_V * FFT_THREADS;             // complex values per workgroup
constexpr int FFT_LDS = FFT_POINTS + FFT_POINTS / 16;       // padded
static_assert(FFT_P_MAX / 2 <= FFT_POINTS, "a row fits one workgroup");

template <int LOG2N2>
__global__ __launch_bounds__(FFT_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void fft_rows(
    RowSrc src, int32_t rows_out, const double2 *__restrict__ tw, double2 *__restrict__ spec, int64_t spec_batch,
    int32_t PS, double *__restrict__ rowsq)
{
    constexpr int32_t N2 = 1 << LOG2N2, P = 2 * N2;
    constexpr int tpr = N2 / FFT_V;                  // threads per row
    constexpr int rpw = FFT_THREADS / tpr;           // rows per workgroup
    constexpr int XL = N2 >= 256 ? N2 / 256 : N2 / 16;  // radix of the last pass (1: none)
    static_assert(N2 >= 32, "rows of at least 64 values");
    __shared__ double2 zl[FFT_LDS], w256[256];
    const int t = threadIdx.x, lr = t / tpr, lt = t - lr * tpr;
    const int32_t b = blockIdx.y;
    const int32_t r = blockIdx.x * rpw + lr;
    double2 *z = zl + lr * (N2 + N2 / 16);
    const bool live = r < rows_out;
    const bool data = r < src.nrows;
    const double sub = src.sub ? *src.sub : 0.0;
    const float *row = src.base + (int64_t)(b + (b >= src.skip)) * src.batch + (int64_t)(data ? r : 0) * src.pitch;

    // packed load: value pair n = lt + i tpr, as one 8-byte load where the row allows it
    // (addresses clamped into the row, values past it replaced by zero)
    float f0[FFT_V], f1[FFT_V];
    const int32_t last = src.ncols - 1;
    if ((reinterpret_cast<uintptr_t>(row) & 7u) == 0 && src.ncols >= 2) {
        const int32_t lastp = (src.ncols >> 1) - 1;
#pragma unroll
        for (int i = 0; i < FFT_V; ++i) {
            const float2 v = reinterpret_cast<const float2 *>(row)[min(lt + i * tpr, lastp)];
            f0[i] = v.x;
            f1[i] = v.y;
        }
        if (src.ncols & 1) {  // the odd last value has no pair
            const float v = row[last];
#pragma unroll
            for (int i = 0; i < FFT_V; ++i)
                if (2 * (lt + i * tpr) == last) f0[i] = v;
        }
    } else {
#pragma unroll
        for (int i = 0; i < FFT_V; ++i) {
            const int32_t u = 2 * (lt + i * tpr);
            f0[i] = row[min(u, last)];
            f1[i] = row[min(u + 1, last)];
        }
    }
    if constexpr (N2 >= 256) w256[t] = tw[t * (P / 256)];
    double2 v[FFT_V];
    double sq = 0.0;
#pragma unroll
    for (int i = 0; i < FFT_V; ++i) {
        const int32_t u = 2 * (lt + i * tpr);
        const double x0 = (data && u < src.ncols) ? (double)f0[i] - sub : 0.0;
        const double x1 = (data && u + 1 < src.ncols) ? (double)f1[i] - sub : 0.0;
        sq = fma(x0, x0, sq);
        sq = fma(x1, x1, sq);
        v[i] = make_double2(x0, x1);
    }
    // the row's sum of squares: over the row's lanes of a wave, then over its waves in order
    {
        __shared__ double part[FFT_THREADS / 64];
#pragma unroll
        for (int off = (tpr < 64 ? tpr : 64) / 2; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
        if constexpr (tpr > 64) {
            if ((t & 63) == 0) part[t >> 6] = sq;
            __syncthreads();
            if (lt == 0) {
                sq = 0.0;
                for (int i = 0; i < tpr / 64; ++i) sq += part[t / 64 + i];
            }
        }
        if (lt == 0 && live) rowsq[(int64_t)b * rows_out + r] = sq;
    }

    // pass L = 1: butterfly j = lt, output q at 16 j + q
    dft16<false>(v);
#pragma unroll
    for (int q = 0; q < FFT_V; ++q) z[17 * lt + q] = v[q];
    __syncthreads();
    // every later pass reads its values at lt + i tpr
    const double2 *zr = z + lt;
    auto at = [&](int i) { return zr[((lt + i * tpr) >> 4) + i * tpr]; };
    if constexpr (N2 >= 256) {
        // pass L = 16: output q at (j - k) 16 + k + 16 q, k = j mod 16, twiddles W256^(q k)
        const int k = lt & 15;
#pragma unroll
        for (int q = 0; q < FFT_V; ++q) v[q] = q == 0 ? at(q) : cmulf(at(q), w256[q * k]);
        dft16<false>(v);
        __syncthreads();
        if constexpr (XL > 1) {
            double2 *zo = z + (lt - k) * 17 + k;
#pragma unroll
            for (int q = 0; q < FFT_V; ++q) zo[17 * q] = v[q];
            __syncthreads();
        }
    }
    if constexpr (XL > 1) {
        // last pass, radix XL: butterflies j = lt + c tpr, inputs q at value c + q (16 / XL),
        // twiddles W_N2^(q j) from W^j, W^2j, W^4j, W^8j; outputs where the inputs were
        constexpr int C = FFT_V / XL;
#pragma unroll
        for (int i = 0; i < FFT_V; ++i) v[i] = at(i);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int32_t j2 = 2 * (lt + c * tpr);  // W_N2^e = tw[2 e]
            double2 w[XL];
#pragma unroll
            for (int q = 1; q < XL; ++q) {
                const int hi = 1 << (31 - __builtin_clz(q));
                w[q] = q == hi ? tw[q * j2] : cmulf(w[hi], w[q - hi]);
            }
#pragma unroll
            for (int q = 1; q < XL; ++q) v[c + q * C] = cmulf(v[c + q * C], w[q]);
            if constexpr (XL == 16)
                dft16<false>(v);
            else
                dft_small<XL, C>(v + c);
        }
    }
    // unpack the two real transforms into the half spectrum of the row: v[i] = Z(lt + i tpr)
#pragma unroll
    for (int i = 0; i < FFT_V; ++i) z[lt + i * tpr + ((lt + i * tpr) >> 4)] = v[i];
    __syncthreads();
    if (live) {
        double2 *out = spec + (int64_t)b * spec_batch + (int64_t)r * PS;
#pragma unroll
        for (int i = 0; i < FFT_V; ++i) {
            const int32_t k = lt + i * tpr, kc = (N2 - k) & (N2 - 1);
            const double2 zk = v[i], zc = z[kc + (kc >> 4)];
            const double2 e = make_double2(0.5 * (zk.x + zc.x), 0.5 * (zk.y - zc.y));
            const double2 o = make_double2(0.5 * (zk.x - zc.x), 0.5 * (zk.y + zc.y));
            const double2 wo = cmulf(tw[k], o);
            out[k] = make_double2(e.x + wo.y, e.y - wo.x);  // E - i w O
        }
        if (lt == 0) out[N2] = make_double2(v[0].x - v[0].y, 0.0);
    }
}

// ---- contraction over template rows -------------------------------------------------------
// Z_j(k) = sum_y A_{y + j}(k) conj(B_y(k)) is a correlation along y for every column k.  The
// template rows go in blocks of M = COL_L - Dg + 1 rows, Dg the lags of a pass: block b
// correlates its M template rows (zero up to COL_L) with the COL_L frame rows from its
// first one on, and the lags j < Dg of that do not wrap around, so with transforms of
// length COL_L along y
//   Z_j = IDFT_j( sum_b DFT(A block b)(q) conj(DFT(B block b)(q)) ).
// The sum over blocks stays in the transform domain: one inverse per workgroup, and COL_L /
// M times one transform per frame value instead of Dg multiply-adds (direct sums over the
// lags in registers took 11.8 of the 21.8 ms of a call over 16 frames of 6144x6160 at R = 65,
// bound by FP64 issue; the blocks take 2.58 and the template's 0.21, and for six stacks of 91
// frames of 512x512 to 4096x4096 at R = 17 0.80 and 0.10 ms instead of 2.15).  Windows of more
// than COL_LAGS lags take several passes of equal width, pass g on the frame rows g Dg
// further down.
//
// The template's block transforms are made once (spec_tmpl) and read by every frame.  A
// workgroup takes COL_KC columns (256-byte row pieces) and a band of blocks of one frame; a
// thread holds 16 of the 256 values of its column, n = 16 a + r: a transform is a
// 16-point one in registers, the twiddle W^(r c), an exchange over LDS, and a second
// 16-point one, after which the thread holds q = r + 16 d.  The sums over blocks stay in 16
// registers pairs in that order, in which the template transforms are stored, and feed the
// inverse as they are.  Bound by the reads of the spectra: workgroups of the same columns
// and blocks but other frames run together on one XCD, so that the template's transforms
// come from its L2.
constexpr int COL_T = 256;  // threads: COL_KC columns x 16
static_assert(COL_L == 256 && COL_KC == 16, "16 values per thread, twice");

struct ColArgs {
    const double2 *A;  // frame spectra: frame f at A + f * a_batch, row r < H at + r * PS
    double2 *Bt;       // template block transforms [n_blk][n_kt][16][COL_T]
    double2 *Zp;       // [F][n_band][D][PS]
    int64_t a_batch;
    int32_t PS, D, Dg, n_grp, M, H, n_blk, n_band, bpb, n_kt, nf;  // bpb: blocks per band
};

// First half of the 256-point transform of a column: thread r of 16 holds n = 16 a + r in
// v[a]; afterwards z holds the values for the second half, which reads z[r][b][col] and
// applies dft16.  wl[e] = W256^e.
template <bool INV>
__device__ __forceinline__ void col_first_half(double2 (&v)[16], double2 *z, const double2 *wl, int r, int col)
{
    dft16<INV>(v);
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        double2 w = wl[r * c];
        if (INV) w.y = -w.y;
        z[(c * 16 + r) * COL_KC + col] = c == 0 ? v[c] : cmulf(v[c], w);
    }
}

__device__ __forceinline__ void col_second_read(double2 (&v)[16], const double2 *z, int r, int col)
{
#pragma unroll
    for (int b = 0; b < 16; ++b) v[b] = z[(r * 16 + b) * COL_KC + col];
}

__device__ __forceinline__ void col_table(double2 *wl)
{
    double s, c;
    sincospi(-(double)threadIdx.x / (COL_L / 2), &s, &c);
    wl[threadIdx.x] = make_double2(c, s);
}

// Transforms of the template's blocks: workgroup (column tile, block); B holds the row
// spectra of the th template rows.
__global__ __launch_bounds__(COL_T) __attribute__((amdgpu_waves_per_eu(2, 2))) void spec_tmpl(
    ColArgs a, const double2 *__restrict__ B, int32_t th)
{
    __shared__ double2 z[COL_L * COL_KC], wl[COL_L];
    const int t = threadIdx.x, col = t & (COL_KC - 1), r = t / COL_KC;
    const int32_t kt = blockIdx.x, blk = blockIdx.y;
    col_table(wl);
    __syncthreads();
    const int32_t y0 = blk * a.M, ny = min(a.M, th - y0);
    const double2 *src = B + (int64_t)y0 * a.PS + kt * COL_KC + col;
    double2 v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int32_t y = 16 * i + r;
        v[i] = src[(int64_t)min(y, ny - 1) * a.PS];
        if (y >= ny) v[i] = make_double2(0.0, 0.0);
    }
    col_first_half<false>(v, z, wl, r, col);
    __syncthreads();
    col_second_read(v, z, r, col);
    dft16<false>(v);
    double2 *out = a.Bt + ((int64_t)blk * a.n_kt + kt) * (16 * COL_T) + t;
#pragma unroll
    for (int d = 0; d < 16; ++d) out[d * COL_T] = v[d];
}

__global__ __launch_bounds__(COL_T) __attribute__((amdgpu_waves_per_eu(2, 2))) void spec_cols(ColArgs a)
{
    __shared__ double2 z[COL_L * COL_KC], wl[COL_L];
    const int t = threadIdx.x, col = t & (COL_KC - 1), r = t / COL_KC;
    // frame fastest, then lag pass, band, column tile
    int32_t id = xcd_logical_id((int32_t)blockIdx.x, (int32_t)gridDim.x);
    const int32_t f = id % a.nf;
    id /= a.nf;
    const int32_t g = id % a.n_grp;
    id /= a.n_grp;
    const int32_t band = id % a.n_band, kt = id / a.n_band;
    col_table(wl);
    __syncthreads();
    const double2 *A = a.A + (int64_t)f * a.a_batch + kt * COL_KC + col;
    double2 acc[16];
#pragma unroll
    for (int d = 0; d < 16; ++d) acc[d] = make_double2(0.0, 0.0);
    const int32_t b1 = min((band + 1) * a.bpb, a.n_blk);
    for (int32_t blk = band * a.bpb; blk < b1; ++blk) {
        const int32_t y0 = blk * a.M + g * a.Dg;
        double2 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = A[(int64_t)min(y0 + 16 * i + r, a.H - 1) * a.PS];
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (y0 + 16 * i + r >= a.H) v[i] = make_double2(0.0, 0.0);  // rows past the frame
        col_first_half<false>(v, z, wl, r, col);
        // the template's transform is on its way while the exchange is waited for
        const double2 *bt = a.Bt + ((int64_t)blk * a.n_kt + kt) * (16 * COL_T) + t;
        double2 b[16];
#pragma unroll
        for (int d = 0; d < 16; ++d) b[d] = bt[d * COL_T];
        __syncthreads();
        col_second_read(v, z, r, col);
        __syncthreads();  // before the next block's first half
        dft16<false>(v);
#pragma unroll
        for (int d = 0; d < 16; ++d) {  // acc += v conj(b)
            acc[d].x = fma(v[d].x, b[d].x, acc[d].x);
            acc[d].x = fma(v[d].y, b[d].y, acc[d].x);
            acc[d].y = fma(v[d].y, b[d].x, acc[d].y);
            acc[d].y = fma(-v[d].x, b[d].y, acc[d].y);
        }
    }
    // inverse: the sums are q = r + 16 d in acc[d], the order its first half takes
    col_first_half<true>(acc, z, wl, r, col);
    __syncthreads();
    col_second_read(acc, z, r, col);
    dft16<true>(acc);
    double2 *zp = a.Zp + ((int64_t)f * a.n_band + band) * a.D * a.PS + kt * COL_KC + col;
#pragma unroll
    for (int d = 0; d < 16; ++d) {
        const int32_t i = r + 16 * d, j = g * a.Dg + i;
        if (i < a.Dg && j < a.D)
            zp[(int64_t)j * a.PS] = make_double2(acc[d].x * (1.0 / COL_L), acc[d].y * (1.0 / COL_L));
    }
}

// ---- scores at the lags of the window --------------------------------------------------
// S[f][j][m] = (1/P) sum_{k=0}^{N2} c_k Re(Z_j(k) e^{+2 pi i k m / P}), c_k = 1 at k = 0 and
// k = N2, else 2; Z_j(k) the sum of the partials over bands in order.  Only D of the P lags m
// are asked for, so the sum is split by residues, k = a + A b with A = P / COL_L:
//   sum_a e^{2 pi i a m / P} sum_b z(a + A b) e^{2 pi i b m / COL_L},
// the inner sums 256-point transforms (as in the contraction, sixteen at a time, of which
// half the inputs are zero) that give 256 consecutive lags, the outer one A products per lag.  A
// workgroup takes one lag j (or, for A < 16, 16 / A of them) of a frame and, by blockIdx.z,
// one of the ranges of 256 lags m.  Bound by the reads of the partials; with D products per k
// and a recurrence for the twiddles, 131 lags of 15 frames at P = 8192 took 698 us, now 86, and
// 35 lags of 85 frames at P = 512 to 4096 in six calls 202, now 66.
template <int LOG2N2>
__global__ __launch_bounds__(COL_T) __attribute__((amdgpu_waves_per_eu(2, 2))) void spec_eval(
    const double2 *__restrict__ Zp, int32_t n_part, int32_t D, int32_t PS, const double2 *__restrict__ tw,
    double *__restrict__ S)
{
    constexpr int32_t N2 = 1 << LOG2N2, P = 2 * N2, A = P > COL_L ? P / COL_L : 1;
    constexpr int SP = COL_L > P ? COL_L / P : 1;  // shorter spectra: every SP-th input
    constexpr int AC = A < COL_KC ? A : COL_KC;  // residues per pass
    static_assert(A % AC == 0, "whole passes");
    __shared__ double2 z[COL_L * COL_KC], wl[COL_L];
    const int t = threadIdx.x, col = t & (COL_KC - 1), r = t / COL_KC;
    const int a0 = col % AC;
    const int32_t j = blockIdx.x * (COL_KC / AC) + col / AC, f = blockIdx.y, m0 = blockIdx.z * COL_L;
    const double2 *z0 = Zp + (int64_t)f * n_part * D * PS + (int64_t)min(j, D - 1) * PS;
    const int64_t pstride = (int64_t)D * PS;
    col_table(wl);
    double acc[16];
#pragma unroll
    for (int d = 0; d < 16; ++d) acc[d] = 0.0;
    for (int32_t a = a0; a < A; a += AC) {
        // inputs b = 16 i + r, zero above N2: b = 128 is k = N2 for the residue 0
        double2 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = make_double2(0.0, 0.0);
        for (int32_t p = 0; p < n_part; ++p) {
            double2 u[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                u[i] = z0[p * pstride + a + A * ((16 * i + r) / SP)];
                if (SP > 1 && r % SP != 0) u[i] = make_double2(0.0, 0.0);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = cadd(v[i], u[i]);
            if (a == 0 && r == 0) v[8] = cadd(v[8], z0[p * pstride + N2]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const double c = a == 0 && i == 0 && r == 0 ? 1.0 : 2.0;
            v[i] = make_double2(c * v[i].x, c * v[i].y);
        }
        __syncthreads();  // the table is written; the last pass's second halves have read z
        col_first_half<true>(v, z, wl, r, col);
        __syncthreads();
        col_second_read(v, z, r, col);
        dft16<true>(v);
#pragma unroll
        for (int d = 0; d < 16; ++d) {
            const double2 w = tw[(int32_t)((int64_t)a * (m0 + r + 16 * d)) & (P - 1)];
            acc[d] = fma(v[d].x, w.x, acc[d]);  // Re(v conj(w))
            acc[d] = fma(v[d].y, w.y, acc[d]);
        }
    }
#pragma unroll
    for (int d = 0; d < 16; ++d) {
        double v = acc[d];
#pragma unroll
        for (int off = AC / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        const int32_t m = m0 + r + 16 * d;
        if (a0 == 0 && j < D && m < D) S[((int64_t)f * D + j) * D + m] = v / (double)P;
    }
}

// Argmax of the spectral scores (full window, centre 0): the window centre of the exact
// refinement.  Equal scores go to the smaller index, as in pick_frame.
constexpr int PICK_THREADS = 1024;

__global__ __launch_bounds__(PICK_THREADS) void spec_pick(const double *__restrict__ S, int32_t D, int32_t R,
                                                          int32_t *__restrict__ centres)
{
    __shared__ Best scratch[PICK_THREADS / 64];
    const int32_t f = blockIdx.x, n = D * D;
    const double *Sf = S + (int64_t)f * n;
    Best b{-INFINITY, 0x7fffffff};
    for (int32_t c0 = threadIdx.x; c0 < n; c0 += 4 * PICK_THREADS) {
        double v[4];  // loaded together
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = Sf[min(c0 + u * PICK_THREADS, n - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) b = better_of(b, Best{v[u], min(c0 + u * PICK_THREADS, n - 1)});
    }
    b = block_best(b, scratch);
    if (threadIdx.x == 0) {
        const int32_t i = b.i < n ? b.i : 0;  // no score above -inf (NaN): any window, the bound settles nothing
        centres[2 * f] = i % D - R;
        centres[2 * f + 1] = i / D - R;
    }
}

// Decision per frame, one workgroup each.  Kept: the exact maximum is not on an inner
// border, and it exceeds the best spectral score outside its +-1 window by more than the
// bound on the spectral error
//   bound = factor ||a||_F ||b||_F,  factor = 4 eps (10 log2(P/2) + c (124 + n_blk) + P + 50),
// (eps = 2^-53; ||a||_F over the frame rows, ||b||_F over the template rows; first-order
// rounding of the row transforms, the contraction, and, with room, the inverse sums: 5 eps per
// radix-2 level, 3 for the outer twiddle and A additions).
// The contraction's term: 5 eps per radix-2 level, 8 levels, of the transforms of a frame
// block, of a template block and back, 4 eps for a product and n_blk additions, against
// sum_b ||A_b|| ||B_b|| <= c ||a|| ||b||, c = ceil(COL_L / M) the blocks a frame row is in.  A kept frame
// gets second = the larger of its window's runner-up and that spectral score, the margin
// and NEAR_TIE from it, and loses CLIPPED (its window is a step of the full search).
// fb[k] = the frame of slot k if it takes the full search, else -1 (that search's slots);
// info[k] says why (1: inner border, 2: not clear of the bound).
// The exact scores of the window come as the tile partials of score_small<3>.
__global__ __launch_bounds__(PICK_THREADS) void spec_settle(const double *__restrict__ partial, int32_t n_tiles,
                                                            const int32_t *__restrict__ centres,
                                                            const double *__restrict__ S, int32_t D, int32_t R,
                                                            const double *__restrict__ rowsq_a, int32_t rows_a,
                                                            const double *__restrict__ rowsq_b, int32_t rows_b,
                                                            double factor, int32_t skip,
                                                            reduce_offset_t *__restrict__ offs,
                                                            int32_t *__restrict__ fb, int32_t *__restrict__ info)
{
    constexpr int NW = PICK_THREADS / 64;
    __shared__ double red[NW][9];
    __shared__ double win[9];
    __shared__ Best scratch[NW];
    __shared__ reduce_offset_t o_sh;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int32_t k = blockIdx.x;
    const int32_t cx = centres[2 * k], cy = centres[2 * k + 1];
    // the 3 x 3 exact scores: threads stride over tiles, lanes by a fixed butterfly, waves in order
    {
        double s[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) s[q] = 0.0;
        const double *pk = partial + (int64_t)k * n_tiles * 9;
        for (int32_t i = t; i < n_tiles; i += PICK_THREADS)
#pragma unroll
            for (int q = 0; q < 9; ++q) s[q] += pk[(int64_t)i * 9 + q];
#pragma unroll
        for (int q = 0; q < 9; ++q) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s[q] += __shfl_xor(s[q], off, 64);
            if (lane == q) red[wv][q] = s[q];
        }
        __syncthreads();
        if (t < 9) {
            double v = 0.0;
            for (int w = 0; w < NW; ++w) v += red[w][t];
            const int32_t dx = cx - 1 + t % 3, dy = cy - 1 + t / 3;
            win[t] = dx >= -R && dx <= R && dy >= -R && dy <= R ? v : -INFINITY;
        }
        __syncthreads();
        pick_frame(win, 3, 1, R, cx, cy, &o_sh, scratch);
        __syncthreads();
    }
    const reduce_offset_t o0 = o_sh;
    // over the workgroup: lanes by a fixed butterfly, then the waves in order
    auto block_sum = [&](const double *v, int32_t n) {
        double s = 0.0;
        for (int32_t r = t; r < n; r += PICK_THREADS) s += v[r];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        __syncthreads();
        if (lane == 0) red[wv][0] = s;
        __syncthreads();
        double tot = 0.0;
        for (int w = 0; w < NW; ++w) tot += red[w][0];
        return tot;
    };
    const double aa = block_sum(rowsq_a + (int64_t)k * rows_a, rows_a);
    const double bb = block_sum(rowsq_b, rows_b);
    // best spectral score outside the +-1 window around the exact maximum
    const double *Sk = S + (int64_t)k * D * D;
    double best = -INFINITY;
    for (int32_t c0 = t; c0 < D * D; c0 += 4 * PICK_THREADS) {
        double v[4];  // loaded together
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = Sk[min(c0 + u * PICK_THREADS, D * D - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t c = min(c0 + u * PICK_THREADS, D * D - 1);
            const int32_t jj = c / D, ii = c - jj * D;
            if (abs(ii - R - o0.dx) > 1 || abs(jj - R - o0.dy) > 1) best = fmax(best, v[u]);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) best = fmax(best, __shfl_xor(best, off, 64));
    __syncthreads();
    if (lane == 0) red[wv][0] = best;
    __syncthreads();
    if (t != 0) return;
    double out_best = red[0][0];
    for (int w = 1; w < NW; ++w) out_best = fmax(out_best, red[w][0]);
    const double bound = factor * sqrt(aa) * sqrt(bb);
    reduce_offset_t o = o0;
    const bool border = ((o.flags & REDUCE_EDGE_X) && o.dx > -R && o.dx < R) ||
                        ((o.flags & REDUCE_EDGE_Y) && o.dy > -R && o.dy < R);
    const bool unsure = !(o.peak > out_best + bound);
    const int32_t kf = k + (k >= skip ? 1 : 0);  // the slot's frame
    fb[k] = border || unsure ? kf : -1;
    info[kf] = (border ? 1 : 0) | (unsure ? 2 : 0);
    if (!border && !unsure) {
        o.second = fmax(o.second, out_best);
        if (o.second == -INFINITY) o.margin = INFINITY;
        else if (o.peak == 0.0) o.margin = (o.peak > o.second) ? INFINITY : 0.0;
        else o.margin = (o.peak - o.second) / fabs(o.peak);
        o.flags &= ~(REDUCE_CLIPPED | REDUCE_NEAR_TIE);
        if (o.margin < REDUCE_NEAR_TIE_MARGIN) o.flags |= REDUCE_NEAR_TIE;
        offs[kf] = o;
    }
}

// ---- host side ---------------------------------------------------------------------------
static size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

bool fft_layout(int32_t W, int32_t H, int32_t N, int32_t R, size_t round_bytes, FftLayout *L)
{
    if (W < 1 || H < 1 || N < 1 || N > 65535 || R < 1 || W - 2 * R < 1 || H - 2 * R < 1 || W > FFT_P_MAX ||
        2 * R + 1 > 1024)
        return false;
    const int32_t th = H - 2 * R;
    int32_t P = 64;
    while (P < W) P <<= 1;
    L->P = P;
    L->N2 = P / 2;
    L->log2n2 = 0;
    while ((1 << L->log2n2) < L->N2) ++L->log2n2;
    L->n_kt = (int32_t)ceil_div(L->N2 + 1, COL_KC);
    L->PS = L->n_kt * COL_KC;
    L->D = 2 * R + 1;
    // lags in passes of equal width, template rows in blocks of M
    L->n_grp = (int32_t)ceil_div(L->D, COL_LAGS);
    L->Dg = (int32_t)ceil_div(L->D, L->n_grp);
    L->M = COL_L - L->Dg + 1;
    L->n_blk = (int32_t)ceil_div(th, L->M);
    // bands of blocks: about 1024 workgroups (two waves of two per compute unit) for four
    // frames; the number of frames itself stays out of it, so that a frame's scores do not
    // depend on how many it is searched with
    const int32_t want = (int32_t)ceil_div(1024, 4 * (int64_t)L->n_kt * L->n_grp);
    L->bpb = (int32_t)ceil_div(L->n_blk, std::min(want, L->n_blk));
    L->n_band = (int32_t)ceil_div(L->n_blk, L->bpb);
    // frames per round of spectra, the rounds of equal size
    const size_t per_frame = sizeof(double2) * (size_t)L->PS * ((size_t)H + (size_t)L->n_band * L->D);
    L->F = (int32_t)std::max<size_t>(1, std::min<size_t>((size_t)N, round_bytes / per_frame));
    L->F = (int32_t)ceil_div(N, ceil_div(N, L->F));
    L->refine = reg_plan(W, H, 1, R);
    L->full = reg_plan(W, H, R, R);
    if (L->refine.D == 0 || L->full.D == 0) return false;
    const size_t per_full = sizeof(double) * (size_t)L->full.n_tiles * L->full.D * L->full.D;
    L->Ffull = (int32_t)std::max<size_t>(1, std::min<size_t>((size_t)N, FFT_FALLBACK_BYTES / per_full));
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += al256(std::max<size_t>(bytes, 1));
        return at;
    };
    L->tw = take(sizeof(double2) * P);
    L->mean_parts = take(sizeof(double) * (size_t)ceil_div(th, MEAN_ROWS));
    L->mean = take(sizeof(double));
    L->Bt = take(sizeof(double2) * 16 * COL_T * (size_t)L->n_kt * L->n_blk);
    L->rowsq_b = take(sizeof(double) * (size_t)th);
    L->A = take(sizeof(double2) * (size_t)L->PS * H * L->F);  // the template's row spectra before the frames'
    L->rowsq_a = take(sizeof(double) * (size_t)H * N);  // every frame's, for the decisions
    L->Zp = take(sizeof(double2) * (size_t)L->PS * L->n_band * L->D * L->F);
    L->S_fft = take(sizeof(double) * (size_t)N * L->D * L->D);
    L->cen = take(sizeof(int32_t) * 2 * (size_t)N);
    L->info = take(sizeof(int32_t) * ((size_t)N + 1));  // by frame, the skipped one among them
    L->fb = take(sizeof(int32_t) * (size_t)N);
    const RegPlan &pr = L->refine, &pf = L->full;
    L->part_r = take(sizeof(double) * (size_t)N * pr.n_tiles * pr.D * pr.D);
    L->part_f = take(per_full * (size_t)L->Ffull);
    L->sc_f = take(sizeof(double) * (size_t)L->Ffull * pf.D * pf.D);
    L->total = o;
    return true;
}

static int fft_check(int32_t W, int32_t H, int32_t N, int32_t R, const char *who)
{
    const std::string w(who);
    if (W < 1 || H < 1 || N < 1) return fail(REDUCE_ERR_SHAPE, w + ": W, H, N must be >= 1");
    if (R < 1) return fail(REDUCE_ERR_RANGE, w + ": radius must be >= 1");
    if (W - 2 * R < 1 || H - 2 * R < 1) return fail(REDUCE_ERR_RANGE, w + ": radius leaves no template");
    if (W > FFT_P_MAX) return fail(REDUCE_ERR_UNSUPPORTED, w + ": rows longer than 8192");
    if (N > 65535) return fail(REDUCE_ERR_UNSUPPORTED, w + ": N above 65535");
    if (2 * R + 1 > 1024) return fail(REDUCE_ERR_UNSUPPORTED, w + ": radius above 511");
    return REDUCE_OK;
}

// P/2 from 32 (P = 64) to 4096 (P = 8192)
template <typename F>
static void log2_dispatch(int32_t log2n2, F &&f)
{
    switch (log2n2) {
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 10: f(std::integral_constant<int, 10>{}); break;
    case 11: f(std::integral_constant<int, 11>{}); break;
    default: f(std::integral_constant<int, 12>{}); break;
    }
}

static void launch_fft_rows(const FftLayout &L, const RowSrc &src, int32_t rows_out, int32_t batches,
                            const double2 *tw, double2 *spec, int64_t spec_batch, double *rowsq, hipStream_t s)
{
    const int rpw = FFT_POINTS / L.N2;
    const dim3 grid((unsigned)ceil_div(rows_out, rpw), (unsigned)batches);
    log2_dispatch(L.log2n2, [&](auto Lc) {
        hipLaunchKernelGGL(fft_rows<decltype(Lc)::value>, grid, dim3(FFT_THREADS), 0, s, src, rows_out, tw,
                           spec, spec_batch, L.PS, rowsq);
    });
}

bool spectra_pay(int32_t W, int32_t H, int32_t N, int32_t R)
{
    if (R < 1 || N < 1 || N > 65535 || W > FFT_P_MAX || 2 * R + 1 > 1024 || W - 2 * R < 1 || H - 2 * R < 1) return false;
    // a launch shape tuned for these sizes is what later calls of them use, so tuning keeps the
    // direct sums also where the spectra are faster (three stacks of 10 frames of 1024x1024 at R = 21 2.1
    // ms tuned, 0.53 untuned); reduce_tune_search times both
    RegShape tuned;
    if (tuned_reg_shape(W, H, R, R, &tuned)) return false;
    // Microseconds of both, from measured calls.  Direct sums: 23 - 40 TFLOP/s (512x512 x 16 at
    // R = 17 347 us, 1024x1024 x 16 1182, 2048x2048 x 16 at R = 33 13264; windows of side 7 and
    // less half of that), so the estimate is a low one.  Spectra: 100 us of dependent small
    // launches and 6.5 us per million row values of the padded frames and the template (the
    // same calls: 130, 206, 599), of which the contraction's part grows with its passes and
    // with the rows its blocks read twice.  The estimates are cautious at the line: 30 shapes
    // drawn at 1.25 to 1.6 times the spectra's estimate took 0.28 - 0.61 of the direct
    // sums' time through spectra, and batches of 11 to 54 equal stacks of them, whose direct tiles share one
    // launch and whose spectral searches run one after the other, 0.36 - 0.65.
    const double D = 2.0 * R + 1.0, T = (double)(W - 2 * R) * (H - 2 * R);
    const double direct = 2.0 * N * T * D * D / 40e6;
    int32_t P = 64;
    while (P < W) P <<= 1;
    const int32_t passes = (int32_t)ceil_div(2 * R + 1, COL_LAGS);
    const double reread = (double)COL_L / (COL_L + 1 - (int32_t)ceil_div(2 * R + 1, passes));
    const double spectral = 100.0 + (4.0 + 2.2 * passes * reread) * 1e-6 * (N + 1.0) * P * H;
    return direct > 1.25 * spectral;
}

int spectral_search(const FftLayout &L, const float *ref, const float *frames, int32_t W, int32_t H, int32_t N,
                    int32_t R, int32_t skip, reduce_offset_t *out, double *scores, int32_t *info, void *ws,
                    hipStream_t s)
{
    unsigned char *b = static_cast<unsigned char *>(ws);
    auto at = [&](size_t off) { return static_cast<void *>(b + off); };
    double2 *tw = static_cast<double2 *>(at(L.tw));
    double *mean = static_cast<double *>(at(L.mean));
    double *rowsq_b = static_cast<double *>(at(L.rowsq_b));
    double2 *As = static_cast<double2 *>(at(L.A));
    double *rowsq_a = static_cast<double *>(at(L.rowsq_a));
    double2 *Zp = static_cast<double2 *>(at(L.Zp));
    double *Sf = scores ? scores : static_cast<double *>(at(L.S_fft));
    int32_t *cen = static_cast<int32_t *>(at(L.cen));
    int32_t *inf = info ? info : static_cast<int32_t *>(at(L.info));
    int32_t *fb = static_cast<int32_t *>(at(L.fb));
    const int32_t D = L.D;
    const int32_t tx0 = R, ty0 = R, tw_ = W - 2 * R, th = H - 2 * R;
    const int64_t a_batch = (int64_t)L.PS * H;
    ProfScope prof("register_fft", s);

    const int32_t n_parts = (int32_t)ceil_div(th, MEAN_ROWS);
    double *mean_parts = static_cast<double *>(at(L.mean_parts));
    hipLaunchKernelGGL(spec_prepare, dim3((unsigned)(n_parts + ceil_div(L.P, MEAN_THREADS))), dim3(MEAN_THREADS), 0, s,
                       ref, W, tx0, ty0, tw_, th, n_parts, mean_parts, tw, L.P);
    register_mean_final(mean_parts, n_parts, (double)tw_ * (double)th, mean, s);
    {
        ProfScope p2("fft_rows", s);
        const RowSrc tsrc{ref + (int64_t)ty0 * W + tx0, 0, W, tw_, th, mean, 0x7fffffff};
        launch_fft_rows(L, tsrc, th, 1, tw, As, 0, rowsq_b, s);
    }
    ColArgs ca;
    ca.A = As;
    ca.Bt = static_cast<double2 *>(at(L.Bt));
    ca.Zp = Zp;
    ca.a_batch = a_batch;
    ca.PS = L.PS;
    ca.D = D;
    ca.Dg = L.Dg;
    ca.n_grp = L.n_grp;
    ca.M = L.M;
    ca.H = H;
    ca.n_blk = L.n_blk;
    ca.n_band = L.n_band;
    ca.bpb = L.bpb;
    ca.n_kt = L.n_kt;
    ca.nf = 0;
    {
        ProfScope p2("spec_corr", s);
        hipLaunchKernelGGL(spec_tmpl, dim3((unsigned)L.n_kt, (unsigned)L.n_blk), dim3(COL_T), 0, s, ca, As, th);
    }
    for (int32_t f0 = 0; f0 < N; f0 += L.F) {
        const int32_t nf = std::min(L.F, N - f0);
        {
            ProfScope p2("fft_rows", s);
            const RowSrc fsrc{frames + (int64_t)(f0 + (f0 > skip)) * W * H, (int64_t)W * H, W, W, H, nullptr,
                              f0 > skip ? 0x7fffffff : skip - f0};
            launch_fft_rows(L, fsrc, H, nf, tw, As, a_batch, rowsq_a + (int64_t)f0 * H, s);
        }
        {
            ProfScope p2("spec_corr", s);
            ca.nf = nf;
            hipLaunchKernelGGL(spec_cols, dim3((unsigned)(L.n_kt * L.n_band * L.n_grp * nf)), dim3(COL_T), 0, s, ca);
        }
        {
            ProfScope p2("spec_eval", s);
            log2_dispatch(L.log2n2, [&](auto Lc) {
                const int64_t lags = std::max<int64_t>(COL_KC / std::max<int64_t>(L.P / COL_L, 1), 1);  // per workgroup
                hipLaunchKernelGGL(spec_eval<decltype(Lc)::value>,
                                   dim3((unsigned)ceil_div(D, lags), (unsigned)nf, (unsigned)ceil_div(D, COL_L)),
                                   dim3(COL_T), 0, s, Zp, L.n_band, D, L.PS, tw, Sf + (int64_t)f0 * D * D);
            });
        }
    }
    hipLaunchKernelGGL(spec_pick, dim3((unsigned)N), dim3(PICK_THREADS), 0, s, Sf, D, R, cen);
    // exact +-1 windows around the spectral maxima and the decisions
    {
        ProfScope p2("fft_refine", s);
        double *part_r = static_cast<double *>(at(L.part_r));
        const int32_t n_tiles = register_small_scores(L.refine, ref, frames, W, H, N, 1, R, cen, tx0, ty0, tw_, th,
                                                      mean, part_r, skip, s);
        const double eps = 1.1102230246251565e-16;  // 2^-53
        const double factor = 4.0 * eps * (10.0 * L.log2n2 + (double)ceil_div(COL_L, L.M) * (124.0 + L.n_blk) +
                                           (double)L.P + 50.0);
        hipLaunchKernelGGL(spec_settle, dim3((unsigned)N), dim3(PICK_THREADS), 0, s, part_r, n_tiles, cen, Sf, D, R,
                           rowsq_a, H, rowsq_b, th, factor, skip, out, fb, inf);
    }
    // the full direct search for the frames not settled (nothing, for most calls)
    {
        ProfScope p2("fft_fallback", s);
        for (int32_t r0 = 0; r0 < N; r0 += L.Ffull) {
            const int32_t n = std::min(L.Ffull, N - r0);
            register_scores(L.full, ref, frames, W, H, n, R, R, nullptr, fb + r0, tx0, ty0, tw_, th, mean,
                            static_cast<double *>(at(L.part_f)), static_cast<double *>(at(L.sc_f)), out, s, WindowMove{});
        }
    }
    return check_launch("search through row spectra");
}

}  // namespace rd

using namespace rd;

extern "C" size_t reduce_register_fft_ws(int32_t W, int32_t H, int32_t N, int32_t radius)
{
    FftLayout L;
    return fft_layout(W, H, N, radius, SPEC_ROUND_BYTES, &L) ? L.total : 0;
}

extern "C" int reduce_register_fft(const float *ref, const float *frames, int32_t W, int32_t H, int32_t N,
                                   int32_t radius, reduce_offset_t *out, double *scores, int32_t *info, void *ws,
                                   size_t ws_bytes, void *stream)
{
    if (!ref || !frames || !out) return fail(REDUCE_ERR_NULL, "reduce_register_fft: NULL buffer");
    const int c = fft_check(W, H, N, radius, "reduce_register_fft");
    if (c != REDUCE_OK) return c;
    FftLayout L;
    if (!fft_layout(W, H, N, radius, SPEC_ROUND_BYTES, &L))
        return fail(REDUCE_ERR_UNSUPPORTED, "reduce_register_fft: no launch shape for these sizes");
    if (!ws || ws_bytes < L.total)
        return fail(REDUCE_ERR_WORKSPACE, "reduce_register_fft: workspace needs " + std::to_string(L.total) + " bytes");
    return spectral_search(L, ref, frames, W, H, N, radius, 0x7fffffff, out, scores, info, ws, as_stream(stream));
}
