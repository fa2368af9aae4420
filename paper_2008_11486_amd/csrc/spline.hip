// Bicubic-spline sub-pixel shift onto the common overlap: the paper's own interpolation
// (Section 2.1 and 2.2; Section 3.2.1 prices its tridiagonal systems, one per image row
// or column).  The interpolant is the tensor-product natural cubic spline through the
// pixel values on the integer grid, evaluated at (x + s_x, y + s_y).
//
// Along one line of L values the natural spline's second derivatives M satisfy
//   M[i-1] + 4 M[i] + M[i+1] = g[i] := 6 (f[i+1] - 2 f[i] + f[i-1]),  0 < i < L-1,
//   M[0] = M[L-1] = 0.
// On an unbounded line the inverse of the (1, 4, 1) operator is h[j] = z^|j| / (2 sqrt 3)
// with z = sqrt 3 - 2, so with g = 0 outside the interior, P = h * g satisfies every
// interior equation, and M = P + A z^i + B z^(L-1-i) adds the two homogeneous solutions
// whose coefficients make both ends zero.  P is not formed as a sum over h: h factors into
// a causal and an anticausal first-order recursion (sp_recur), which a thread runs over
// its own run of knots, started 16 knots outside it (|z|^17 < 2e-10).  On [i, i+1], with
// t = x - i,
//   S(x) = (1-t) f[i] + t f[i+1] + ((1-t)^3 - (1-t)) M[i] / 6 + (t^3 - t) M[i+1] / 6.
// Positions are clamped into [0, L-1] (inside the overlap they never need it); a clamped
// position takes f[0] or f[L-1].
//
// One pass, FP32 arithmetic: a workgroup walks down a strip of columns, forms the row
// splines of 32 frame rows at a time at the shifted x of its columns, keeps them in LDS and
// takes the column splines of those at the shifted y.  The shift is the same for the whole
// frame, so output u sits on knot x0 + fx + u (before clamping) with the same fraction: a
// thread that owns a run of knots holds in registers everything its run's outputs need.
#include <algorithm>
#include <string>
#include <type_traits>

#include "common.h"
#include "shift_core.h"  // clampi

namespace rd {

constexpr int SP_T = 16;                          // recursion warm-up, knots
constexpr double SP_Z = -0.26794919243112270;     // sqrt 3 - 2
constexpr double SP_H0 = 0.28867513459481287;     // 1 / (2 sqrt 3)

struct SpTaps {
    float v[SP_T + 1];
};
__host__ __device__ constexpr SpTaps sp_taps()
{
    SpTaps t{};
    double p = 1.0;
    for (int j = 0; j <= SP_T; ++j) {
        t.v[j] = (float)(SP_H0 * p);
        p *= SP_Z;
    }
    return t;
}

// z^n for n >= 0 (zero once it is far below single precision)
__device__ __forceinline__ float sp_zpow(int32_t n)
{
    if (n < 0 || n >= 64) return 0.0f;
    const float a = exp2f((float)n * -1.8999686269529916f);  // log2 |z|
    return (n & 1) ? -a : a;
}

// The end-correction coefficients (A, B) of one line from P[0] and P[L-1].
__device__ __forceinline__ void sp_ends(float P0, float PL, int32_t L, float &A, float &B)
{
    const float zL = sp_zpow(L - 1);
    const float den = 1.0f - zL * zL;
    A = (-P0 + PL * zL) / den;
    B = (-PL + P0 * zL) / den;
}

// P[0] (end 0) or P[L-1] (end 1) of a line read through get(i), i in [0, L): h * g with
// g zero outside 1 .. L-2, which reaches 16 knots in.
template <typename Get>
__device__ __forceinline__ float sp_end_p(Get get, int32_t L, int end)
{
    constexpr SpTaps h = sp_taps();
    float p = 0.0f;
#pragma unroll
    for (int j = 1; j <= SP_T; ++j) {
        const int32_t m = end ? L - 1 - j : j;
        if (m >= 1 && m <= L - 2) p += h.v[j] * (6.0f * (get(m + 1) - 2.0f * get(m) + get(m - 1)));
    }
    return p;
}

// The four weights of S for a fixed fraction t: S = a f[i] + b f[i+1] + c M[i] + d M[i+1].
struct SpW {
    float a, b, c, d;
};
__device__ __forceinline__ SpW sp_weights(float t)
{
    const float u = 1.0f - t;
    return SpW{u, t, (u * u * u - u) * (1.0f / 6.0f), (t * t * t - t) * (1.0f / 6.0f)};
}
__device__ __forceinline__ float sp_apply(const SpW &wt, float fi, float fi1, float Mi, float Mi1)
{
    return fmaf(wt.d, Mi1, fmaf(wt.c, Mi, fmaf(wt.b, fi1, wt.a * fi)));
}

// P (up to the end corrections) of knots s .. s+K from fw[r] = f[s - SP_T - 1 + r]: the
// inverse of (1, 4, 1) on the unbounded line factors as (-z) / ((1 - z S^-1)(1 - z S)),
// S the shift, so P = -6 z d with c[m] = D2f[m] + z c[m-1] (causal) and
// d[m] = c[m] + z d[m+1] (anticausal), D2f[m] = f[m+1] - 2 f[m] + f[m-1].  Both
// recursions start SP_T knots outside the run with zero state; the state they miss is
// below z^17 (2e-10) of the data.
template <int K>
__device__ __forceinline__ void sp_recur(const float (&fw)[K + 2 * SP_T + 3], float (&p)[K + 1])
{
    const float z = (float)SP_Z, scale = (float)(-6.0 * SP_Z);
    float c[K + SP_T + 1];  // causal state at knots s .. s+K+SP_T
    float st = 0.0f;
#pragma unroll
    for (int r = 0; r <= K + 2 * SP_T; ++r) {  // knot s - SP_T + r
        const float g = fmaf(-2.0f, fw[r + 1], fw[r + 2] + fw[r]);
        st = fmaf(z, st, g);
        if (r >= SP_T) c[r - SP_T] = st;
    }
    float d = 0.0f;
#pragma unroll
    for (int r = K + SP_T; r >= 0; --r) {
        d = fmaf(z, d, c[r]);
        if (r <= K) p[r] = scale * d;
    }
}

// The recursion reads staged values clamped into the line, so next to an end its g holds
// D2f[0] = f[1] - f[0] and D2f[L-1] = f[L-2] - f[L-1] instead of zero (further out the
// clamped values give exactly zero).  Their responses, 6 h[i] e0 and 6 h[L-1-i] e1, have
// the shape of the two end corrections, so they are taken out of (A, B): returns the
// coefficients to add to P from P[0], P[L-1] of the true g and the four end values.
__device__ __forceinline__ void sp_ends_raw(float P0, float PL, int32_t L, float f0, float f1, float fl2, float fl1,
                                            float &A, float &B)
{
    sp_ends(P0, PL, L, A, B);
    const float c6 = (float)(6.0 * SP_H0);
    A -= c6 * fmaf(-2.0f, f0, f1 + f0);    // the recursion's own g at knot 0
    B -= c6 * fmaf(-2.0f, fl1, fl1 + fl2);  // and at knot L-1
}

// The outputs of a run of K knots s .. s+K-1 (M of knot s+K is p[K]): fw and p as in
// sp_recur.  Knots at or beyond an end first get their M (zero at both ends, plus the
// end corrections near them); a knot outside 0 .. L-2 is a clamped position, whose value
// is the staged (clamped) line value.
template <int K>
__device__ __forceinline__ void sp_outputs(const float (&fw)[K + 2 * SP_T + 3], float (&p)[K + 1], int32_t s,
                                           int32_t L, bool near, float A, float B, const SpW &wt, float (&o)[K])
{
    // (the powers of z by products along the run: a power per knot and end, an exp2 each, made
    // the correction cost more than the recursions in rows of one run)
    if (near) {
        const float z = (float)SP_Z;
        float e = A * sp_zpow(max(s, 0));  // A z^i, from knot max(s, 0) on
#pragma unroll
        for (int r = 0; r <= K; ++r) {
            p[r] += e;
            e = s + r >= 0 ? e * z : e;
        }
        e = B * sp_zpow(max(L - 1 - (s + K), 0));  // B z^(L-1-i), from knot min(s + K, L - 1) back
#pragma unroll
        for (int r = K; r >= 0; --r) {
            p[r] += e;
            e = s + r <= L - 1 ? e * z : e;
        }
#pragma unroll
        for (int r = 0; r <= K; ++r) p[r] = s + r <= 0 || s + r >= L - 1 ? 0.0f : p[r];
    }
#pragma unroll
    for (int r = 0; r < K; ++r) {
        o[r] = sp_apply(wt, fw[r + SP_T + 1], fw[r + SP_T + 2], p[r], p[r + 1]);
        if (near) {
            const int32_t i = s + r;
            if (i < 0 || i > L - 2) o[r] = fw[r + SP_T + 1];
        }
    }
}

// ---- both passes in one --------------------------------------------------------------------
constexpr int SP_C = 64;                     // output columns of a strip
constexpr int SP_V = 32;                     // frame rows per batch, output rows per tile
constexpr int SP_Q = 16;                     // knots per thread, along x and along y
constexpr int SP_THREADS = SP_V * SP_C / SP_Q;
constexpr int SP_X = SP_C + 1 + 2 * SP_T + 2;  // staged values of a row; odd modulo 16, so that the 16 rows x 4
                                               // runs of a wave's windows start on distinct banks
constexpr int SP_RING = 96;                  // ring of row-spline lines: three batches (a tile reads 67 lines)
constexpr int SP_RP = SP_C + 1;              // its pitch: a wave stores 16 rows x 4 runs at once
constexpr int SP_NR = SP_V * 64 / SP_THREADS;  // rows a wave stages
static_assert(SP_X % 2 == 1 && SP_X > 64 && SP_X <= 128, "two loads per staged row");
constexpr int SP_AHEAD = SP_RING / SP_V - 1;   // batches formed before a tile
static_assert(SP_RING % SP_V == 0 && SP_V + 2 * SP_T + 3 <= SP_RING, "a tile's lines");

// The line ends matter to knots within SP_T + 1 of them only (|z|^18 < 6e-11 of the end's
// second derivative); a run of knots from ka on with an end that near, or with
// knots outside the line, is an end run.
__device__ __forceinline__ bool sp_end_run(int32_t ka, int32_t run, int32_t L)
{
    return L < 2 || ka <= SP_T + 1 || ka + run >= L - 2 - SP_T;
}

// (A, B) of a line from the values of an end run's window, get(i) = f[i].
template <typename Get>
__device__ __forceinline__ void sp_run_ends(Get get, int32_t ka, int32_t run, int32_t L, float &A, float &B)
{
    // with no knot of the line in the run every output is a clamped value
    const bool any = ka + run >= 0 && ka <= L - 1 && L >= 2;
    const bool near0 = any && ka <= SP_T + 1, nearL = any && ka + run >= L - 2 - SP_T;
    A = B = 0.0f;
    if (near0 || nearL)
        sp_ends_raw(near0 ? sp_end_p(get, L, 0) : 0.0f, nearL ? sp_end_p(get, L, 1) : 0.0f, L,
                    near0 ? get(0) : 0.0f, near0 ? get(1) : 0.0f, nearL ? get(L - 2) : 0.0f,
                    nearL ? get(L - 1) : 0.0f, A, B);
}

// A workgroup takes a strip of 64 output columns and n_tile tiles of 32 output rows of frame k.
// Batch b is the frame rows kb0 - 17 + 32 b ... of the walk whose first output row sits on
// knot kb0 (rows and columns clamped into the frame): 32 rows x 99 values are staged in LDS,
// four threads per row run the two recursions over 16 knots each and put the row splines
// into the ring, line m of the walk at ring row m mod 96.  Tile i reads lines 32 i ... 32 i
// + 66, batches i to i + 2; a thread has one column and 16 knots.  The next batch's loads
// are in flight while a batch and a tile are computed.
//
// Bound by HBM and by the recursions' issue alike.  Row and column passes over a workspace
// moved the frames twice (0.79 ms for 180 frames of 1020x1020, 0.68 with the end corrections
// by products); in one pass 0.49 ms, reading and writing once being 0.31 at the copy rate; batches of 64 rows 0.50.
// Strips of 64 columns read 99 for them, mostly from L2: neighbouring strips run on one XCD.
__global__ __launch_bounds__(SP_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void spline_shift(
    const float *__restrict__ in, float *__restrict__ out, int32_t W, int32_t H, const float *__restrict__ offs,
    int32_t x0, int32_t y0, int32_t w, int32_t h, int32_t n_strip, int32_t n_seg, int32_t n_tile)
{
    __shared__ float st[SP_V * SP_X];
    __shared__ float ring[SP_RING * SP_RP];
    const int32_t id = xcd_logical_id((int32_t)blockIdx.x, (int32_t)gridDim.x);
    const int32_t strip = id % n_strip, sk = id / n_strip, seg = sk % n_seg, k = sk / n_seg;
    const int32_t c0 = strip * SP_C, v_lo = seg * n_tile * SP_V, v_hi = min(v_lo + n_tile * SP_V, h);
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const float sx = offs[2 * k], sy = offs[2 * k + 1];
    const float flx = floorf(sx), fly = floorf(sy);
    const int32_t ka = x0 + c0 + (int32_t)flx;   // knot of the strip's first column (before clamping)
    const int32_t kb0 = y0 + v_lo + (int32_t)fly;  // knot of the walk's first row
    const int32_t xb = ka - SP_T - 1, yb = kb0 - SP_T - 1;
    const float *f = in + (int64_t)k * W * H;
    const SpW wx = sp_weights(sx - flx), wy = sp_weights(sy - fly);
    const bool end_x = sp_end_run(ka, SP_C, W);
    // the second load of a row repeats its last value in the lanes past it
    const int32_t cx0 = clampi(xb + lane, 0, W - 1), cx1 = clampi(xb + min(64 + lane, SP_X - 1), 0, W - 1);
    float r0[SP_NR], r1[SP_NR];
    auto load = [&](int32_t b) {  // wave wv: rows wv, wv + 4, ... of batch b
#pragma unroll
        for (int i = 0; i < SP_NR; ++i) {
            const float *row = f + (int64_t)clampi(yb + SP_V * b + wv + (SP_THREADS / 64) * i, 0, H - 1) * W;
            r0[i] = row[cx0];
            r1[i] = row[cx1];
        }
    };
    const int32_t tiles = (v_hi - v_lo + SP_V - 1) / SP_V;
    load(0);
    for (int32_t b = 0, slot = 0; b < tiles + SP_AHEAD; ++b, slot = slot + SP_V < SP_RING ? slot + SP_V : 0) {
        // the previous batch's windows have been read (barrier after them)
#pragma unroll
        for (int i = 0; i < SP_NR; ++i) st[(wv + (SP_THREADS / 64) * i) * SP_X + lane] = r0[i];
        if (lane < SP_X - 64) {
#pragma unroll
            for (int i = 0; i < SP_NR; ++i) st[(wv + (SP_THREADS / 64) * i) * SP_X + 64 + lane] = r1[i];
        }
        if (b + 1 < tiles + SP_AHEAD) load(b + 1);
        __syncthreads();  // the batch is staged, and the ring's older half has been read
        {
            const int rr = t >> 2, q0 = SP_Q * (t & 3);
            float fw[SP_Q + 2 * SP_T + 3], p[SP_Q + 1], o[SP_Q];
            const float *win = st + rr * SP_X;
#pragma unroll
            for (int r = 0; r < SP_Q + 2 * SP_T + 3; ++r) fw[r] = win[q0 + r];
            float A = 0.0f, B = 0.0f;
            int32_t kx = ka;
            asm volatile("" : "+s"(kx));  // the tests of the run's knots are not kept across batches (they spill)
            if (end_x) sp_run_ends([&](int32_t i) { return win[i - xb]; }, kx, SP_C, W, A, B);
            sp_recur<SP_Q>(fw, p);
            sp_outputs<SP_Q>(fw, p, kx + q0, W, end_x, A, B, wx, o);
            float *line = ring + (slot + rr) * SP_RP + q0;
#pragma unroll
            for (int r = 0; r < SP_Q; ++r) line[r] = o[r];
        }
        __syncthreads();
        if (b < SP_AHEAD) continue;
        // the tile's first row in the walk; its lines are i0 ..., in the ring from the slot after
        // this batch's on (the oldest)
        const int32_t i0 = SP_V * (b - SP_AHEAD);
        const int32_t s0 = slot + SP_V < SP_RING ? slot + SP_V : 0;
        const int c = lane, q0 = SP_Q * wv;
        const int32_t kb = kb0 + i0;
        auto line = [&](int32_t m) {  // line m of the walk
            const int32_t r = s0 + m - i0;
            return ring[(r < SP_RING ? r : r - SP_RING) * SP_RP + c];
        };
        float fw[SP_Q + 2 * SP_T + 3], p[SP_Q + 1], o[SP_Q];
        // the window's first line sits at a multiple of 16 in the ring: each place where it wraps
        // has its own reads at fixed offsets (an address per read was a fifth of the pass)
        const int32_t w0 = s0 + q0;  // < SP_RING
        const float *first = ring + w0 * SP_RP + c;
        auto window = [&](auto Wc) {
            constexpr int wrap = decltype(Wc)::value;  // reads from `wrap` on start over
#pragma unroll
            for (int r = 0; r < SP_Q + 2 * SP_T + 3; ++r) fw[r] = first[(r < wrap ? r : r - SP_RING) * SP_RP];
        };
        static_assert(SP_RING == 96 && SP_Q == 16, "places of the wrap");
        switch (w0) {
        case 48: window(std::integral_constant<int, 48>{}); break;
        case 64: window(std::integral_constant<int, 32>{}); break;
        case 80: window(std::integral_constant<int, 16>{}); break;
        default: window(std::integral_constant<int, SP_RING>{}); break;
        }
        const bool end_y = sp_end_run(kb, SP_V, H);
        float A = 0.0f, B = 0.0f;
        if (end_y) sp_run_ends([&](int32_t i) { return line(i - yb); }, kb, SP_V, H, A, B);
        sp_recur<SP_Q>(fw, p);
        sp_outputs<SP_Q>(fw, p, kb + q0, H, end_y, A, B, wy, o);
        if (c0 + c < w) {
            const int32_t v = v_lo + i0 + q0;
            float *dst = out + ((int64_t)k * h + v) * w + c0;  // uniform over the wave
            if (v + SP_Q <= v_hi) {
#pragma unroll
                for (int r = 0; r < SP_Q; ++r, dst += w) dst[c] = o[r];
            } else {
#pragma unroll
                for (int r = 0; r < SP_Q; ++r, dst += w)
                    if (v + r < v_hi) dst[c] = o[r];
            }
        }
    }
}

}  // namespace rd

using namespace rd;

// The one pass needs no workspace.  The entry point keeps the one that its interface asks for
// (N * H rows of w floats at a pitch of whole 256-byte segments) and touches none of it.
static int32_t spline_pitch(int32_t w) { return (w + 63) & ~63; }

extern "C" size_t reduce_shift_spline_ws(int32_t W, int32_t H, int32_t N)
{
    if (W < 1 || H < 1 || N < 1) return 0;
    return sizeof(float) * (size_t)N * H * (size_t)spline_pitch(W);
}

extern "C" int reduce_shift_spline(const float *in, float *out, int32_t W, int32_t H, int32_t N, const float *offs,
                                   const int32_t *rect, void *ws, size_t ws_bytes, void *stream)
{
    if (!in || !out || !offs || !rect || !ws) return fail(REDUCE_ERR_NULL, "reduce_shift_spline: NULL argument");
    if (W < 1 || H < 1 || N < 1) return fail(REDUCE_ERR_SHAPE, "reduce_shift_spline: W, H, N must be >= 1");
    const int32_t x0 = rect[0], y0 = rect[1], w = rect[2], h = rect[3];
    if (w < 1 || h < 1 || w > W || h > H) return fail(REDUCE_ERR_SHAPE, "reduce_shift_spline: empty or oversized rect");
    if (N > 65535 || H > 65535) return fail(REDUCE_ERR_UNSUPPORTED, "reduce_shift_spline: N or H above 65535");
    const int32_t wp = spline_pitch(w);
    const size_t need = sizeof(float) * (size_t)N * H * (size_t)wp;
    if (ws_bytes < need)
        return fail(REDUCE_ERR_WORKSPACE, "reduce_shift_spline: workspace needs " + std::to_string(need) + " bytes");
    hipStream_t s = as_stream(stream);
    ProfScope prof("shift_spline", s);
    // one walk down the whole strip where the strips fill the chip (four workgroups per compute
    // unit); with fewer, walks are cut, each cut forming one more batch of row splines
    const int32_t n_strip = (int32_t)ceil_div(w, SP_C), tiles = (int32_t)ceil_div(h, SP_V);
    const int64_t cuts = std::min<int64_t>(tiles, ceil_div(1024, (int64_t)n_strip * N));
    const int32_t n_tile = (int32_t)ceil_div(tiles, cuts), n_seg = (int32_t)ceil_div(tiles, n_tile);
    const int64_t grid = (int64_t)n_strip * n_seg * N;
    if (grid > INT32_MAX) return fail(REDUCE_ERR_UNSUPPORTED, "reduce_shift_spline: too many strips");
    hipLaunchKernelGGL(spline_shift, dim3((unsigned)grid), dim3(SP_THREADS), 0, s, in, out, W, H, offs, x0, y0, w, h,
                       n_strip, n_seg, n_tile);
    return check_launch("reduce_shift_spline");
}
