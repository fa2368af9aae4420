// Device routine of the sigma-clipped mean over one pixel column held by a group of
// L lanes; used by the stage-wise combine kernel and by the fused batch kernel so
// both evaluate identical operations in identical order.
#pragma once

#include <type_traits>

#include "common.h"

namespace rd {

constexpr int COMB_TILE = 256;
constexpr int COMB_MAX_N = 48;        // LDS tile [N][256] floats stays within 48 KB
constexpr int COMB_MAX_N_COLS = 128;  // one lane per column: the column in registers

template <int MAXV>
struct ClipResult {
    float mean;      // mean of the kept values, rounded to float
    uint64_t kept;   // bit i: value lane + L*i is kept
    int dropped;     // values dropped over all iterations (whole group)
};

template <int L>
__device__ __forceinline__ double group_sum(double v)
{
#pragma unroll
    for (int off = 1; off < L; off <<= 1) v += __shfl_xor(v, off, L);
    return v;
}

template <int L>
__device__ __forceinline__ int group_sum(int v)
{
#pragma unroll
    for (int off = 1; off < L; off <<= 1) v += __shfl_xor(v, off, L);
    return v;
}

// Iterative clip: mean m and population sigma of the kept values, drop |x - m| >
// ksigma * sigma (all decided against the same m, sigma), stop when nothing drops
// or after max_iters passes, return the mean of what is kept.  Lane `lane` of the
// group owns the values col[(lane + L*i) * COMB_TILE], read from LDS on every pass
// (the compiler barrier keeps them from being hoisted into registers).  With L = 1
// the sums run over the frames in index order.
template <int L, int MAXV>
__device__ __forceinline__ ClipResult<MAXV> clip_column(const float *col, int32_t N, int lane, double ksigma,
                                                        int32_t max_iters)
{
    uint64_t kept = 0;
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
        if (lane + L * i < N) kept |= (1ull << i);
    int n = N;
    int dropped = 0;
    for (int32_t it = 0; it < max_iters; ++it) {
        asm volatile("" ::: "memory");
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < MAXV; ++i)
            if ((kept >> i) & 1ull) s = __dadd_rn(s, (double)col[(lane + L * i) * COMB_TILE]);
        s = group_sum<L>(s);
        const double m = s / (double)n;
        double q = 0.0;
#pragma unroll
        for (int i = 0; i < MAXV; ++i)
            if ((kept >> i) & 1ull) {
                const double d = __dsub_rn((double)col[(lane + L * i) * COMB_TILE], m);
                q = __dadd_rn(q, __dmul_rn(d, d));
            }
        q = group_sum<L>(q);
        const double thr = __dmul_rn(ksigma, sqrt(q / (double)n));
        int drop = 0;
#pragma unroll
        for (int i = 0; i < MAXV; ++i)
            if (((kept >> i) & 1ull) && fabs(__dsub_rn((double)col[(lane + L * i) * COMB_TILE], m)) > thr) {
                kept &= ~(1ull << i);
                ++drop;
            }
        drop = group_sum<L>(drop);
        n -= drop;
        dropped += drop;
        if (drop == 0) break;
    }
    asm volatile("" ::: "memory");
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
        if ((kept >> i) & 1ull) s = __dadd_rn(s, (double)col[(lane + L * i) * COMB_TILE]);
    s = group_sum<L>(s);
    ClipResult<MAXV> r;
    r.mean = (float)(s / (double)n);
    r.kept = kept;
    r.dropped = dropped;
    return r;
}

// Clip the COMB_TILE pixel columns staged in LDS (tile[k * COMB_TILE + px] = value of
// frame k at pixel p0 + px) with groups of L lanes; the first COMB_TILE threads take
// part.  Writes out[p0 + px] and the keep mask; returns the values this thread
// dropped (counted in each group's lane 0).
template <int L, int MAXV>
__device__ __forceinline__ unsigned clip_tile(const float *tile, int64_t p0, int64_t plane, int32_t N,
                                              double ksigma, int32_t max_iters, float *out, uint8_t *keep)
{
    const int t = threadIdx.x;
    if (t >= COMB_TILE) return 0u;
    const int lane = t % L;
    const int group = t / L;
    constexpr int GROUPS = COMB_TILE / L;
    unsigned dropped_here = 0;
    for (int r = 0; r < L; ++r) {
        const int px = group + GROUPS * r;
        const int64_t p = p0 + px;
        ClipResult<MAXV> res = clip_column<L, MAXV>(tile + px, N, lane, ksigma, max_iters);
        if (p < plane) {
            if (lane == 0) out[p] = res.mean;
            if (keep) {
#pragma unroll
                for (int i = 0; i < MAXV; ++i) {
                    const int k = lane + L * i;
                    if (k < N) keep[k * plane + p] = (uint8_t)((res.kept >> i) & 1u);
                }
            }
            if (lane == 0) dropped_here += (unsigned)res.dropped;
        }
    }
    return dropped_here;
}

// Sum of one unsigned per thread over a 256-thread workgroup.
__device__ __forceinline__ unsigned block_sum_u32(unsigned v)
{
    __shared__ unsigned part[COMB_TILE / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    unsigned t = 0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += part[i];
    return t;
}

// ---- one thread per pixel column ---------------------------------------------------------
// f(i, exists) for i < N in order, i a constant after unrolling, eight at a time behind one
// uniform test; in the group that N ends in, f also sees values past it (exists = false),
// which hold the last frame's and are to be selected away, not branched around: branches per
// value made the compiler keep the column in scratch.
template <int MAXV, typename F>
__device__ __forceinline__ void each_value(int32_t N, F f)
{
    static_assert(MAXV % 8 == 0, "whole groups of eight");
    asm volatile("" : "+s"(N));  // each pass makes its own tests: kept across passes they spill
#pragma unroll
    for (int c = 0; c < MAXV; c += 8) {
        if (c + 8 <= N) {
#pragma unroll
            for (int j = 0; j < 8; ++j) f(c + j, true);
        } else if (c < N) {
#pragma unroll
            for (int j = 0; j < 8; ++j) f(c + j, c + j < N);
        }
    }
}

// The same for loops that fill a column's values: f(i) also past N up to the next eight.
template <int MAXV, typename F>
__device__ __forceinline__ void each_group(int32_t N, F f)
{
    asm volatile("" : "+s"(N));
#pragma unroll
    for (int c = 0; c < MAXV; c += 8)
        if (c < N) {
#pragma unroll
            for (int j = 0; j < 8; ++j) f(c + j);
        }
}

typedef float f32x2v __attribute__((ext_vector_type(2)));

// The planes of the frames in turn: a uniform address, moved on by one plane per step and
// opaque to the compiler, which would otherwise form all N plane addresses before the first
// load and hold them for the later loops (hundreds of spilled scalar registers).
template <typename T>
struct PlaneWalk {
    typedef __attribute__((address_space(1))) T G;  // global: not a flat access
    G *at;
    int64_t pstride;
    int32_t left;  // steps until the last plane, where the walk stays
    __device__ __forceinline__ PlaneWalk(T *first, int64_t stride, int32_t N) : pstride(stride), left(N - 1)
    {
        const uint64_t a = reinterpret_cast<uint64_t>(first);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
        at = (G *)(((uint64_t)hi << 32) | lo);
    }
    __device__ __forceinline__ G *next(int i)
    {
        G *r = at;
        at += i < left ? pstride : 0;
        asm volatile("" : "+s"(at));
        return r;
    }
};

// The kept values of a column are those inside [lo, hi]: |x - m| > threshold is monotonic in
// x on either side of m, also as rounded, so an iteration keeps an interval of floats, and
// what several iterations keep (nothing dropped comes back) is the interval they share.  The
// tests of a pass are then two float comparisons where a flag per value took a 64-bit mask
// and selects.  A missing value (NaN) is in no interval.
struct ClipState {
    float lo, hi;  // kept: lo <= x <= hi
    double s;      // sum of the kept values in frame order
    int n;         // their number
};

// Sum and number of the kept values.  ALL: every value is kept (before the first drop,
// without missing values).  Not-kept values add +0 to a sum that starts at +0: nothing.
template <int MAXV, bool ALL, typename X>
__device__ __forceinline__ void clip_sum(X x, int32_t N, ClipState &c)
{
    c.s = 0.0;
    c.n = ALL ? N : 0;
    each_value<MAXV>(N, [&](int i, bool exists) {
        const float v = x(i);
        const bool k = exists && (ALL || (v >= c.lo && v <= c.hi));
        c.s = __dadd_rn(c.s, (double)(k ? v : 0.0f));
        if (!ALL) c.n += k ? 1 : 0;
    });
}

// Squared deviations of the kept values from m, in frame order, and the largest deviation.  A
// not-kept value's deviation is replaced by 0, which adds exactly nothing.
template <int MAXV, bool ALL, typename X>
__device__ __forceinline__ void clip_squares(X x, int32_t N, const ClipState &c, double m, double &q, double &dmax)
{
    q = 0.0;
    dmax = 0.0;
    each_value<MAXV>(N, [&](int i, bool exists) {
        const float v = x(i);
        double d = __dsub_rn((double)v, m);
        if (ALL)
            d = exists ? d : 0.0;
        else
            d = exists && v >= c.lo && v <= c.hi ? d : 0.0;
        q = __dadd_rn(q, __dmul_rn(d, d));
        dmax = fmax(dmax, fabs(d));
    });
}

// Floats in order as integers, and back.
__device__ __forceinline__ int32_t float_key(float v)
{
    const int32_t i = __float_as_int(v);
    return i ^ ((i >> 31) & 0x7fffffff);
}

__device__ __forceinline__ float key_float(int32_t k) { return __int_as_float(k ^ ((k >> 31) & 0x7fffffff)); }

// The largest float x with x - m <= thr as rounded (m and thr finite): the rounded sum m + thr
// or its neighbour below, except where m + thr nearly cancels, when many floats round to one
// difference and the end is found by bisection (33 steps at most).
__device__ __forceinline__ float clip_end(double m, double thr)
{
    auto ok = [&](int32_t k) { return __dsub_rn((double)key_float(k), m) <= thr; };
    const int32_t k = float_key((float)__dadd_rn(m, thr));
    int32_t in, out;  // the end is in [in, out): ok(in), not ok(out)
    if (ok(k)) {
        if (!ok(k + 1)) return key_float(k);
        in = k + 1;
        out = float_key(INFINITY);
    } else {
        if (ok(k - 1)) return key_float(k - 1);
        in = float_key(-INFINITY);
        out = k - 1;
    }
    while ((int64_t)out - in > 1) {
        const int32_t mid = (int32_t)(((int64_t)in + out) >> 1);
        if (ok(mid)) in = mid;
        else out = mid;
    }
    return key_float(in);
}

// The kept interval after an iteration with mean m and threshold thr: the floats with
// |x - m| <= thr as rounded, within the interval so far.
__device__ __forceinline__ void clip_narrow(ClipState &c, double m, double thr)
{
    c.hi = fminf(c.hi, clip_end(m, thr));
    c.lo = fmaxf(c.lo, -clip_end(-m, thr));
}

// The clip of one column, its values read through x(i).  The arithmetic is that of clip_column
// with one lane (sums in frame order in double, m = s / n, q = sum of (x - m)^2, threshold
// ksigma * sqrt(q / n), drop |x - m| > threshold); when an iteration drops nothing (the
// largest |x - m| tells) its own mean is the final mean.
//
// First iteration: true, with the mean, when the column settles there (nothing drops, or no
// iterations are asked for).
template <int MAXV, bool MISS, typename X>
__device__ __forceinline__ bool clip_first(X x, int32_t N, double ksigma, int32_t max_iters, ClipState &c,
                                           double &m, double &thr)
{
    c.lo = -INFINITY;
    c.hi = INFINITY;
    clip_sum<MAXV, !MISS>(x, N, c);
    m = c.s / (double)c.n;
    if (max_iters == 0) return true;
    double q, dmax;
    clip_squares<MAXV, !MISS>(x, N, c, m, q, dmax);
    thr = __dmul_rn(ksigma, sqrt(q / (double)c.n));
    return !(dmax > thr);
}

// The rest of the clip of a column whose first iteration (mean m, threshold thr, all values
// present in c) drops values.  c.lo, c.hi bound the kept values afterwards.
template <int MAXV, typename X>
__device__ __forceinline__ float clip_rest(X x, int32_t N, double ksigma, int32_t max_iters, ClipState &c, double m,
                                           double thr, unsigned &dropped)
{
    for (int32_t it = 1;; ++it) {
        const int n = c.n;
        clip_narrow(c, m, thr);
        clip_sum<MAXV, false>(x, N, c);
        dropped += (unsigned)(n - c.n);
        m = c.s / (double)c.n;
        if (it >= max_iters) break;
        double q, dmax;
        clip_squares<MAXV, false>(x, N, c, m, q, dmax);
        thr = __dmul_rn(ksigma, sqrt(q / (double)c.n));
        if (!(dmax > thr)) break;
    }
    return (float)m;
}

// Values in registers.  Each read goes through an empty asm statement that marks the value
// as changed, so every pass converts it to double again instead of holding the column's
// converted values across the passes (twice the registers; with them a compute unit holds
// fewer waves and the kernel ran 10% slower).
template <int MAXV>
struct RegColumn {
    const float (&x)[MAXV];
    __device__ __forceinline__ float operator()(int i) const
    {
        float v = x[i];
        asm volatile("" : "+v"(v));
        return v;
    }
};

// PX adjacent pixel columns per thread: each frame's PX values come in as one vector
// load (frame k's plane starts at aligned + k * pstride; pstride >= plane, and pstride
// and the pointers aligned to PX floats; with PX = 4 an even pstride is enough, a frame
// that starts 8-byte aligned taking two 8-byte loads).  Each thread runs the first
// iteration of its columns; a column that drops values there (a few percent of them, but
// in most waves at least one lane) goes to a queue in LDS, and once the workgroup's first
// iterations are done its threads take the queued columns one each (their values, means and
// thresholds kept in LDS for the first QCAP queued, else loaded and formed again) and run
// the rest of the clip, so the later iterations run on full waves instead of holding every wave
// that has one such lane.  No LDS copy for columns of 33 - 48 values (45 frames of 4096x2048:
// 0.71 ms loading them again, 2.05 holding them until the queue is written); columns of
// 49 - 128 values are built for three waves per SIMD and hold them (a quarter of 97-frame
// columns drop a value).
// Columns at or past `plane` are
// neither written nor counted.  The whole workgroup must call this (it synchronises).
template <int MAXV, int PX, bool MISS = false, int QCAP = (MAXV <= 32 ? 128 : MAXV <= 48 ? 0 : 96)>
__device__ __forceinline__ unsigned combine_cols_block(const float *__restrict__ aligned, int64_t plane,
                                                       int64_t pstride, int32_t N, double ksigma, int32_t max_iters,
                                                       float *__restrict__ out, uint8_t *__restrict__ keep,
                                                       int64_t block)
{
    __shared__ int32_t queue[COMB_TILE * PX];         // columns (of this workgroup) that drop values
    __shared__ float qv[MAXV * (QCAP > 0 ? QCAP : 1)];  // value i of queue entry e at qv[i * QCAP + e]
    // mean, threshold and number of values of the queued column's first iteration
    __shared__ double qm[QCAP > 0 ? QCAP : 1], qt[QCAP > 0 ? QCAP : 1];
    __shared__ int32_t qn[QCAP > 0 ? QCAP : 1];
    __shared__ int32_t queued;
    if (threadIdx.x == 0) queued = 0;
    const int64_t p0 = (block * COMB_TILE + threadIdx.x) * PX;
    const int64_t pb = block * COMB_TILE * PX;  // first column of the workgroup
    float xs[PX][MAXV];
    PlaneWalk<const float> in(aligned + pb, pstride, N);
    if (PX > 1 && p0 + PX <= plane) {
        const uint32_t o = threadIdx.x * PX;
        each_group<MAXV>(N, [&](int i) {
            // planes are aligned to two floats; the two pairs of PX = 4 become one load
            const auto src = in.next(i) + o;
#pragma unroll
            for (int c = 0; c < PX; c += 2) {
                const f32x2v v = *(const __attribute__((address_space(1))) f32x2v *)(src + c);
                xs[c][i] = v[0];
                if constexpr (PX > 1) xs[c + 1][i] = v[1];
            }
        });
    } else {
        // one column at a time; one past the plane reads the plane's last
        uint32_t o[PX];
#pragma unroll
        for (int c = 0; c < PX; ++c) o[c] = (uint32_t)(min(p0 + c, plane - 1) - pb);
        each_group<MAXV>(N, [&](int i) {
            const auto src = in.next(i);
#pragma unroll
            for (int c = 0; c < PX; ++c) xs[c][i] = src[o[c]];
        });
    }
    // first iterations; a column that drops values goes to the workgroup's queue
    double mean[PX], thr[PX];
    int n1[PX];
    bool done[PX];
    bool all = p0 + PX <= plane;
#pragma unroll
    for (int c = 0; c < PX; ++c) {
        ClipState st;
        done[c] = clip_first<MAXV, MISS>(RegColumn<MAXV>{xs[c]}, N, ksigma, max_iters, st, mean[c], thr[c]);
        n1[c] = st.n;
        all = all && done[c];
    }
    __syncthreads();  // the queue is empty
    if (PX > 1 && all) {
        if constexpr (PX == 4)
            *reinterpret_cast<float4 *>(out + p0) = make_float4((float)mean[0], (float)mean[1], (float)mean[2],
                                                                   (float)mean[3]);
        else if constexpr (PX == 2)
            *reinterpret_cast<float2 *>(out + p0) = make_float2((float)mean[0], (float)mean[1]);
    } else {
#pragma unroll
        for (int c = 0; c < PX; ++c)
            if (p0 + c < plane) {
                if (done[c]) {
                    out[p0 + c] = (float)mean[c];
                } else {
                    const int32_t e = atomicAdd(&queued, 1);
                    queue[e] = (int32_t)threadIdx.x * PX + c;
                    if (e < QCAP) {
                        each_group<MAXV>(N, [&](int i) { qv[i * QCAP + e] = xs[c][i]; });
                        qm[e] = mean[c];
                        qt[e] = thr[c];
                        qn[e] = n1[c];
                    }
                }
            }
    }
    if (keep) {  // a settled column keeps every value (every value present)
        PlaneWalk<uint8_t> to(keep + pb, plane, N);
        each_value<MAXV>(N, [&](int i, bool exists) {
            const auto dst = to.next(i) + threadIdx.x * PX;
#pragma unroll
            for (int c = 0; c < PX; ++c)
                if (exists && p0 + c < plane && done[c]) dst[c] = (uint8_t)(!MISS || xs[c][i] == xs[c][i]);
        });
    }
    __syncthreads();
    // the queued columns, one per thread: the whole clip (values from LDS, past QCAP
    // entries loaded again)
    unsigned dropped = 0;
    const int32_t nq = queued;
    for (int32_t e = threadIdx.x; e < nq; e += COMB_TILE) {
        const uint32_t o = (uint32_t)queue[e];
        const int64_t p = pb + o;
        float x[MAXV];
        if (e < QCAP)
            each_group<MAXV>(N, [&](int i) { x[i] = qv[i * QCAP + e]; });
        else {
            PlaneWalk<const float> again(aligned + pb, pstride, N);
            each_group<MAXV>(N, [&](int i) { x[i] = again.next(i)[o]; });
        }
        ClipState st;
        double m, t;
        if (e < QCAP) {
            st.lo = -INFINITY;
            st.hi = INFINITY;
            st.n = qn[e];
            m = qm[e];
            t = qt[e];
        } else {
            clip_first<MAXV, MISS>(RegColumn<MAXV>{x}, N, ksigma, max_iters, st, m, t);
        }
        out[p] = clip_rest<MAXV>(RegColumn<MAXV>{x}, N, ksigma, max_iters, st, m, t, dropped);
        if (keep) {
            PlaneWalk<uint8_t> to(keep + pb, plane, N);
            each_value<MAXV>(N, [&](int i, bool exists) {
                const auto dst = to.next(i) + o;
                if (exists) *dst = (uint8_t)(x[i] >= st.lo && x[i] <= st.hi);
            });
        }
    }
    return dropped;
}

// Register class of a stack of 49 - 128 frames: a class's loops cover its MAXV values in groups
// of eight whatever N is.  65 - 104 frames have a class of their own (three waves per SIMD
// as the largest): 104 frames of 1000x600 take 102 us in it, 105 in the next 113.
template <typename F>
inline void deep_dispatch(int32_t N, F &&f)
{
    if (N <= 64) f(std::integral_constant<int, 64>{});
    else if (N <= 104) f(std::integral_constant<int, 104>{});
    else f(std::integral_constant<int, 128>{});
}

}  // namespace rd
