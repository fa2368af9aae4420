// Many stacks of uneven frame counts and sizes in one launch per phase.
//
// The host turns the stacks into one table of work items, grouped by phase:
//
//   CAL        calibrate a band of rows of one frame into the workspace
//   MEANPART   sum MEAN_ROWS template rows of the calibrated reference
//   MEANFINAL  template mean of the reference
//   SCORE      one tile of partial correlation scores (the stack's tuned launch shape)
//   SSCORE     the same for windows of side <= 5 (one tile of 240 x 256 template pixels per item)
//   SUM        64 candidate scores of one frame from its tile partials
//   PICK       argmax, runner-up, parabola of one frame
//   RECT       common overlap of the stack from its offsets
//   SHIFT      a 16-row strip of one frame's bilinear shift onto the overlap
//   MASK       aligned values that read a bad pixel become NaN, one row of one frame
//   COMB*      sigma-clipped mean of a block of pixel columns of a stack of 49 to 128
//              frames (with a bad-pixel map: the mean of the values that are not missing)
//   FUSE*      for a tile of output pixels of a stack of up to 48 frames: every frame's
//              aligned (and masked) values and the clipped mean, in one pass (one launch
//              per class of up to 16, 32 or 48 frames, without and with a bad-pixel map;
//              such stacks take no SHIFT, MASK or COMB item and keep no aligned frames)
//
// Each phase is one kernel launch with one workgroup per item over all stacks; the
// stream orders the phases, so every dependency is met at a kernel boundary and no
// workgroup waits for another.  The search items go out in an XCD-aware order.  Each
// item calls the same device routines as the stage-wise kernels with the same launch
// shape, so results are bit-identical to them.  Items of the shift and combine phases
// are counted for the whole frame (the overlap is only known on the device) and those
// outside the overlap return at once.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <utility>
#include <vector>

#include "calibrate_core.h"
#include "combine_core.h"
#include "common.h"
#include "fftreg.h"
#include "register_core.h"
#include "register_plan.h"
#include "shift_core.h"

namespace rd {

ScoreArgs make_score_args(const RegPlan &p, const float *ref, const float *frames, const int32_t *centers,
                          const double *mean, double *partial, int32_t W, int32_t H, int32_t N, int32_t R,
                          int32_t Rmax, int32_t tx0, int32_t ty0, int32_t tw, int32_t th, int32_t skip);

constexpr int BATCH_THREADS = 512;

// Plane stride (floats) of the aligned-frame workspace for an overlap of w x h: padded
// to 4 floats so that every frame's plane starts 16-byte aligned.
__host__ __device__ inline int64_t al_plane(int64_t w, int64_t h) { return (w * h + 3) & ~(int64_t)3; }

enum ItemType : int32_t {
    IT_CAL = 0, IT_MEANPART, IT_MEANFINAL, IT_SCORE, IT_SSCORE, IT_SUM, IT_PICK, IT_RECT, IT_SHIFT, IT_MASK,
    IT_COMBDEEP, IT_COMBMISS, IT_FUSE16, IT_FUSE32, IT_FUSE48, IT_FUSE16M, IT_FUSE32M, IT_FUSE48M
};
constexpr int N_PHASES = IT_FUSE48M + 1;

struct Item {
    int32_t type, stack, a, pad;
};

struct StackDev {
    // caller buffers
    const uint16_t *raw;
    int64_t rrp, rfp;
    const float *dark, *flat;
    int64_t crp;
    const float *bias;     // or NULL
    const uint8_t *mask;   // bad-pixel map [H][W] or NULL
    float *out;
    int32_t *out_rect;
    reduce_offset_t *offsets;
    int64_t *n_rej;
    // sizes and parameters
    int32_t W, H, N, ref, R, max_iters, integer_mode, K;
    float ksigma;
    // workspace
    float *cal;           // [N][H][W]
    float *al;            // [N][h][w] aligned frames (room for [N][H][W])
    double *mean_parts;   // [n_mean_parts]
    double *mean;         // [1]
    double *partial;      // [N-1][n_tiles][D*D]
    double *scores;       // [N-1][D*D]
    float *soffs;         // [N][2] offsets applied by the shift
    int32_t *rect;        // [4]
    unsigned long long *slots;  // counters of dropped values (see add_dropped) or NULL
    int32_t n_mean_parts;
    ScoreArgs sa;
};

struct BatchArgs {
    const Item *items;
    const StackDev *stacks;
};

// Counters of dropped values of a large stack (see add_dropped).
constexpr int REJ_SLOTS = 64;
constexpr int REJ_STRIDE = 8;    // 64 bytes apart
constexpr int REJ_TILES = 4096;  // tiles from which on a stack has them
static_assert(REJ_SLOTS <= CAL_BLOCK, "zeroed by one calibration workgroup");

// ---- phase kernels: one workgroup per item ------------------------------------------------
__global__ __launch_bounds__(CAL_BLOCK) void batch_cal(BatchArgs a, int32_t first)
{
    const Item it = a.items[first + blockIdx.x];
    const StackDev &s = a.stacks[it.stack];
    if (it.a == 0) {  // the counts of dropped values start at zero (a launch of its own took 4 us)
        if (s.n_rej && threadIdx.x == 0) *s.n_rej = 0;
        if (s.slots && threadIdx.x < REJ_SLOTS) s.slots[threadIdx.x * REJ_STRIDE] = 0;
    }
    const int64_t i = (int64_t)it.a * CAL_BLOCK + threadIdx.x;
    if (s.W >= CAL_VEC)
        calibrate_group8(s.raw, s.rrp, s.rfp, s.bias, s.dark, s.flat, s.crp, s.cal, s.W, s.H, s.N, i);
    else
        calibrate_pixel(s.raw, s.rrp, s.rfp, s.bias, s.dark, s.flat, s.crp, s.cal, s.W, s.H, s.N, i);
}

__global__ __launch_bounds__(MEAN_THREADS) void batch_meanpart(BatchArgs a, int32_t first)
{
    __shared__ double scratch[MEAN_THREADS / 64];
    const Item it = a.items[first + blockIdx.x];
    const StackDev &s = a.stacks[it.stack];
    const double v = tmpl_part_sum(s.sa.ref, s.W, s.sa.tx0, s.sa.ty0, s.sa.tw, s.sa.th, it.a, scratch);
    if (threadIdx.x == 0) s.mean_parts[it.a] = v;
}

__global__ __launch_bounds__(MEAN_THREADS) void batch_meanfinal(BatchArgs a, int32_t first)
{
    __shared__ double scratch[MEAN_THREADS / 64];
    const Item it = a.items[first + blockIdx.x];
    const StackDev &s = a.stacks[it.stack];
    const double m =
        tmpl_mean_of_parts(s.mean_parts, s.n_mean_parts, (double)s.sa.tw * (double)s.sa.th, scratch);
    if (threadIdx.x == 0) *s.mean = m;
}

// One launch per group of stacks that share a search shape (register block K, threads,
// LDS), with exactly that workgroup size and LDS, as the stage-wise launch uses.
template <int K>
__global__ __launch_bounds__(BATCH_THREADS) void batch_score(BatchArgs a, int32_t first, int32_t count)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const Item it = a.items[first + xcd_logical_id((int32_t)blockIdx.x, count)];
    const StackDev &s = a.stacks[it.stack];
    score_tile<K>(s.sa, it.a, smem);
}

__global__ __launch_bounds__(SMALL_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void batch_score_small(
    BatchArgs a, int32_t first)
{
    __shared__ double red[SMALL_LDS_DOUBLES];
    const Item it = a.items[first + blockIdx.x];
    const StackDev &s = a.stacks[it.stack];
    small_dispatch(s.sa.D, [&](auto Dc) { score_small_tile<decltype(Dc)::value>(s.sa, it.a, red); });
}

__global__ __launch_bounds__(64 * SUM_WAVES) void batch_sum(BatchArgs a, int32_t first)
{
    __shared__ double part[SUM_WAVES][64];
    const Item it = a.items[first + blockIdx.x];
    const StackDev &s = a.stacks[it.stack];
    const int32_t D = s.sa.D;
    const int32_t blocks = (D * D + 63) / 64;
    const int32_t k = it.a / blocks, cb = it.a - k * blocks;
    sum_candidate_block(s.partial + (int64_t)k * s.sa.n_tiles * D * D, s.sa.n_tiles, D, s.R, s.R, 0, 0, cb,
                        s.scores + (int64_t)k * D * D, part);
}

__global__ __launch_bounds__(256) void batch_pick(BatchArgs a, int32_t first)
{
    __shared__ Best scratch[4];
    const Item it = a.items[first + blockIdx.x];
    const StackDev &s = a.stacks[it.stack];
    const int32_t D = s.sa.D, k = it.a;
    const int32_t kf = k + (k >= s.ref ? 1 : 0);
    pick_frame(s.scores + (int64_t)k * D * D, D, s.R, s.R, 0, 0, s.offsets + kf, scratch);
}

__global__ void batch_rect(BatchArgs a, int32_t first)
{
    if (threadIdx.x != 0) return;
    const StackDev &s = a.stacks[a.items[first + blockIdx.x].stack];
    // reference frame: offset 0 by definition
    reduce_offset_t z;
    z.dx = z.dy = 0;
    z.sx = z.sy = 0.0f;
    z.peak = 0.0;
    z.second = -INFINITY;
    z.margin = INFINITY;
    z.flags = 0;
    z.pad = 0;
    s.offsets[s.ref] = z;
    double xl = -1e300, xh = 1e300, yl = -1e300, yh = 1e300;
    for (int32_t k = 0; k < s.N; ++k) {
        float sx = 0.0f, sy = 0.0f;
        if (k != s.ref) {
            const reduce_offset_t o = s.offsets[k];
            sx = s.integer_mode ? (float)o.dx : o.sx;
            sy = s.integer_mode ? (float)o.dy : o.sy;
        }
        s.soffs[2 * k] = sx;
        s.soffs[2 * k + 1] = sy;
        const double lo_x = ceil(-(double)sx), hi_x = floor((double)(s.W - 1) - (double)sx);
        const double lo_y = ceil(-(double)sy), hi_y = floor((double)(s.H - 1) - (double)sy);
        xl = lo_x > xl ? lo_x : xl;
        xh = hi_x < xh ? hi_x : xh;
        yl = lo_y > yl ? lo_y : yl;
        yh = hi_y < yh ? hi_y : yh;
    }
    int32_t r[4] = {0, 0, 0, 0};  // no overlap: empty output
    if (xl <= xh && yl <= yh) {
        r[0] = (int32_t)xl;
        r[1] = (int32_t)yl;
        r[2] = (int32_t)(xh - xl) + 1;
        r[3] = (int32_t)(yh - yl) + 1;
    }
    for (int i = 0; i < 4; ++i) {
        s.rect[i] = r[i];
        s.out_rect[i] = r[i];
    }
}

__global__ __launch_bounds__(SH_BLOCK) void batch_shift(BatchArgs a, int32_t first)
{
    const Item it = a.items[first + blockIdx.x];
    const StackDev &s = a.stacks[it.stack];
    const int32_t x0 = s.rect[0], y0 = s.rect[1], w = s.rect[2], h = s.rect[3];
    const int32_t xblks = (int32_t)ceil_div(s.W, (int64_t)SH_BLOCK * SH_VEC);
    const int32_t strips = (int32_t)ceil_div(s.H, SH_ROWS);
    const int32_t k = it.a / (strips * xblks);
    const int32_t r = it.a - k * strips * xblks;
    const int32_t strip = r / xblks, xblk = r - strip * xblks;
    if (w < 1 || h < 1) return;
    const int vs = shift_vec_store(w, reinterpret_cast<uintptr_t>(s.al));
    const bool aligned = s.W % 4 == 0;
    const int64_t pstride = al_plane(w, h);
    if (s.integer_mode)
        shift_strip<true, SH_VEC>(s.cal, s.al, s.W, s.H, k, s.soffs[2 * k], s.soffs[2 * k + 1], strip, xblk, x0, y0,
                                  w, h, pstride, vs, aligned);
    else
        shift_strip<false, SH_VEC>(s.cal, s.al, s.W, s.H, k, s.soffs[2 * k], s.soffs[2 * k + 1], strip, xblk, x0,
                                   y0, w, h, pstride, vs, aligned);
}

// ---- shift + clipped mean in one pass ---------------------------------------------------
// A tile of FUSE_COLS x FUSE_ROWS output pixels of every frame: first the aligned values, a
// work unit being FUSE_Q columns of all the tile's rows of one frame, whose FUSE_ROWS + 1 tap
// rows are loaded at once (16 and 4 bytes at element alignment) and each used for the two
// output rows it lies between, into an LDS tile [N][FUSE_ROWS][FUSE_COLS]; then one thread per
// pixel runs the first iteration of the clip on its column of the tile, and the few columns
// that drop a value go through the rest of it together (see combine_cols_block), again from
// the tile.  With a bad-pixel map (MASK) the taps' map bytes come in the same way, values
// that read a bad pixel are NaN, and the clip leaves them out.
//
// Bound by the loads of the calibrated frames and, about equally, double arithmetic (a tap's
// conversion, four products and three sums per value, eight operations in the clip).  With
// 256 consecutive pixels per workgroup, two tap rows loaded for each output row, 11 frames of
// 4096x4096 with 3 of 2048x2048 took 490 us, now 376; 23 of 2048x2048 with 30 of 1024x1024 437, now 305;
// 16 masked frames of 6144x6160 as a shift, a mask and a clip (which write and read the
// aligned frames) 2100, now 1020.  Registers are held to what the LDS tile allows in waves:
// 16 frames took 400 us at seven waves per SIMD, 376 at eight.
constexpr int FUSE_COLS = 64;
constexpr int FUSE_ROWS = 4;
constexpr int FUSE_PX = FUSE_COLS * FUSE_ROWS;
constexpr int FUSE_Q = 4;
constexpr int FUSE_QCAP = 64;  // queued columns whose first iteration is kept
static_assert(FUSE_PX == COMB_TILE, "one pixel per thread in the clip");

typedef float fuse_f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t fuse_u32 __attribute__((aligned(1)));

// Aligned values of frame k at FUSE_Q output pixels (u0 + e) of rows v0 .. v0 + FUSE_ROWS - 1
// into dst [row][FUSE_COLS], exactly as shift_strip makes them: taps in rows
// clamp(y0 + v + iy) and the one below (when the vertical fraction is not zero), columns
// clamp(x0 + u + ix) and the one to the right (when the horizontal fraction is not zero),
// from the calibrated frame; and NaN where mask_shifted_kernel would write it.
template <bool MASK, bool INTEGER>
__device__ __forceinline__ void aligned_unit(const StackDev &s, int32_t k, int32_t u0, int32_t v0, int32_t x0,
                                             int32_t y0, float *__restrict__ dst)
{
    constexpr int Q = FUSE_Q, R = FUSE_ROWS;
    const ShiftSetup ss = shift_setup(s.soffs[2 * k], s.soffs[2 * k + 1]);
    const bool step = !INTEGER && ss.a > 0.0;
    const bool down = !INTEGER && ss.b > 0.0;
    const int32_t c0 = x0 + u0 + ss.ix, j0 = y0 + v0 + ss.iy;
    const float *f = s.cal + (int64_t)k * s.W * s.H;
    auto store = [&](float (&o)[Q], uint64_t bad, int r) {
        if constexpr (MASK) {  // byte e of bad: column c0 + e of either tap row
            const uint64_t b = step ? bad | (bad >> 8) : bad;
            if ((uint32_t)b) {
#pragma unroll
                for (int e = 0; e < Q; ++e)
                    if ((b >> (8 * e)) & 0xff) o[e] = __builtin_nanf("");
            }
        }
        *reinterpret_cast<float4 *>(dst + r * FUSE_COLS) = make_float4(o[0], o[1], o[2], o[3]);
    };
    auto values = [&](const float (&t0)[Q + 1], const float (&t1)[Q + 1], uint64_t bad, int r) {
        float o[Q];
#pragma unroll
        for (int e = 0; e < Q; ++e) {
            // the right-hand tap is the next column only when it carries weight
            const float f10 = step ? t0[e + 1] : t0[e], f11 = step ? t1[e + 1] : t1[e];
            o[e] = INTEGER ? t0[e] : bilerp(ss.a, ss.b, t0[e], f10, t1[e], f11);
        }
        store(o, bad, r);
    };
    if (c0 >= 0 && c0 + Q + 1 <= s.W && j0 >= 0) {
        // rows j0 .. j0 + R: the lower tap row of an output row is the upper one of the next
        // (past the last frame row both are that row)
        float t[R + 1][Q + 1];
        uint64_t m[R + 1];
        int64_t at = (int64_t)j0 * s.W + c0;
        if (j0 >= s.H) at = (int64_t)(s.H - 1) * s.W + c0;
#pragma unroll
        for (int i = 0; i <= R; ++i) {
            const fuse_f4 v = *reinterpret_cast<const fuse_f4 *>(f + at);
#pragma unroll
            for (int e = 0; e < Q; ++e) t[i][e] = v[e];
            t[i][Q] = f[at + Q];
            m[i] = 0;
            if constexpr (MASK)
                m[i] = *reinterpret_cast<const fuse_u32 *>(s.mask + at) | ((uint64_t)s.mask[at + Q] << 32);
            at += j0 + i + 1 < s.H ? s.W : 0;
        }
        if (step && down) {
            // bilerp with each tap converted once
            const double ra = 1.0 - ss.a, rb = 1.0 - ss.b;
            const double w00 = __dmul_rn(ra, rb), w10 = __dmul_rn(ss.a, rb), w01 = __dmul_rn(ra, ss.b),
                         w11 = __dmul_rn(ss.a, ss.b);
            double d0[Q + 1], d1[Q + 1];
#pragma unroll
            for (int e = 0; e <= Q; ++e) d0[e] = (double)t[0][e];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float o[Q];
#pragma unroll
                for (int e = 0; e <= Q; ++e) {
                    float f1 = t[r + 1][e];
                    asm volatile("" : "+v"(f1));  // converted here, not all rows beforehand
                    d1[e] = (double)f1;
                }
#pragma unroll
                for (int e = 0; e < Q; ++e)
                    o[e] = (float)__dadd_rn(__dadd_rn(__dadd_rn(__dmul_rn(w00, d0[e]), __dmul_rn(w10, d0[e + 1])),
                                                      __dmul_rn(w01, d1[e])),
                                            __dmul_rn(w11, d1[e + 1]));
                store(o, m[r] | m[r + 1], r);
                __builtin_amdgcn_sched_barrier(0);  // one row at a time: bounds the registers in flight
#pragma unroll
                for (int e = 0; e <= Q; ++e) d0[e] = d1[e];
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float t1[Q + 1];
#pragma unroll
                for (int e = 0; e <= Q; ++e) t1[e] = down ? t[r + 1][e] : t[r][e];
                values(t[r], t1, down ? m[r] | m[r + 1] : m[r], r);
            }
        }
    } else {
#pragma unroll 1
        for (int r = 0; r < R; ++r) {
            const int32_t j = clampi(j0 + r, 0, s.H - 1), j1 = clampi(down ? j + 1 : j, 0, s.H - 1);
            float t0[Q + 1], t1[Q + 1];
            uint64_t bad = 0;
#pragma unroll
            for (int e = 0; e <= Q; ++e) {
                const int32_t c = clampi(c0 + e, 0, s.W - 1);
                t0[e] = f[(int64_t)j * s.W + c];
                t1[e] = f[(int64_t)j1 * s.W + c];
                if constexpr (MASK)
                    bad |= (uint64_t)(s.mask[(int64_t)j * s.W + c] | s.mask[(int64_t)j1 * s.W + c]) << (8 * e);
            }
            values(t0, t1, bad, r);
        }
    }
}

// The number of dropped values: one addition per tile to one address takes 12 ns, longer than
// the rest of the tile (16 masked frames of 6144x6160, 147000 tiles: 1820 us, of which
// 1100 without it), so stacks of many tiles add into REJ_SLOTS counters, which batch_rejected
// adds up after the launch.
__device__ __forceinline__ void add_dropped(const StackDev &s, int32_t item, unsigned total)
{
    unsigned long long *n = s.slots ? s.slots + item % REJ_SLOTS * REJ_STRIDE
                                    : reinterpret_cast<unsigned long long *>(s.n_rej);
    if (total) atomicAdd(n, (unsigned long long)total);
}

__global__ __launch_bounds__(REJ_SLOTS) void batch_rejected(BatchArgs a)
{
    const StackDev &s = a.stacks[blockIdx.x];
    if (!s.slots || !s.n_rej) return;
    unsigned long long v = s.slots[threadIdx.x * REJ_STRIDE];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    // added: stacks may share a count (all are zeroed before any of them adds)
    if (threadIdx.x == 0 && v) atomicAdd(reinterpret_cast<unsigned long long *>(s.n_rej), v);
}

template <int MAXV, bool MASK>
__global__ __launch_bounds__(COMB_TILE) __attribute__((amdgpu_waves_per_eu(MAXV == 16 ? (MASK ? 7 : 8) : 5)))
void batch_fused(BatchArgs a, int32_t first, int32_t count)
{
    extern __shared__ float tile[];  // [MAXV][FUSE_ROWS][FUSE_COLS]
    __shared__ int32_t queue[FUSE_PX];  // pixels that drop values
    __shared__ double qm[FUSE_QCAP], qt[FUSE_QCAP];  // mean, threshold and number of values of their first iteration
    __shared__ int32_t qn[FUSE_QCAP];
    __shared__ int32_t queued;
    // XCD-aware order: the tap row that two rows of tiles share is in one L2
    const Item it = a.items[first + xcd_logical_id((int32_t)blockIdx.x, count)];
    const StackDev &s = a.stacks[it.stack];
    const int32_t x0 = s.rect[0], y0 = s.rect[1], w = s.rect[2], h = s.rect[3];
    const int32_t tiles_x = (w + FUSE_COLS - 1) / FUSE_COLS, tiles = tiles_x * ((h + FUSE_ROWS - 1) / FUSE_ROWS);
    if (w < 1 || h < 1 || it.a >= tiles) return;  // uniform over the workgroup
    const int32_t ty = it.a / tiles_x, u0 = (it.a - ty * tiles_x) * FUSE_COLS, v0 = ty * FUSE_ROWS;
    const int32_t N = __builtin_amdgcn_readfirstlane(s.N);
    const double ksigma = (double)s.ksigma;
    const int t = threadIdx.x;
    constexpr int UNITS = FUSE_COLS / FUSE_Q;  // work units per frame
    const int q = t % UNITS;
    unsigned dropped = 0;
    {
        if (t == 0) queued = 0;
#pragma unroll
        for (int i = 0; i < MAXV * UNITS / COMB_TILE; ++i) {
            const int32_t k = t / UNITS + i * (COMB_TILE / UNITS);
            if (k < N && u0 + q * FUSE_Q < w) {
                float *dst = tile + k * FUSE_PX + q * FUSE_Q;
                if (s.integer_mode)
                    aligned_unit<MASK, true>(s, k, u0 + q * FUSE_Q, v0, x0, y0, dst);
                else
                    aligned_unit<MASK, false>(s, k, u0 + q * FUSE_Q, v0, x0, y0, dst);
            }
        }
        __syncthreads();
        // first iterations; the pixels that drop values go to the queue (see combine_cols_block)
        {
            float x[MAXV];
            each_group<MAXV>(N, [&](int i) { x[i] = tile[i * FUSE_PX + t]; });
            const int32_t u = u0 + t % FUSE_COLS, v = v0 + t / FUSE_COLS;
            ClipState st;
            double m, thr;
            const bool done = clip_first<MAXV, MASK>(RegColumn<MAXV>{x}, N, ksigma, s.max_iters, st, m, thr);
            if (u < w && v < h) {
                if (done) {
                    s.out[(int64_t)v * w + u] = (float)m;
                } else {
                    const int32_t e = atomicAdd(&queued, 1);
                    queue[e] = t;
                    if (e < FUSE_QCAP) {
                        qm[e] = m;
                        qt[e] = thr;
                        qn[e] = st.n;
                    }
                }
            }
        }
        __syncthreads();
        if (t < queued) {
            const int32_t c = queue[t], u = u0 + c % FUSE_COLS, v = v0 + c / FUSE_COLS;
            float x[MAXV];
            each_group<MAXV>(N, [&](int i) { x[i] = tile[i * FUSE_PX + c]; });
            ClipState st;
            double m, thr;
            if (t < FUSE_QCAP) {
                st.lo = -INFINITY;
                st.hi = INFINITY;
                st.n = qn[t];
                m = qm[t];
                thr = qt[t];
            } else {
                clip_first<MAXV, MASK>(RegColumn<MAXV>{x}, N, ksigma, s.max_iters, st, m, thr);
            }
            s.out[(int64_t)v * w + u] =
                clip_rest<MAXV>(RegColumn<MAXV>{x}, N, ksigma, s.max_iters, st, m, thr, dropped);
        }
    }
    if (s.n_rej) {
        const unsigned total = block_sum_u32(dropped);
        if (t == 0) add_dropped(s, it.a, total);
    }
}

// Row v = it.a / N of frame k = it.a % N of a stack with a bad-pixel map (the frames
// of a row consecutive, so that they share the map rows in L2): aligned values that
// read a bad pixel become NaN (missing in the combine).
__global__ __launch_bounds__(256) void batch_mask(BatchArgs a, int32_t first, int32_t count)
{
    // XCD-aware order: the frames of a row, and neighbouring rows, on one XCD (one L2)
    const Item it = a.items[first + xcd_logical_id((int32_t)blockIdx.x, count)];
    const StackDev &s = a.stacks[it.stack];
    const int32_t v = it.a / s.N, k = it.a - v * s.N;
    const int32_t x0 = s.rect[0], y0 = s.rect[1], w = s.rect[2], h = s.rect[3];
    if (v >= h) return;  // uniform over the workgroup
    const ShiftSetup ss = shift_setup(s.soffs[2 * k], s.soffs[2 * k + 1]);
    float *row = s.al + (int64_t)k * al_plane(w, h) + (int64_t)v * w;
    for (int32_t u = threadIdx.x; u < w; u += blockDim.x)
        if (reads_bad_pixel(s.mask, s.W, s.H, ss, s.integer_mode != 0, x0 + u, y0 + v)) row[u] = __builtin_nanf("");
}

// Stacks of 49 - 128 frames (MISS: with a bad-pixel map): the block's columns with all their
// values in registers (see combine_deep); MAXV covers the deepest stack of the phase.
template <int MAXV, bool MISS>
__global__ __launch_bounds__(COMB_TILE) __attribute__((amdgpu_waves_per_eu(3, 3))) void batch_comb_deep(
    BatchArgs a, int32_t first)
{
    const Item it = a.items[first + blockIdx.x];
    const StackDev &s = a.stacks[it.stack];
    const int64_t plane = (int64_t)s.rect[2] * s.rect[3];
    if (it.a >= ceil_div(plane, (int64_t)COMB_TILE)) return;  // uniform over the workgroup
    const unsigned dropped = combine_cols_block<MAXV, 1, MISS>(s.al, plane, al_plane(s.rect[2], s.rect[3]), s.N,
                                                               (double)s.ksigma, s.max_iters, s.out, nullptr, it.a);
    if (s.n_rej) {
        const unsigned total = block_sum_u32(dropped);
        if (threadIdx.x == 0 && total)
            atomicAdd(reinterpret_cast<unsigned long long *>(s.n_rej), (unsigned long long)total);
    }
}

// ---- host side ---------------------------------------------------------------------------
static size_t al(size_t b) { return (b + 255) & ~(size_t)255; }

// Tiles of the fused phase, for the whole frame.
static int64_t fuse_tiles(int32_t W, int32_t H) { return ceil_div(W, FUSE_COLS) * ceil_div(H, FUSE_ROWS); }

struct StackLayout {
    RegPlan plan;
    bool spec;      // registers through row spectra, laid out as fft
    FftLayout fft;
    size_t cal, al, mean_parts, mean, partial, scores, soffs, rect, slots;  // slots: 0 for none
    int32_t count[N_PHASES];
};

struct ScoreGroup {
    int32_t K, threads;
    size_t lds;
    std::vector<int32_t> stacks;  // by decreasing search work
    int32_t first, count;         // item range within the SCORE phase
};

struct BatchLayout {
    std::vector<StackLayout> st;
    size_t items, stacks, total;
    int32_t n_items;
    int32_t first[N_PHASES], count[N_PHASES];
    size_t score_lds;
    size_t spec_ws = 0, spec = 0;  // workspace of the largest spectral search and its offset
    int32_t deep_n = 0;  // deepest stack of the deep combine phase
    int32_t miss_n = 0;  // deepest stack of the combine with missing values
    std::vector<ScoreGroup> groups;
};

static double search_cost(const StackLayout &sl)
{
    const RegPlan &p = sl.plan;
    return (double)sl.count[IT_SCORE] * p.BR * p.TX * p.C;
}

static int validate(const reduce_stack_t *stacks, int32_t n)
{
    for (int32_t i = 0; i < n; ++i) {
        const reduce_stack_t &s = stacks[i];
        const std::string who = "reduce_stack_batch: stack " + std::to_string(i);
        if (!s.raw || !s.dark || !s.flat || !s.out || !s.out_rect || !s.offsets)
            return fail(REDUCE_ERR_NULL, who + ": NULL buffer");
        if (s.W < 1 || s.H < 1 || s.N < 1) return fail(REDUCE_ERR_SHAPE, who + ": W, H, N must be >= 1");
        if (s.raw_row_pitch < s.W || s.raw_frame_pitch < s.raw_row_pitch * (int64_t)(s.H - 1) + s.W ||
            s.cal_row_pitch < s.W)
            return fail(REDUCE_ERR_SHAPE, who + ": pitch smaller than the frame");
        if (s.N > COMB_MAX_N_COLS) return fail(REDUCE_ERR_UNSUPPORTED, who + ": N above 128");
        if (s.ref_index < 0 || s.ref_index >= s.N) return fail(REDUCE_ERR_RANGE, who + ": ref_index out of range");
        if (s.radius < 0 || s.W - 2 * s.radius < 1 || s.H - 2 * s.radius < 1)
            return fail(REDUCE_ERR_RANGE, who + ": radius leaves no template");
        if (!(s.ksigma > 0.0f) || s.max_iters < 0) return fail(REDUCE_ERR_RANGE, who + ": bad clip parameters");
        if (reg_plan(s.W, s.H, s.radius, s.radius).D == 0)
            return fail(REDUCE_ERR_UNSUPPORTED, who + ": radius too large for any launch shape");
        if (s.search != REDUCE_SEARCH_DIRECT && s.search != REDUCE_SEARCH_SPECTRAL)
            return fail(REDUCE_ERR_RANGE, who + ": unknown search");
        if (s.search == REDUCE_SEARCH_SPECTRAL && s.N > 1 &&
            (s.radius < 1 || reduce_register_fft_ws(s.W, s.H, s.N, s.radius) == 0))
            return fail(REDUCE_ERR_UNSUPPORTED, who + ": no search through row spectra for these sizes");
    }
    return REDUCE_OK;
}

// A stack registers through row spectra where it asks for them and, by_rule, where
// reduce_register takes them for its N - 1 searched frames (a stack of one frame has nothing to
// register).  The rule and the launch shapes read the tuner's table, which another thread may change at
// any time, so they are settled here once per call and everything that follows goes by the
// layout.
static BatchLayout layout_of(const reduce_stack_t *stacks, int32_t n, bool by_rule)
{
    BatchLayout L;
    size_t off = 0;
    L.score_lds = 0;
    for (int p = 0; p < N_PHASES; ++p) L.count[p] = 0;
    for (int32_t i = 0; i < n; ++i) {
        const reduce_stack_t &s = stacks[i];
        StackLayout sl{};  // every phase count starts at zero
        sl.plan = reg_plan(s.W, s.H, s.radius, s.radius);
        const RegPlan &p = sl.plan;
        const int64_t fp = (int64_t)s.W * s.H;
        const int32_t nreg = s.N - 1;
        // a stack of up to 48 frames takes the fused phase (no aligned frames in the workspace)
        const bool fuse = s.N <= 48;
        sl.cal = off;
        off += al(sizeof(float) * fp * s.N);
        sl.al = off;
        if (!fuse) off += al(sizeof(float) * al_plane(s.W, s.H) * s.N);
        const int32_t n_mean_parts = (int32_t)ceil_div(s.H - 2 * s.radius, MEAN_ROWS);
        sl.mean_parts = off;
        off += al(sizeof(double) * n_mean_parts);
        sl.mean = off;
        off += 256;
        sl.spec = nreg > 0 &&
                  (s.search == REDUCE_SEARCH_SPECTRAL || (by_rule && spectra_pay(s.W, s.H, nreg, s.radius))) &&
                  fft_layout(s.W, s.H, nreg, s.radius, SPEC_ROUND_BYTES, &sl.fft);
        const int32_t ndir = sl.spec ? 0 : nreg;  // frames of the direct search
        sl.partial = off;
        off += al(sizeof(double) * (size_t)std::max(ndir, 0) * p.n_tiles * p.D * p.D);
        sl.scores = off;
        off += al(sizeof(double) * (size_t)std::max(ndir, 0) * p.D * p.D);
        if (sl.spec) L.spec_ws = std::max(L.spec_ws, sl.fft.total);
        sl.soffs = off;
        off += al(sizeof(float) * 2 * s.N);
        sl.rect = off;
        off += 256;
        sl.slots = fuse && fuse_tiles(s.W, s.H) >= REJ_TILES ? off : 0;
        if (sl.slots) off += al(sizeof(uint64_t) * REJ_SLOTS * REJ_STRIDE);
        sl.count[IT_CAL] = (int32_t)ceil_div(s.W >= CAL_VEC ? cal_groups(s.W) * s.H : fp, CAL_BLOCK);
        sl.count[IT_MEANPART] = ndir > 0 ? n_mean_parts : 0;
        sl.count[IT_MEANFINAL] = ndir > 0 ? 1 : 0;
        sl.count[IT_SCORE] = p.K != 0 ? ndir * p.wg_per_frame : 0;
        sl.count[IT_SSCORE] = p.K == 0 ? ndir * p.wg_per_frame : 0;
        sl.count[IT_SUM] = ndir * (int32_t)ceil_div((int64_t)p.D * p.D, 64);
        sl.count[IT_PICK] = ndir;
        sl.count[IT_RECT] = 1;
        sl.count[IT_SHIFT] =
            fuse ? 0 : s.N * (int32_t)ceil_div(s.H, SH_ROWS) * (int32_t)ceil_div(s.W, (int64_t)SH_BLOCK * SH_VEC);
        // enough items for the whole frame (the overlap is only known on the device); a stack
        // with a bad-pixel map takes the clip that leaves missing values out
        const bool miss = s.mask != nullptr;
        sl.count[IT_MASK] = miss && !fuse ? s.N * s.H : 0;
        if (fuse) {
            const int32_t fb = (int32_t)fuse_tiles(s.W, s.H);
            sl.count[s.N <= 16 ? (miss ? IT_FUSE16M : IT_FUSE16)
                               : s.N <= 32 ? (miss ? IT_FUSE32M : IT_FUSE32) : (miss ? IT_FUSE48M : IT_FUSE48)] = fb;
        }
        const int32_t deep_blocks = s.N > 48 ? (int32_t)ceil_div(fp, (int64_t)COMB_TILE) : 0;
        sl.count[miss ? IT_COMBMISS : IT_COMBDEEP] = deep_blocks;
        if (s.N > 48) (miss ? L.miss_n : L.deep_n) = std::max(miss ? L.miss_n : L.deep_n, s.N);
        for (int q = 0; q < N_PHASES; ++q) L.count[q] += sl.count[q];
        if (ndir > 0 && p.K != 0) L.score_lds = std::max(L.score_lds, p.lds);
        L.st.push_back(sl);
    }
    int64_t total = 0;
    for (int q = 0; q < N_PHASES; ++q) {
        L.first[q] = (int32_t)total;
        total += L.count[q];
    }
    L.n_items = total > INT32_MAX ? -1 : (int32_t)total;
    // search groups by shape, in order of first appearance; stacks within a group by cost
    int32_t next = L.first[IT_SCORE];
    for (int32_t i = 0; i < n; ++i) {
        const StackLayout &sl = L.st[i];
        if (sl.count[IT_SCORE] == 0) continue;
        ScoreGroup *g = nullptr;
        for (ScoreGroup &c : L.groups)
            if (c.K == sl.plan.K && c.threads == sl.plan.threads && c.lds == sl.plan.lds) g = &c;
        if (!g) {
            L.groups.push_back(ScoreGroup{sl.plan.K, sl.plan.threads, sl.plan.lds, {}, 0, 0});
            g = &L.groups.back();
        }
        g->stacks.push_back(i);
    }
    for (ScoreGroup &g : L.groups) {
        std::stable_sort(g.stacks.begin(), g.stacks.end(),
                         [&](int32_t x, int32_t y) { return search_cost(L.st[x]) > search_cost(L.st[y]); });
        g.first = next;
        g.count = 0;
        for (int32_t i : g.stacks) g.count += L.st[i].count[IT_SCORE];
        next += g.count;
    }
    L.spec = off;  // one spectral search at a time
    off += al(L.spec_ws);
    L.items = off;
    off += al(sizeof(Item) * (size_t)std::max<int64_t>(total, 0));
    L.stacks = off;
    off += al(sizeof(StackDev) * (size_t)n);
    L.total = off;
    return L;
}

struct BatchEntry {
    uint64_t hash = 0;
    bool ready = false;
    std::vector<unsigned char> host;  // uploaded descriptor bytes (kept alive with the entry)
};

static std::mutex g_batch_mu;
static std::map<void *, BatchEntry> g_entries;  // by workspace address

static uint64_t fnv1a(const void *p, size_t n, uint64_t h = 1469598103934665603ull)
{
    const unsigned char *b = static_cast<const unsigned char *>(p);
    for (size_t i = 0; i < n; ++i) {
        h ^= b[i];
        h *= 1099511628211ull;
    }
    return h;
}

// Host image of the descriptors of every stack and of the item table.
static int build_descriptors(const reduce_stack_t *stacks, int32_t n, void *ws, const BatchLayout &L,
                             BatchEntry *e)
{
    unsigned char *base = static_cast<unsigned char *>(ws);
    std::vector<StackDev> sd(n);
    for (int32_t i = 0; i < n; ++i) {
        const reduce_stack_t &st = stacks[i];
        const StackLayout &sl = L.st[i];
        StackDev &d = sd[i];
        d.raw = st.raw;
        d.rrp = st.raw_row_pitch;
        d.rfp = st.raw_frame_pitch;
        d.dark = st.dark;
        d.flat = st.flat;
        d.bias = st.bias;
        d.mask = st.mask;
        d.crp = st.cal_row_pitch;
        d.out = st.out;
        d.out_rect = st.out_rect;
        d.offsets = st.offsets;
        d.n_rej = st.n_rej;
        d.slots = sl.slots ? reinterpret_cast<unsigned long long *>(base + sl.slots) : nullptr;
        d.W = st.W;
        d.H = st.H;
        d.N = st.N;
        d.ref = st.ref_index;
        d.R = st.radius;
        d.max_iters = st.max_iters;
        d.integer_mode = st.integer_mode ? 1 : 0;
        d.K = sl.plan.K;
        d.ksigma = st.ksigma;
        d.cal = reinterpret_cast<float *>(base + sl.cal);
        d.al = reinterpret_cast<float *>(base + sl.al);
        d.mean_parts = reinterpret_cast<double *>(base + sl.mean_parts);
        d.mean = reinterpret_cast<double *>(base + sl.mean);
        d.partial = reinterpret_cast<double *>(base + sl.partial);
        d.scores = reinterpret_cast<double *>(base + sl.scores);
        d.soffs = reinterpret_cast<float *>(base + sl.soffs);
        d.rect = reinterpret_cast<int32_t *>(base + sl.rect);
        d.n_mean_parts = (int32_t)ceil_div(st.H - 2 * st.radius, MEAN_ROWS);
        const int32_t R = st.radius;
        const float *ref = d.cal + (int64_t)d.ref * st.W * st.H;
        d.sa = make_score_args(sl.plan, ref, d.cal, nullptr, d.mean, d.partial, st.W, st.H, std::max(st.N - 1, 1), R,
                               R, R, R, st.W - 2 * R, st.H - 2 * R, d.ref);
    }
    // the table, phase by phase; within a phase the largest stacks first
    std::vector<int32_t> order(n);
    for (int32_t i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
        const auto cost = [&](int32_t z) {
            const RegPlan &p = L.st[z].plan;
            return (double)(L.st[z].count[IT_SCORE] + L.st[z].count[IT_SSCORE]) * p.BR * p.TX * p.C +
                   (double)std::accumulate(L.st[z].count + IT_SHIFT, L.st[z].count + N_PHASES, 0);
        };
        return cost(x) > cost(y);
    });
    std::vector<Item> items;
    items.reserve(L.n_items);
    for (int q = 0; q < N_PHASES; ++q) {
        if (q == IT_SCORE) {
            for (const ScoreGroup &g : L.groups)
                for (int32_t i : g.stacks)
                    for (int32_t a = 0; a < L.st[i].count[q]; ++a) items.push_back({q, i, a, 0});
            continue;
        }
        for (int32_t i : order)
            for (int32_t a = 0; a < L.st[i].count[q]; ++a) items.push_back({q, i, a, 0});
    }
    if ((int32_t)items.size() != L.n_items) return fail(REDUCE_ERR_SHAPE, "reduce_stack_batch: item count");
    e->host.assign(L.total - L.items, 0);
    std::memcpy(e->host.data(), items.data(), sizeof(Item) * items.size());
    std::memcpy(e->host.data() + (L.stacks - L.items), sd.data(), sizeof(StackDev) * sd.size());
    return REDUCE_OK;
}

template <typename F>
static void score_dispatch_host(int K, F &&f)
{
    switch (K) {
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 12: f(std::integral_constant<int, 12>{}); break;
    case 17: f(std::integral_constant<int, 17>{}); break;
    case 18: f(std::integral_constant<int, 18>{}); break;
    default: f(std::integral_constant<int, 22>{}); break;
    }
}

static int launch_phases(const reduce_stack_t *stacks, int32_t n, void *ws, const BatchLayout &L, hipStream_t s)
{
    unsigned char *base = static_cast<unsigned char *>(ws);
    BatchArgs a;
    a.items = reinterpret_cast<const Item *>(base + L.items);
    a.stacks = reinterpret_cast<const StackDev *>(base + L.stacks);
    if (L.count[IT_CAL] > 0)
        hipLaunchKernelGGL(batch_cal, dim3(L.count[IT_CAL]), dim3(CAL_BLOCK), 0, s, a, L.first[IT_CAL]);
    if (L.count[IT_MEANPART] > 0)
        hipLaunchKernelGGL(batch_meanpart, dim3(L.count[IT_MEANPART]), dim3(MEAN_THREADS), 0, s, a,
                           L.first[IT_MEANPART]);
    if (L.count[IT_MEANFINAL] > 0)
        hipLaunchKernelGGL(batch_meanfinal, dim3(L.count[IT_MEANFINAL]), dim3(MEAN_THREADS), 0, s, a,
                           L.first[IT_MEANFINAL]);
    if (L.count[IT_SCORE] > 0) {
        for (const ScoreGroup &g : L.groups) {
            ProfScope prof("batch_score", s);  // one record per dispatch
            score_dispatch_host(g.K, [&](auto Kc) {
                constexpr int K = decltype(Kc)::value;
                hipLaunchKernelGGL(batch_score<K>, dim3(g.count), dim3(g.threads), g.lds, s, a, g.first, g.count);
            });
        }
    }
    if (L.count[IT_SSCORE] > 0)
        hipLaunchKernelGGL(batch_score_small, dim3(L.count[IT_SSCORE]), dim3(SMALL_THREADS), 0, s, a,
                           L.first[IT_SSCORE]);
    if (L.count[IT_SUM] > 0)
        hipLaunchKernelGGL(batch_sum, dim3(L.count[IT_SUM]), dim3(64 * SUM_WAVES), 0, s, a, L.first[IT_SUM]);
    if (L.count[IT_PICK] > 0)
        hipLaunchKernelGGL(batch_pick, dim3(L.count[IT_PICK]), dim3(256), 0, s, a, L.first[IT_PICK]);
    // the stacks that register through row spectra, one after the other in the shared space
    for (int32_t i = 0; i < n; ++i) {
        const reduce_stack_t &st = stacks[i];
        if (!L.st[i].spec) continue;
        ProfScope prof("batch_spectral", s);
        const float *cal = reinterpret_cast<const float *>(base + L.st[i].cal);
        const int rc = spectral_search(L.st[i].fft, cal + (int64_t)st.ref_index * st.W * st.H, cal, st.W, st.H,
                                       st.N - 1, st.radius, st.ref_index, st.offsets, nullptr, nullptr,
                                       base + L.spec, s);
        if (rc != REDUCE_OK) return rc;
    }
    hipLaunchKernelGGL(batch_rect, dim3(L.count[IT_RECT]), dim3(64), 0, s, a, L.first[IT_RECT]);
    {
        ProfScope prof("batch_shift", s);
        if (L.count[IT_SHIFT] > 0)
            hipLaunchKernelGGL(batch_shift, dim3(L.count[IT_SHIFT]), dim3(SH_BLOCK), 0, s, a, L.first[IT_SHIFT]);
    }
    if (L.count[IT_MASK] > 0)
        hipLaunchKernelGGL(batch_mask, dim3(L.count[IT_MASK]), dim3(256), 0, s, a, L.first[IT_MASK],
                           L.count[IT_MASK]);
    {
        ProfScope prof("batch_comb", s);
        if (L.count[IT_COMBDEEP] > 0)
            deep_dispatch(L.deep_n, [&](auto Vc) {
                hipLaunchKernelGGL((batch_comb_deep<decltype(Vc)::value, false>), dim3(L.count[IT_COMBDEEP]),
                                   dim3(COMB_TILE), 0, s, a, L.first[IT_COMBDEEP]);
            });
        if (L.count[IT_COMBMISS] > 0)
            deep_dispatch(L.miss_n, [&](auto Vc) {
                hipLaunchKernelGGL((batch_comb_deep<decltype(Vc)::value, true>), dim3(L.count[IT_COMBMISS]),
                                   dim3(COMB_TILE), 0, s, a, L.first[IT_COMBMISS]);
            });
    }
    if (std::any_of(L.count + IT_FUSE16, L.count + N_PHASES, [](int32_t c) { return c > 0; })) {
        ProfScope prof("batch_fused", s);
        const auto fused = [&](int phase, auto maxv, auto masked) {
            constexpr int V = decltype(maxv)::value;
            if (L.count[phase] > 0)
                hipLaunchKernelGGL((batch_fused<V, decltype(masked)::value>), dim3(L.count[phase]), dim3(COMB_TILE),
                                   sizeof(float) * FUSE_PX * V, s, a, L.first[phase], L.count[phase]);
        };
        fused(IT_FUSE16, std::integral_constant<int, 16>{}, std::false_type{});
        fused(IT_FUSE32, std::integral_constant<int, 32>{}, std::false_type{});
        fused(IT_FUSE48, std::integral_constant<int, 48>{}, std::false_type{});
        fused(IT_FUSE16M, std::integral_constant<int, 16>{}, std::true_type{});
        fused(IT_FUSE32M, std::integral_constant<int, 32>{}, std::true_type{});
        fused(IT_FUSE48M, std::integral_constant<int, 48>{}, std::true_type{});
    }
    if (std::any_of(L.st.begin(), L.st.end(), [](const StackLayout &l) { return l.slots != 0; }))
        hipLaunchKernelGGL(batch_rejected, dim3(n), dim3(REJ_SLOTS), 0, s, a);
    return check_launch("reduce_stack_batch");
}

}  // namespace rd

using namespace rd;

extern "C" size_t reduce_stack_batch_ws(const reduce_stack_t *stacks, int32_t n)
{
    if (!stacks || n < 1) return 0;
    if (validate(stacks, n) != REDUCE_OK) return 0;
    return layout_of(stacks, n, true).total;
}

extern "C" int reduce_stack_batch(const reduce_stack_t *stacks, int32_t n, void *ws, size_t ws_bytes, void *stream)
{
    if (!stacks) return fail(REDUCE_ERR_NULL, "reduce_stack_batch: NULL stacks");
    if (n < 1) return fail(REDUCE_ERR_SHAPE, "reduce_stack_batch: no stacks");
    const int v = validate(stacks, n);
    if (v != REDUCE_OK) return v;
    BatchLayout L = layout_of(stacks, n, true);
    if (ws_bytes < L.total) {  // one that holds the direct sums is searched with them, as by reduce_register
        BatchLayout direct = layout_of(stacks, n, false);
        if (direct.total < L.total) L = std::move(direct);
    }
    if (L.n_items < 0) return fail(REDUCE_ERR_UNSUPPORTED, "reduce_stack_batch: too many work items");
    for (int q = 0; q < N_PHASES; ++q)
        if (L.count[q] > 0x7fffffff / 2) return fail(REDUCE_ERR_UNSUPPORTED, "reduce_stack_batch: too many items");
    if (L.score_lds > 65536) return fail(REDUCE_ERR_UNSUPPORTED, "reduce_stack_batch: search tile above 64 KB");
    if (!ws || ws_bytes < L.total)
        return fail(REDUCE_ERR_WORKSPACE, "reduce_stack_batch: workspace needs " + std::to_string(L.total) + " bytes");
    hipStream_t s = as_stream(stream);

    // the host image of the descriptors is rebuilt only when the stacks, their launch
    // shapes or their searches change; it is uploaded into the workspace on every call
    uint64_t h = fnv1a(stacks, sizeof(reduce_stack_t) * (size_t)n);
    for (const StackLayout &sl : L.st) {
        h = fnv1a(&sl.plan, sizeof(RegPlan), h);
        h = fnv1a(&sl.spec, sizeof(sl.spec), h);
    }
    h = fnv1a(&L.total, sizeof(L.total), h);
    std::lock_guard<std::mutex> lk(g_batch_mu);
    BatchEntry &e = g_entries[ws];
    if (!e.ready || e.hash != h) {
        // an earlier call on this workspace may still read the old descriptors
        if (e.ready && hipStreamSynchronize(s) != hipSuccess)
            return fail(REDUCE_ERR_HIP, "reduce_stack_batch: synchronize before new descriptors");
        e = BatchEntry{};
        const int rc = build_descriptors(stacks, n, ws, L, &e);
        if (rc != REDUCE_OK) {
            g_entries.erase(ws);
            return rc;
        }
        e.hash = h;
        e.ready = true;
    }
    if (hipMemcpyAsync(static_cast<unsigned char *>(ws) + L.items, e.host.data(), e.host.size(),
                       hipMemcpyHostToDevice, s) != hipSuccess)
        return fail(REDUCE_ERR_HIP, "reduce_stack_batch: descriptor upload");
    ProfScope prof("stack_batch", s);
    return launch_phases(stacks, n, ws, L, s);
}
