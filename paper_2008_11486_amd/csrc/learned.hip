// Offset-proposal network: input preparation, BF16 matrix-core convolutions with FP32
// accumulation (forward and backward), mean pool, linear head, Huber loss and AdamW.
//
// Network: four 3x3 convolutions with stride 2 and zero padding 1 (2 -> 32 -> 32 -> 32
// -> 32 channels), each followed by ReLU; the mean over all pixels of the last
// activation; a linear layer 32 -> 2 giving (dx, dy) in downsampled pixels.
// Activations are [B][H][W][C] bfloat16 (channels contiguous).  Master parameters
// are one flat FP32 vector W1 b1 W2 b2 W3 b3 W4 b4 Wl bl with conv weights
// W[t][cin][cout], t = 3 ky + kx.
//
// Convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16: a wave computes 16
// output pixels x 16 output channels per instruction with K = 32 (one tap x 32 input
// channels, or all 18 (tap, channel) pairs of the 2-channel input layer).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "common.h"
#include "learned.h"

namespace rd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest, ties to even
__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);
    u = u + 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ bf16x8 load8(const uint16_t *p)
{
    const uint4 v = *reinterpret_cast<const uint4 *>(p);
    return __builtin_bit_cast(bf16x8, v);
}

// ---- network input: 4x4 block mean, standardisation, asinh, bfloat16 --------------------
constexpr int DS_BLOCK = 256;

__device__ __forceinline__ double block_sum_d(double v, double *scratch)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < DS_BLOCK / 64; ++i) t += scratch[i];
    __syncthreads();
    return t;
}

// One pass per frame: the 4x4 block means (summed in double, stored as float), and per
// workgroup the sums of d = v - c and d^2, with c the frame's first block mean (a shift
// that keeps the one-pass variance free of cancellation; every workgroup recomputes it,
// the first one stores it).
__device__ __forceinline__ double box4(const float *__restrict__ src, int32_t W)
{
    double s = 0.0;
    for (int y = 0; y < 4; ++y)
        for (int x = 0; x < 4; ++x) s += (double)src[(int64_t)y * W + x];
    return s / 16.0;
}

__global__ __launch_bounds__(DS_BLOCK) void ds_boxmean(const float *__restrict__ frames, int32_t W, int32_t H,
                                                       float *__restrict__ m, double *__restrict__ part,
                                                       double *__restrict__ shift)
{
    __shared__ double scratch[DS_BLOCK / 64];
    const int32_t w = W / 4, h = H / 4;
    const int64_t n = (int64_t)w * h;
    const int32_t f = blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * DS_BLOCK + threadIdx.x;
    const float *frame = frames + (int64_t)f * W * H;
    const double c = box4(frame, W);
    double d = 0.0;
    if (i < n) {
        const int32_t jy = (int32_t)(i / w), jx = (int32_t)(i - (int64_t)jy * w);
        const double v = box4(frame + (int64_t)(4 * jy) * W + 4 * jx, W);
        m[(int64_t)f * n + i] = (float)v;
        d = v - c;
    }
    const double t1 = block_sum_d(d, scratch);
    const double t2 = block_sum_d(d * d, scratch);
    if (threadIdx.x == 0) {
        double *pp = part + 2 * ((int64_t)f * gridDim.x + blockIdx.x);
        pp[0] = t1;
        pp[1] = t2;
        if (blockIdx.x == 0) shift[f] = c;
    }
}

// Per frame: mean = c + S1 / n and population sigma = sqrt(S2 / n - (S1 / n)^2), the
// partial sums added over workgroups in a fixed order.
__global__ __launch_bounds__(DS_BLOCK) void ds_finish(const double *__restrict__ part, int32_t nparts, double n,
                                                      const double *__restrict__ shift, double *__restrict__ mean,
                                                      double *__restrict__ sd)
{
    __shared__ double scratch[DS_BLOCK / 64];
    const int32_t f = blockIdx.x;
    double s1 = 0.0, s2 = 0.0;
    for (int32_t i = threadIdx.x; i < nparts; i += DS_BLOCK) {
        s1 += part[2 * ((int64_t)f * nparts + i)];
        s2 += part[2 * ((int64_t)f * nparts + i) + 1];
    }
    s1 = block_sum_d(s1, scratch);
    s2 = block_sum_d(s2, scratch);
    if (threadIdx.x == 0) {
        const double a = s1 / n;
        mean[f] = shift[f] + a;
        sd[f] = sqrt(fmax(s2 / n - a * a, 0.0));
    }
}

// asinh(z) in float, within 2^-19 of itself for 2^-60 <= |z| <= 2^30: below 1/2 the Taylor
// series through z^13 (the first term left out is 2^-20.1 of the result at most), above it
// log2 of z + sqrt(z^2 + 1) (at least 0.69, so its half ulp and those under it stay relative).
__device__ __forceinline__ float asinh_fast(float z)
{
    const float a = fabsf(z), q = z * z;
    float p = 10395.0f / 599040.0f;
    p = fmaf(p, q, -945.0f / 42240.0f);
    p = fmaf(p, q, 105.0f / 3456.0f);
    p = fmaf(p, q, -15.0f / 336.0f);
    p = fmaf(p, q, 3.0f / 40.0f);
    p = fmaf(p, q, -1.0f / 6.0f);
    const float small = fmaf(a * q, p, a);
    const float large = 0.693147181f * __builtin_amdgcn_logf(a + __builtin_amdgcn_sqrtf(q + 1.0f));
    return copysignf(a < 0.5f ? small : large, z);
}

// Four values per thread: standardise, asinh, round to bfloat16.  The result is that of double
// arithmetic rounded to float and to bfloat16, to the bit: both roundings are monotone,
// so where the ends of an interval that is four times as wide as the float evaluation's
// error round alike, every value inside it does; the few others (1 in 500), and values
// outside the evaluation's range, go through the double function, whose 500
// double-precision instructions bound this kernel before (220 us for 32 images of 1024x1024; now 62,
// of which memory takes 41).
__global__ __launch_bounds__(DS_BLOCK) void ds_normalize(const float *__restrict__ m, int64_t n,
                                                         const double *__restrict__ mean,
                                                         const double *__restrict__ sd, uint16_t *__restrict__ out)
{
    const int32_t f = blockIdx.y;
    const int64_t i0 = ((int64_t)blockIdx.x * DS_BLOCK + threadIdx.x) * 4;
    if (i0 >= n) return;
    const double s = sd[f], mu = mean[f], inv = 1.0 / s;
    const float *src = m + (int64_t)f * n;
    uint16_t *dst = out + (int64_t)f * n;
    const int cnt = (int)min((int64_t)4, n - i0);
    const bool vec = cnt == 4 && n % 4 == 0;
    float v[4];
    if (vec) {
        const float4 u = *reinterpret_cast<const float4 *>(src + i0);
        v[0] = u.x;
        v[1] = u.y;
        v[2] = u.z;
        v[3] = u.w;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = src[i0 + min(j, cnt - 1)];
    }
    uint16_t z[4];
    uint32_t open = 0;  // the values that go through the double function
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float x = (float)(((double)v[j] - mu) * inv);
        const float w = asinh_fast(x), e = fabsf(w) * 0x1p-18f;
        const uint16_t lo = f2bf(w - e), hi = f2bf(w + e);
        z[j] = lo;
        // (a zero sigma gives infinities or NaN here)
        if (!(fabsf(x) >= 0x1p-60f && fabsf(x) <= 0x1p30f && lo == hi)) open |= 1u << j;
    }
    while (open) {
        const int k = __builtin_ctz(open);
        open &= open - 1;
        const float u = k == 0 ? v[0] : k == 1 ? v[1] : k == 2 ? v[2] : v[3];
        const uint16_t r = f2bf((float)asinh(s > 0.0 ? ((double)u - mu) / s : 0.0));
#pragma unroll
        for (int j = 0; j < 4; ++j) z[j] = j == k ? r : z[j];
    }
    if (vec && (reinterpret_cast<uintptr_t>(out) & 7u) == 0) {
        *reinterpret_cast<uint2 *>(dst + i0) = make_uint2(z[0] | ((uint32_t)z[1] << 16), z[2] | ((uint32_t)z[3] << 16));
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j < cnt) dst[i0 + j] = z[j];
    }
}

// ---- weight packing ---------------------------------------------------------------------
// Forward operand of layer l: [ksteps][32 cout][32 k] bf16, k = input channel of tap
// kstep (3x3 layers with 32 inputs) or k = 2 t + c for the 2-channel input layer
// (one kstep, k >= 18 zero).  Backward-data operand of layers 2..4: [9][32 cin][32 cout].
__global__ void pack_weights(const float *__restrict__ params, uint16_t *__restrict__ wf,
                             uint16_t *__restrict__ wd)
{
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // layer 1: 32 x 32 forward entries
    if (tid < 1024) {
        const int32_t co = (int32_t)(tid / 32), k = (int32_t)(tid % 32);
        float v = 0.0f;
        if (k < 18) v = params[(k >> 1) * 2 * CNN_CH + (k & 1) * CNN_CH + co];
        wf[tid] = f2bf(v);
        return;
    }
    int64_t r = tid - 1024;
    if (r < 3 * 9 * 1024) {  // layers 2..4, forward layout
        const int32_t l = (int32_t)(r / (9 * 1024));
        const int32_t rem = (int32_t)(r % (9 * 1024));
        const int32_t t = rem / 1024, co = (rem % 1024) / 32, ci = rem % 32;
        const float *w = params + cnn_weight_offset(l + 1);
        wf[1024 + r] = f2bf(w[(t * CNN_CH + ci) * CNN_CH + co]);
        return;
    }
    r -= 3 * 9 * 1024;
    if (r < 3 * 9 * 1024) {  // layers 2..4, backward-data layout [t][cin][cout]
        const int32_t l = (int32_t)(r / (9 * 1024));
        const int32_t rem = (int32_t)(r % (9 * 1024));
        const float *w = params + cnn_weight_offset(l + 1);
        wd[r] = f2bf(w[rem]);
    }
}

// ---- convolution forward ---------------------------------------------------------------------
// The weights are the matrix instruction's first operand and 16 consecutive output pixels of a
// row the second, so a lane ends up with one pixel; the weight rows are dealt so that its
// 2 x 4 values are eight consecutive channels, one 16-byte store, and a wave writes 1 KB in
// one piece without a trip through LDS.  Accumulation order: taps in order, one instruction
// per tap and 16 channels.
//
// Channel of row r of the first (and, + 4, of the second) weight tile, so that the lane with
// rows 4 g .. 4 g + 3 of both holds channels 8 g .. 8 g + 7.
__device__ __forceinline__ int tile_channel(int r) { return 8 * (r >> 2) + (r & 3); }

__device__ __forceinline__ uint4 pack8(const float (&v)[8])
{
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = (uint32_t)f2bf(v[2 * j]) | ((uint32_t)f2bf(v[2 * j + 1]) << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// bias, ReLU, bfloat16
__device__ __forceinline__ uint4 relu8(const f32x4 &acc0, const f32x4 &acc1, const float (&b)[8])
{
    float v[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] = fmaxf(acc0[j] + b[j], 0.0f);
        v[4 + j] = fmaxf(acc1[j] + b[4 + j], 0.0f);
    }
    return pack8(v);
}

// One row of a [H][W][32] plane as a buffer: reads past either end give zero and writes there
// are dropped, so the loops over rows have no branches, whose joins would wait for
// every load in flight.  A row that does not exist is an empty buffer.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_row(const uint16_t *plane, int32_t row, int32_t H, int32_t W)
{
    const bool in = row >= 0 && row < H;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(plane) + (int64_t)min(max(row, 0), H - 1) * W * CNN_CH,
                                             0, in ? W * (CNN_CH * 2) : 0, 0x00027000);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 row_load8(__amdgpu_buffer_rsrc_t row, uint32_t off)
{
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(row, off, 0, 0));
}

__device__ __forceinline__ void row_store8(__amdgpu_buffer_rsrc_t row, uint32_t off, uint4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), row, off, 0, 0);
}

constexpr uint32_t ROW_NONE = 0x80000000u;  // an offset past the end of every row

constexpr int CONV_ROWS = 8;  // output rows per workgroup; its four waves take 16 columns each

// Layer 1 (two input channels): the input rows of the tile are staged in LDS with both
// channels in one word, so a tap is one word and the pixel operand (18 of 32 products, the
// rest zeros) four LDS reads.  Bound by the stores; 16 pairs of 1024x1024 took 140 us with one
// row per workgroup and the transposed result sent through LDS, now 67 (268 MB written).
__global__ __launch_bounds__(256) void conv_first(const uint16_t *__restrict__ ref, int64_t ref_stride,
                                                  const uint16_t *__restrict__ img, int32_t H, int32_t W,
                                                  const uint16_t *__restrict__ wf, const float *__restrict__ bias,
                                                  uint16_t *__restrict__ y)
{
    constexpr int XC = 2 * 64 + 1;        // staged input columns
    constexpr int XR = 2 * CONV_ROWS + 1;  // and rows
    __shared__ uint32_t in2[XR * XC + 3];
    const int32_t Ho = (H + 1) / 2, Wo = (W + 1) / 2;
    const int32_t b = blockIdx.z, oy0 = blockIdx.y * CONV_ROWS, gx0 = blockIdx.x * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, kg = lane >> 4;
    const bf16x8 w0 = load8(wf + tile_channel(m) * 32 + kg * 8);
    const bf16x8 w1 = load8(wf + (tile_channel(m) + 4) * 32 + kg * 8);
    float bv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) bv[j] = bias[8 * kg + j];
    const uint16_t *rb = ref + (int64_t)b * ref_stride, *ib = img + (int64_t)b * H * W;

    // input rows 2 oy0 - 1 + r, columns 2 gx0 - 1 + col
    constexpr int PER = (XR * XC + 255) / 256;
    uint16_t va[PER], vb[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = i * 256 + threadIdx.x, r = e / XC, col = e - r * XC;
        const int32_t iy = 2 * oy0 + r - 1, ix = 2 * gx0 - 1 + col;
        const bool in = e < XR * XC && iy >= 0 && iy < H && ix >= 0 && ix < W;
        const int64_t p = in ? (int64_t)iy * W + ix : 0;
        va[i] = rb[p];
        vb[i] = ib[p];
        if (!in) va[i] = vb[i] = 0;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = i * 256 + threadIdx.x;
        if (e < XR * XC) in2[e] = (uint32_t)va[i] | ((uint32_t)vb[i] << 16);
    }
    __syncthreads();
    const int32_t ox = gx0 + 16 * wave + m;
    int at[4];  // the lane's taps 4 kg .. 4 kg + 3
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = min(4 * kg + j, 8);
        at[j] = (t / 3) * XC + 2 * (16 * wave + m) + t % 3;
    }
#pragma unroll
    for (int r = 0; r < CONV_ROWS; ++r) {
        const int32_t oy = oy0 + r;
        uint32_t e[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            e[j] = in2[2 * r * XC + at[j]];
            if (4 * kg + j > 8) e[j] = 0;
        }
        const bf16x8 a = __builtin_bit_cast(bf16x8, make_uint4(e[0], e[1], e[2], e[3]));
        f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, a, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, a, acc1, 0, 0, 0);
        row_store8(plane_row(y + (int64_t)b * Ho * Wo * CNN_CH, oy, Ho, Wo), (uint32_t)ox * 64 + kg * 16,
                   relu8(acc0, acc1, bv));
    }
}

// Layers 2 - 4 (32 input channels): a wave keeps the weights of all nine taps in registers and
// walks down CONV_ROWS output rows; of the three input rows of an output row it keeps the
// last for the next and has that one's other two loaded before this one's products.  Bound by
// memory: the three layers of 16 pairs of 1024x1024 took 170 us a row and four pixel
// groups per workgroup (nine loads per row, the result through LDS), now 115 (440 MB).
__global__ __launch_bounds__(256) void conv_next(const uint16_t *__restrict__ x, int32_t H, int32_t W,
                                                 const uint16_t *__restrict__ wf, const float *__restrict__ bias,
                                                 uint16_t *__restrict__ y)
{
    const int32_t Ho = (H + 1) / 2, Wo = (W + 1) / 2;
    const int32_t b = blockIdx.z, oy0 = blockIdx.y * CONV_ROWS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, kg = lane >> 4;
    const int32_t ox = blockIdx.x * 64 + 16 * wave + m;
    bf16x8 w0[9], w1[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        w0[t] = load8(wf + (t * 32 + tile_channel(m)) * 32 + kg * 8);
        w1[t] = load8(wf + (t * 32 + tile_channel(m) + 4) * 32 + kg * 8);
    }
    float bv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) bv[j] = bias[8 * kg + j];
    const uint16_t *xb = x + (int64_t)b * H * W * CNN_CH;
    uint16_t *yb = y + (int64_t)b * Ho * Wo * CNN_CH;
    const uint32_t o1 = (uint32_t)ox * 128 + kg * 16;  // column 2 ox; 64 bytes to a pixel
    const uint32_t o0 = ox > 0 ? o1 - 64 : ROW_NONE;
    auto load_row = [&](int32_t iy, bf16x8 (&v)[3]) {  // columns 2 ox - 1 .. 2 ox + 1
        const __amdgpu_buffer_rsrc_t row = plane_row(xb, iy, H, W);
        v[0] = row_load8(row, o0);
        v[1] = row_load8(row, o1);
        v[2] = row_load8(row, o1 + 64);
    };
    bf16x8 top[3], mid[3], bot[3];
    load_row(2 * oy0 - 1, top);
    load_row(2 * oy0, mid);
    load_row(2 * oy0 + 1, bot);
#pragma unroll
    for (int r = 0; r < CONV_ROWS; ++r) {
        const int32_t oy = oy0 + r;
        bf16x8 mid_n[3], bot_n[3];
        if (r + 1 < CONV_ROWS) {
            load_row(2 * oy + 2, mid_n);
            load_row(2 * oy + 3, bot_n);
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const bf16x8 a = t < 3 ? top[t % 3] : t < 6 ? mid[t % 3] : bot[t % 3];
            acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0[t], a, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[t], a, acc1, 0, 0, 0);
        }
        row_store8(plane_row(yb, oy, Ho, Wo), (uint32_t)ox * 64 + kg * 16, relu8(acc0, acc1, bv));
        if (r + 1 < CONV_ROWS) {
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                top[kx] = bot[kx];
                mid[kx] = mid_n[kx];
                bot[kx] = bot_n[kx];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ---- mean pool and linear head ----------------------------------------------------------------
// pool_partial: workgroup (chunk, image) sums POOL_CHUNK pixels of every channel (eight
// pixel groups, then the groups in order, in double).  pool_head: one workgroup per
// image adds the chunk sums in chunk order, pool[c] = sum / P, then pred = Wl pool + bl.
constexpr int POOL_CHUNK = 128;

__global__ __launch_bounds__(256) void pool_partial(const uint16_t *__restrict__ x4, int64_t P, int32_t nchunk,
                                                    double *__restrict__ part)
{
    __shared__ double red[8][CNN_CH];
    const int32_t b = blockIdx.y, ch = blockIdx.x;
    const int c = threadIdx.x % CNN_CH, g = threadIdx.x / CNN_CH;  // 8 pixel groups
    const int64_t p0 = (int64_t)ch * POOL_CHUNK, p1 = min(p0 + POOL_CHUNK, P);
    double s = 0.0;
    for (int64_t p = p0 + g; p < p1; p += 8) s += (double)bf2f(x4[((int64_t)b * P + p) * CNN_CH + c]);
    red[g][c] = s;
    __syncthreads();
    if (threadIdx.x < CNN_CH) {
        double t = 0.0;
        for (int i = 0; i < 8; ++i) t += red[i][threadIdx.x];
        part[((int64_t)b * nchunk + ch) * CNN_CH + threadIdx.x] = t;
    }
}

__global__ __launch_bounds__(64) void pool_head(const double *__restrict__ part, int32_t nchunk, int64_t P,
                                                const float *__restrict__ params, double *__restrict__ pool,
                                                float *__restrict__ pred)
{
    __shared__ double pl[CNN_CH];
    const int32_t b = blockIdx.x;
    if (threadIdx.x < CNN_CH) {
        double t = 0.0;
        for (int32_t i = 0; i < nchunk; ++i) t += part[((int64_t)b * nchunk + i) * CNN_CH + threadIdx.x];
        pl[threadIdx.x] = t / (double)P;
        pool[b * CNN_CH + threadIdx.x] = pl[threadIdx.x];
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const int j = threadIdx.x;
        const float *wl = params + cnn_head_offset();
        double v = (double)wl[2 * CNN_CH + j];
        for (int cc = 0; cc < CNN_CH; ++cc) v += pl[cc] * (double)wl[j * CNN_CH + cc];
        pred[2 * b + j] = (float)v;
    }
}

// ---- loss and head backward ------------------------------------------------------------------
// One workgroup: Huber loss, head gradients (double sums over the batch in order) and
// the gradient with respect to the pooled features.
__global__ __launch_bounds__(256) void head_backward(const float *__restrict__ pred, const float *__restrict__ target,
                                                     int32_t B, double delta, const double *__restrict__ pool,
                                                     const float *__restrict__ params, float *__restrict__ loss,
                                                     float *__restrict__ grad, double *__restrict__ dpool)
{
    __shared__ double dpred[2 * 1024];
    __shared__ double lpart[256];
    const float *wl = params + cnn_head_offset();
    double l = 0.0;
    for (int32_t i = threadIdx.x; i < 2 * B; i += 256) {
        const double e = (double)pred[i] - (double)target[i];
        const double ae = fabs(e);
        l += ae <= delta ? 0.5 * e * e : delta * (ae - 0.5 * delta);
        dpred[i] = (ae <= delta ? e : (e > 0 ? delta : -delta)) / (2.0 * B);
    }
    lpart[threadIdx.x] = l;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < 256; ++i) t += lpart[i];
        *loss = (float)(t / (2.0 * B));
    }
    float *gh = grad + cnn_head_offset();
    if (threadIdx.x < 2 * CNN_CH) {  // dWl[j][c]
        const int j = threadIdx.x / CNN_CH, c = threadIdx.x % CNN_CH;
        double sacc = 0.0;
        for (int32_t b = 0; b < B; ++b) sacc += dpred[2 * b + j] * pool[b * CNN_CH + c];
        gh[j * CNN_CH + c] = (float)sacc;
    } else if (threadIdx.x < 2 * CNN_CH + 2) {  // dbl[j]
        const int j = threadIdx.x - 2 * CNN_CH;
        double sacc = 0.0;
        for (int32_t b = 0; b < B; ++b) sacc += dpred[2 * b + j];
        gh[2 * CNN_CH + j] = (float)sacc;
    }
    for (int32_t i = threadIdx.x; i < B * CNN_CH; i += 256) {
        const int32_t b = i / CNN_CH, c = i % CNN_CH;
        dpool[i] = dpred[2 * b] * (double)wl[c] + dpred[2 * b + 1] * (double)wl[CNN_CH + c];
    }
}

// Gradient of the last pre-activation: the pool's 1/P spread, masked by ReLU.
__global__ void pool_backward(const uint16_t *__restrict__ x4, int64_t P, int32_t B,
                              const double *__restrict__ dpool, uint16_t *__restrict__ dz)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)B * P * CNN_CH) return;
    const int32_t c = (int32_t)(i % CNN_CH);
    const int32_t b = (int32_t)(i / (P * CNN_CH));
    const double g = bf2f(x4[i]) > 0.0f ? dpool[b * CNN_CH + c] / (double)P : 0.0;
    dz[i] = f2bf((float)g);
}

// ---- weight gradient ---------------------------------------------------------------------------
// dW[t][ci][co] = sum over output pixels of X[input pixel of tap t][ci] * dZ[pixel][co], the
// pixels along K: A[m = co][k = pixel], B[k = pixel][n = ci] (n = (ky, kx, ci) for the
// 2-channel input layer).  Bound by HBM (X and dZ read once).  Both operands lie with their
// channels contiguous, so K has to be brought together first: a thread loads the same 8
// channels of 4 pixels (16 bytes each) and stores them to LDS as [channel][pixel], 4 pixels
// per 8-byte store, and a fragment is then one 16-byte LDS read (the form that read eight
// 2-byte values per fragment, and two-byte global loads for the tiles, was bound by those:
// 4.83 -> 0.27 ms for a batch of 16 of 1024x1024, all layers; reading X and dZ
// once takes 0.16 ms).
//
// A workgroup holds WG_GRP groups of four waves; a group walks down the output rows of
// strips of WG_PX output pixels, in its own LDS.  The input of a row of outputs is three
// rows, kept by row: even row 2 oy, odd rows 2 oy - 1 and 2 oy + 1 (the second is the
// first of the next step, so a step loads two), each split by column parity, so that the
// pixels of tap kx = 1 (even columns) and of kx = 2 (odd columns) are consecutive.  kx = 0
// reads the odd columns one pixel earlier: it takes the same fragment with dZ one pixel
// later instead (dZ is held twice, at p and at p + 1), so every fragment is aligned.  The
// next step's loads are in flight while a step is computed.  The groups' sums are added in
// order and one partial is written per workgroup; wgrad_reduce adds the partials in order.
constexpr int WG_PX = 64;               // output pixels per strip row
constexpr int WG_GRP = 4;               // groups of 256 threads per workgroup
constexpr int WG_PITCH = WG_PX + 8;     // LDS row of one channel (16-byte rows, spread over the banks)

template <int CIN>
__global__ __launch_bounds__(256 * WG_GRP) void wgrad(const uint16_t *__restrict__ x, const uint16_t *__restrict__ ref,
                                                      int64_t ref_stride, const uint16_t *__restrict__ img, int32_t B,
                                                      int32_t H, int32_t W, const uint16_t *__restrict__ dz,
                                                      float *__restrict__ wpart, float *__restrict__ bpart)
{
    constexpr int NACC = CIN == 2 ? 1 : 9;
    constexpr int NW = 9 * CIN * CNN_CH;
    struct Group {
        uint16_t x[3][2][CIN][WG_PITCH];     // [odd row | odd row | even row][column parity][ci][pixel]
        uint16_t z[2][CNN_CH][WG_PITCH];     // [at p | at p + 1][co][pixel]
    };
    __shared__ __align__(16) Group lds[WG_GRP];
    static_assert(sizeof(lds) >= sizeof(float) * (NW + 16 * CNN_CH), "the sums of the groups reuse the tiles");
    const int grp = threadIdx.x >> 8, t = threadIdx.x & 255;
    const int lane = t & 63, wave = t >> 6, m = lane & 15, kg = lane >> 4;
    Group &g = lds[grp];
    const int32_t Ho = (H + 1) / 2, Wo = (W + 1) / 2;
    const int32_t nxb = (Wo + WG_PX - 1) / WG_PX;
    const int64_t steps = (int64_t)B * nxb * Ho;  // (image, strip, output row), the row fastest
    const int64_t ngrp = (int64_t)gridDim.x * WG_GRP;
    const int64_t per = (steps + ngrp - 1) / ngrp;
    const int64_t s0 = ((int64_t)blockIdx.x * WG_GRP + grp) * per;

    // what a thread loads of a step: of the input rows 2 oy (row 0) and 2 oy + 1 (row 1), and
    // of dZ.  CIN = 32: channels 8 oct .. of the pixels 4 quad .. 4 quad + 3 of one column
    // parity of one row; CIN = 2: one pixel of each row.
    const int oct = t & 3, par = (t >> 2) & 1, quad = (t >> 3) & 15, row = t >> 7;
    const int zv = (t >> 6) & 1, zquad = (t >> 2) & 15;  // threads 0 .. 127 load dZ at p + zv
    struct Step {
        int32_t b, oy, ox0;
        bool ok;
    };
    auto step_at = [&](int64_t it) {
        const int64_t s = s0 + it;
        Step q;
        q.ok = it < per && s < steps;
        const int64_t strip = q.ok ? s / Ho : 0;
        q.oy = q.ok ? (int32_t)(s - strip * Ho) : 0;
        q.b = (int32_t)(strip / nxb);
        q.ox0 = (int32_t)(strip - (int64_t)q.b * nxb) * WG_PX;
        return q;
    };
    uint4 xr[CIN == 2 ? 1 : 4], zr[4];
    uint16_t x2[2];
    auto load_x32 = [&](const Step &q, int32_t iy, uint4 (&r)[CIN == 2 ? 1 : 4]) {
#pragma unroll
        for (int j = 0; j < (CIN == 2 ? 0 : 4); ++j) {
            const int32_t ix = 2 * (q.ox0 + 4 * quad + j) + par;
            r[j] = make_uint4(0u, 0u, 0u, 0u);
            if (q.ok && iy >= 0 && iy < H && ix < W)
                r[j] = *reinterpret_cast<const uint4 *>(x + (((int64_t)q.b * H + iy) * W + ix) * CNN_CH + oct * 8);
        }
    };
    auto load_x2 = [&](const Step &q, int32_t iy) -> uint16_t {
        const int32_t ix = 2 * q.ox0 + (t & 127);
        if (!(q.ok && iy >= 0 && iy < H && ix < W)) return 0;
        const int64_t p = (int64_t)iy * W + ix;
        return t < 128 ? ref[(int64_t)q.b * ref_stride + p] : img[(int64_t)q.b * H * W + p];
    };
    auto load_step = [&](const Step &q) {
        if constexpr (CIN == 2) {
            x2[0] = load_x2(q, 2 * q.oy);
            x2[1] = load_x2(q, 2 * q.oy + 1);
        } else {
            load_x32(q, 2 * q.oy + row, xr);
        }
        if (t < 128) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int32_t p = q.ox0 + 4 * zquad + j + zv;
                zr[j] = make_uint4(0u, 0u, 0u, 0u);
                if (q.ok && p < Wo)
                    zr[j] = *reinterpret_cast<const uint4 *>(dz + (((int64_t)q.b * Ho + q.oy) * Wo + p) * CNN_CH +
                                                             oct * 8);
            }
        }
    };
    // four pixels of eight channels -> eight 8-byte stores [channel][4 pixels]
    auto put8 = [&](const uint4 (&r)[4], uint16_t *dst) {
        const uint32_t w[4][4] = {{r[0].x, r[0].y, r[0].z, r[0].w}, {r[1].x, r[1].y, r[1].z, r[1].w},
                                  {r[2].x, r[2].y, r[2].z, r[2].w}, {r[3].x, r[3].y, r[3].z, r[3].w}};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;  // high or low halves of two words
            *reinterpret_cast<uint2 *>(dst + c * WG_PITCH) =
                make_uint2(__builtin_amdgcn_perm(w[1][c >> 1], w[0][c >> 1], sel),
                           __builtin_amdgcn_perm(w[3][c >> 1], w[2][c >> 1], sel));
        }
    };

    f32x4 acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) bsum[c] = 0.0f;

    Step q = step_at(0);
    load_step(q);
    for (int64_t it = 0; it < per; ++it) {
        __syncthreads();  // the previous step's fragments have been read
        // odd row 2 oy - 1 in slot oy & 1, odd row 2 oy + 1 in the other, even row in slot 2
        const int s_up = q.oy & 1, s_dn = s_up ^ 1;
        if constexpr (CIN == 2) {
            g.x[2][t & 1][t >> 7][(t & 127) >> 1] = x2[0];
            g.x[s_dn][t & 1][t >> 7][(t & 127) >> 1] = x2[1];
        } else {
            put8(xr, &g.x[row ? s_dn : 2][par][oct * 8][4 * quad]);
        }
        if (t < 128) {
            put8(zr, &g.z[zv][oct * 8][4 * zquad]);
            if (zv == 0) {
                const uint32_t *w = reinterpret_cast<const uint32_t *>(zr);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        bsum[2 * c] += __uint_as_float(w[4 * j + c] << 16);
                        bsum[2 * c + 1] += __uint_as_float(w[4 * j + c] & 0xffff0000u);
                    }
            }
        }
        if (it == 0 || q.oy == 0) {  // a strip's first step also needs the row above
            if constexpr (CIN == 2) {
                g.x[s_up][t & 1][t >> 7][(t & 127) >> 1] = load_x2(q, 2 * q.oy - 1);
            } else if (row == 0) {
                uint4 up[4];
                load_x32(q, 2 * q.oy - 1, up);
                put8(up, &g.x[s_up][par][oct * 8][4 * quad]);
            }
        }
        const Step nq = step_at(it + 1);
        load_step(nq);
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < WG_PX / 32; ++kk) {
            const int p = kk * 32 + kg * 8;
            if constexpr (CIN == 2) {
                // waves 0, 1: the 12 columns (ky, kx = 1, 2, ci) with dZ at p; waves 2, 3: the 6
                // columns (ky, kx = 0, ci) with dZ at p + 1; the columns past them are not stored
                const int late = wave >> 1;
                const int n = min(m, late ? 5 : 11);
                const int ky = late ? n >> 1 : n >> 2, odd = late ? 1 : (n >> 1) & 1;
                const int slot = ky == 1 ? 2 : (ky == 0 ? s_up : s_dn);
                const bf16x8 a = load8(&g.z[late][(wave & 1) * 16 + m][p]);
                const bf16x8 b = load8(&g.x[slot][odd][n & 1][p]);
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[0], 0, 0, 0);
            } else {
                const int mt = wave & 1, nt = wave >> 1;
                const bf16x8 a0 = load8(&g.z[0][mt * 16 + m][p]);
                const bf16x8 a1 = load8(&g.z[1][mt * 16 + m][p]);
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) {
                    const int slot = ky == 1 ? 2 : (ky == 0 ? s_up : s_dn);
                    const bf16x8 e = load8(&g.x[slot][0][nt * 16 + m][p]);
                    const bf16x8 o = load8(&g.x[slot][1][nt * 16 + m][p]);
                    acc[NACC == 9 ? 3 * ky : 0] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, o, acc[NACC == 9 ? 3 * ky : 0], 0, 0, 0);
                    acc[NACC == 9 ? 3 * ky + 1 : 0] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, e, acc[NACC == 9 ? 3 * ky + 1 : 0], 0, 0, 0);
                    acc[NACC == 9 ? 3 * ky + 2 : 0] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, o, acc[NACC == 9 ? 3 * ky + 2 : 0], 0, 0, 0);
                }
            }
        }
        q = nq;
    }
    // the groups in order into one partial: D[co = 16 mt + 4 kg + j][n]
    float *sum = reinterpret_cast<float *>(lds);  // [9 * CIN][32], then the bias sums [16][32]
    float *bred = sum + NW;
    for (int gg = 0; gg < WG_GRP; ++gg) {
        __syncthreads();
        if (grp != gg) continue;
        auto add = [&](float *slot, float v) { *slot = gg == 0 ? v : *slot + v; };
        if constexpr (CIN == 2) {
            const int late = wave >> 1;
            if (m < (late ? 6 : 12)) {
                const int tap = late ? 3 * (m >> 1) : 3 * (m >> 2) + 1 + ((m >> 1) & 1);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    add(&sum[(tap * CIN + (m & 1)) * CNN_CH + (wave & 1) * 16 + kg * 4 + j], acc[0][j]);
            }
        } else {
            const int mt = wave & 1, nt = wave >> 1;
#pragma unroll
            for (int tap = 0; tap < NACC; ++tap)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    add(&sum[(tap * CIN + nt * 16 + m) * CNN_CH + mt * 16 + kg * 4 + j], acc[tap][j]);
        }
        if (t < 64)
#pragma unroll
            for (int c = 0; c < 8; ++c) add(&bred[zquad * CNN_CH + oct * 8 + c], bsum[c]);
    }
    __syncthreads();
    float *wp = wpart + (int64_t)blockIdx.x * 9 * CNN_CH * CNN_CH;
    for (int i = threadIdx.x; i < NW; i += 256 * WG_GRP) wp[i] = sum[i];
    if (threadIdx.x < CNN_CH) {
        float s = 0.0f;
        for (int i = 0; i < 16; ++i) s += bred[i * CNN_CH + threadIdx.x];
        bpart[(int64_t)blockIdx.x * CNN_CH + threadIdx.x] = s;
    }
}

// Sum of the partials: n_w weight and CNN_CH bias entries.  A workgroup takes 32 entries; its
// eight rows of threads each add every eighth partial in order (eight loads in flight each,
// where one thread per entry waited on a serial chain of 256: 62 -> 5 us a layer), and
// the eight sums are added in row order.
__global__ __launch_bounds__(256) void wgrad_reduce(const float *__restrict__ wpart, const float *__restrict__ bpart,
                                                    int32_t chunks, int32_t n_w, float *__restrict__ gw,
                                                    float *__restrict__ gb)
{
    __shared__ float part[8][32];
    const int e = threadIdx.x & 31, r = threadIdx.x >> 5;
    const int32_t i = blockIdx.x * 32 + e;  // n_w is a multiple of 32: a workgroup is all weights or all biases
    const bool w = i < n_w;
    const float *src = w ? wpart + i : bpart + (i - n_w);
    const int64_t pitch = w ? 9 * CNN_CH * CNN_CH : CNN_CH;
    float s = 0.0f;
#pragma unroll 8
    for (int32_t c = r; c < chunks; c += 8) s += src[c * pitch];
    part[r][e] = s;
    __syncthreads();
    if (r == 0) {
        float v = 0.0f;
        for (int k = 0; k < 8; ++k) v += part[k][e];
        *(w ? gw + i : gb + (i - n_w)) = v;
    }
}

// ---- data gradient -------------------------------------------------------------------------------
// dX[iy][ix][ci] = sum over the taps whose output pixel exists of dZ[oy][ox][co] W[t][ci][co];
// the result times the ReLU mask of X is the previous layer's dZ.  A lane takes the 2 x 2 input
// pixels (2 q, 2 q + 1) x (2 j, 2 j + 1), which need dZ at rows q, q + 1 and columns j, j + 1:
// four loads for the nine taps, whose weights stay in registers, as operands dealt like the
// forward's, so the mask is read and the result written in 16-byte pieces, both pixels of a
// pair by neighbouring instructions.  The wave walks down DG_ROWS row pairs and keeps the lower
// row of dZ for the next.  Bound by memory: the three layers of 16 pairs of 1024x1024 took 304 us with
// one parity per wave and a pass through LDS, now 157 (790 MB).
constexpr int DG_ROWS = 4;

__global__ __launch_bounds__(256) void dgrad(const uint16_t *__restrict__ dz, const uint16_t *__restrict__ wd,
                                             const uint16_t *__restrict__ xin, int32_t H, int32_t W,
                                             uint16_t *__restrict__ dzin)
{
    const int32_t Ho = (H + 1) / 2, Wo = (W + 1) / 2;
    const int32_t b = blockIdx.z, q0 = blockIdx.y * DG_ROWS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, kg = lane >> 4;
    const int32_t j = blockIdx.x * 64 + 16 * wave + m;
    bf16x8 w0[9], w1[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        w0[t] = load8(wd + ((int64_t)t * CNN_CH + tile_channel(m)) * CNN_CH + kg * 8);
        w1[t] = load8(wd + ((int64_t)t * CNN_CH + tile_channel(m) + 4) * CNN_CH + kg * 8);
    }
    const uint16_t *zb = dz + (int64_t)b * Ho * Wo * CNN_CH;
    const uint16_t *xb = xin + (int64_t)b * H * W * CNN_CH;
    uint16_t *gb = dzin + (int64_t)b * H * W * CNN_CH;
    const uint32_t zo = (uint32_t)j * 64 + kg * 16, xo = (uint32_t)j * 128 + kg * 16;
    bf16x8 z[2][2], zn[2];  // rows q and q + 1, columns j and j + 1; row q + 2
    bf16x8 xm[2][2], xn[2][2];
    auto load_z = [&](int32_t oy, bf16x8 (&v)[2]) {
        const __amdgpu_buffer_rsrc_t row = plane_row(zb, oy, Ho, Wo);
        v[0] = row_load8(row, zo);
        v[1] = row_load8(row, zo + 64);
    };
    auto load_x = [&](int32_t q, bf16x8 (&v)[2][2]) {
#pragma unroll
        for (int py = 0; py < 2; ++py) {
            const __amdgpu_buffer_rsrc_t row = plane_row(xb, 2 * q + py, H, W);
            v[py][0] = row_load8(row, xo);
            v[py][1] = row_load8(row, xo + 64);
        }
    };
    load_z(q0, z[0]);
    load_z(q0 + 1, z[1]);
    load_x(q0, xm);
#pragma unroll
    for (int i = 0; i < DG_ROWS; ++i) {
        const int32_t q = q0 + i;
        if (i + 1 < DG_ROWS) {
            load_z(q + 2, zn);
            load_x(q + 1, xn);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int py = 0; py < 2; ++py) {
            const __amdgpu_buffer_rsrc_t out = plane_row(gb, 2 * q + py, H, W);
#pragma unroll
            for (int px = 0; px < 2; ++px) {
                f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) {
                    if ((py + 1 - ky) & 1) continue;
                    const int dq = (py + 1 - ky) / 2;  // row q + dq of dZ
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx) {
                        if ((px + 1 - kx) & 1) continue;
                        const int dj = (px + 1 - kx) / 2;
                        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0[3 * ky + kx], z[dq][dj], acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[3 * ky + kx], z[dq][dj], acc1, 0, 0, 0);
                    }
                }
                const uint4 xw = __builtin_bit_cast(uint4, xm[py][px]);
                const uint32_t xv[4] = {xw.x, xw.y, xw.z, xw.w};
                float g[8];
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    g[c] = bf2f((uint16_t)(xv[c / 2] >> (16 * (c & 1)))) > 0.0f ? (c < 4 ? acc0[c & 3] : acc1[c & 3])
                                                                              : 0.0f;
                row_store8(out, xo + 64 * px, pack8(g));
            }
        }
        if (i + 1 < DG_ROWS) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                z[0][e] = z[1][e];
                z[1][e] = zn[e];
                xm[0][e] = xn[0][e];
                xm[1][e] = xn[1][e];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ---- AdamW on the FP32 master parameters ------------------------------------------------------
__global__ void adamw(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                      const float *__restrict__ g, int64_t n, float lr, float beta1, float beta2, float eps, float wd,
                      float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
    const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1, vh = vi / c2;
    p[i] = p[i] - lr * (mh / (sqrtf(vh) + eps) + wd * p[i]);
}

// ---- host side -----------------------------------------------------------------------------------
static size_t al(size_t b) { return (b + 255) & ~(size_t)255; }

CnnLayout cnn_layout(int32_t B, int32_t h, int32_t w)
{
    CnnLayout L;
    size_t off = 0;
    L.wf = off;
    off += al(sizeof(uint16_t) * (1024 + 3 * 9 * 1024));
    L.wd = off;
    off += al(sizeof(uint16_t) * 3 * 9 * 1024);
    int32_t hh = h, ww = w;
    for (int l = 0; l < 4; ++l) {
        hh = (hh + 1) / 2;
        ww = (ww + 1) / 2;
        L.hs[l] = hh;
        L.ws[l] = ww;
        L.act[l] = off;
        off += al(sizeof(uint16_t) * (size_t)B * hh * ww * CNN_CH);
    }
    L.pool = off;
    off += al(sizeof(double) * (size_t)B * CNN_CH);
    L.ppart = off;
    off += al(sizeof(double) * (size_t)B * ceil_div((int64_t)L.hs[3] * L.ws[3], POOL_CHUNK) * CNN_CH);
    L.fwd_total = off;
    // backward: two gradient planes the size of the largest activation, partial sums
    const size_t big = sizeof(uint16_t) * (size_t)B * L.hs[0] * L.ws[0] * CNN_CH;
    L.dz[0] = off;
    off += al(big);
    L.dz[1] = off;
    off += al(big);
    L.dpool = off;
    off += al(sizeof(double) * (size_t)B * CNN_CH);
    L.wpart = off;
    off += al(sizeof(float) * (size_t)CNN_WGRAD_CHUNKS * 9 * CNN_CH * CNN_CH);
    L.bpart = off;
    off += al(sizeof(float) * (size_t)CNN_WGRAD_CHUNKS * 9 * CNN_CH);
    L.total = off;
    return L;
}

int cnn_forward_launch(const uint16_t *ref, int64_t ref_stride, const uint16_t *img, int32_t B, int32_t h,
                       int32_t w, const float *params, float *pred, void *ws, hipStream_t s)
{
    const CnnLayout L = cnn_layout(B, h, w);
    unsigned char *base = static_cast<unsigned char *>(ws);
    uint16_t *wf = reinterpret_cast<uint16_t *>(base + L.wf);
    uint16_t *wd = reinterpret_cast<uint16_t *>(base + L.wd);
    hipLaunchKernelGGL(pack_weights, dim3((unsigned)ceil_div(1024 + 6 * 9 * 1024, 256)), dim3(256), 0, s, params, wf,
                       wd);
    ProfScope prof("cnn_forward", s);
    int32_t hh = h, ww = w;
    const uint16_t *in = nullptr;
    for (int l = 0; l < 4; ++l) {
        uint16_t *out = reinterpret_cast<uint16_t *>(base + L.act[l]);
        const float *bias = params + cnn_weight_offset(l) + 9 * (l == 0 ? 2 : CNN_CH) * CNN_CH;
        const dim3 grid((unsigned)ceil_div(L.ws[l], 64), (unsigned)ceil_div(L.hs[l], CONV_ROWS), (unsigned)B);
        if (l == 0)
            hipLaunchKernelGGL(conv_first, grid, dim3(256), 0, s, ref, ref_stride, img, hh, ww, wf, bias, out);
        else
            hipLaunchKernelGGL(conv_next, grid, dim3(256), 0, s, in, hh, ww, wf + 1024 + (size_t)(l - 1) * 9 * 1024,
                               bias, out);
        in = out;
        hh = L.hs[l];
        ww = L.ws[l];
    }
    const int64_t P4 = (int64_t)L.hs[3] * L.ws[3];
    const int32_t nchunk = (int32_t)ceil_div(P4, POOL_CHUNK);
    double *ppart = reinterpret_cast<double *>(base + L.ppart);
    hipLaunchKernelGGL(pool_partial, dim3((unsigned)nchunk, (unsigned)B), dim3(256), 0, s, in, P4, nchunk, ppart);
    hipLaunchKernelGGL(pool_head, dim3(B), dim3(64), 0, s, ppart, nchunk, P4, params,
                       reinterpret_cast<double *>(base + L.pool), pred);
    return check_launch("reduce_cnn_forward");
}

int cnn_backward_launch(const uint16_t *ref, int64_t ref_stride, const uint16_t *img, int32_t B, int32_t h,
                        int32_t w, const float *params, const float *pred, const float *target, double delta,
                        float *loss, float *grad, void *ws, hipStream_t s)
{
    const CnnLayout L = cnn_layout(B, h, w);
    unsigned char *base = static_cast<unsigned char *>(ws);
    const uint16_t *wd = reinterpret_cast<const uint16_t *>(base + L.wd);
    double *pool = reinterpret_cast<double *>(base + L.pool);
    double *dpool = reinterpret_cast<double *>(base + L.dpool);
    float *wpart = reinterpret_cast<float *>(base + L.wpart);
    float *bpart = reinterpret_cast<float *>(base + L.bpart);
    uint16_t *dz[2] = {reinterpret_cast<uint16_t *>(base + L.dz[0]), reinterpret_cast<uint16_t *>(base + L.dz[1])};
    ProfScope prof("cnn_backward", s);
    hipLaunchKernelGGL(head_backward, dim3(1), dim3(256), 0, s, pred, target, B, delta, pool, params, loss, grad,
                       dpool);
    const int64_t P4 = (int64_t)L.hs[3] * L.ws[3];
    const uint16_t *x4 = reinterpret_cast<const uint16_t *>(base + L.act[3]);
    hipLaunchKernelGGL(pool_backward, dim3((unsigned)ceil_div((int64_t)B * P4 * CNN_CH, 256)), dim3(256), 0, s, x4,
                       P4, B, dpool, dz[0]);
    int cur = 0;
    for (int l = 3; l >= 0; --l) {
        const int32_t hin = l ? L.hs[l - 1] : h, win = l ? L.ws[l - 1] : w;
        const uint16_t *xin = l ? reinterpret_cast<const uint16_t *>(base + L.act[l - 1]) : nullptr;
        const int64_t steps = (int64_t)B * ceil_div(L.ws[l], WG_PX) * L.hs[l];  // strip rows
        const int32_t chunks = (int32_t)std::min<int64_t>(CNN_WGRAD_CHUNKS, ceil_div(steps, WG_GRP));
        if (l == 0)
            hipLaunchKernelGGL(wgrad<2>, dim3(chunks), dim3(256 * WG_GRP), 0, s, nullptr, ref, ref_stride, img, B, hin, win,
                               dz[cur], wpart, bpart);
        else
            hipLaunchKernelGGL(wgrad<32>, dim3(chunks), dim3(256 * WG_GRP), 0, s, xin, nullptr, 0, nullptr, B, hin, win,
                               dz[cur], wpart, bpart);
        const int32_t cin = l == 0 ? 2 : CNN_CH;
        const int32_t n_w = 9 * cin * CNN_CH;
        float *gw = grad + cnn_weight_offset(l);
        hipLaunchKernelGGL(wgrad_reduce, dim3((unsigned)((n_w + CNN_CH) / 32)), dim3(256), 0, s, wpart, bpart,
                           chunks, n_w, gw, gw + n_w);
        if (l > 0) {
            const dim3 grid((unsigned)ceil_div((win + 1) / 2, 64), (unsigned)ceil_div((hin + 1) / 2, DG_ROWS),
                            (unsigned)B);
            hipLaunchKernelGGL(dgrad, grid, dim3(256), 0, s, dz[cur], wd + (size_t)(l - 1) * 9 * 1024, xin, hin, win,
                               dz[cur ^ 1]);
            cur ^= 1;
        }
    }
    return check_launch("reduce_cnn_backward");
}

}  // namespace rd

using namespace rd;

extern "C" size_t reduce_cnn_input_ws(int32_t W, int32_t H, int32_t N)
{
    if (W < 4 || H < 4 || W % 4 || H % 4 || N < 1) return 0;
    const int64_t n = (int64_t)(W / 4) * (H / 4);
    const int64_t nparts = ceil_div(n, DS_BLOCK);
    return al(sizeof(float) * n * N) + al(2 * sizeof(double) * nparts * N) + 3 * al(sizeof(double) * N);
}

extern "C" int reduce_cnn_input(const float *frames, int32_t W, int32_t H, int32_t N, uint16_t *out, void *ws,
                                size_t ws_bytes, void *stream)
{
    if (!frames || !out) return fail(REDUCE_ERR_NULL, "reduce_cnn_input: NULL buffer");
    if (W < 4 || H < 4 || N < 1) return fail(REDUCE_ERR_SHAPE, "reduce_cnn_input: W, H >= 4 and N >= 1 needed");
    if (W % 4 || H % 4) return fail(REDUCE_ERR_SHAPE, "reduce_cnn_input: W and H must be multiples of 4");
    if (N > 65535) return fail(REDUCE_ERR_UNSUPPORTED, "reduce_cnn_input: N above 65535");
    const size_t need = reduce_cnn_input_ws(W, H, N);
    if (!ws || ws_bytes < need)
        return fail(REDUCE_ERR_WORKSPACE, "reduce_cnn_input: workspace needs " + std::to_string(need) + " bytes");
    hipStream_t s = as_stream(stream);
    const int64_t n = (int64_t)(W / 4) * (H / 4);
    const int32_t nparts = (int32_t)ceil_div(n, DS_BLOCK);
    unsigned char *base = static_cast<unsigned char *>(ws);
    float *m = reinterpret_cast<float *>(base);
    unsigned char *b1 = base + al(sizeof(float) * n * N);
    double *part = reinterpret_cast<double *>(b1);
    unsigned char *b2 = b1 + al(2 * sizeof(double) * nparts * N);
    double *shift = reinterpret_cast<double *>(b2);
    double *mean = reinterpret_cast<double *>(b2 + al(sizeof(double) * N));
    double *sd = reinterpret_cast<double *>(b2 + 2 * al(sizeof(double) * N));
    ProfScope prof("cnn_input", s);
    hipLaunchKernelGGL(ds_boxmean, dim3((unsigned)nparts, (unsigned)N), dim3(DS_BLOCK), 0, s, frames, W, H, m, part,
                       shift);
    hipLaunchKernelGGL(ds_finish, dim3(N), dim3(DS_BLOCK), 0, s, part, nparts, (double)n, shift, mean, sd);
    hipLaunchKernelGGL(ds_normalize, dim3((unsigned)ceil_div(n, 4 * DS_BLOCK), (unsigned)N), dim3(DS_BLOCK), 0, s,
                       m, n, mean, sd, out);
    return check_launch("reduce_cnn_input");
}

extern "C" int64_t reduce_cnn_num_params(void) { return CNN_NPARAMS; }

extern "C" size_t reduce_cnn_ws(int32_t B, int32_t h, int32_t w)
{
    if (B < 1 || h < 16 || w < 16) return 0;
    return cnn_layout(B, h, w).total;
}

extern "C" int reduce_cnn_ws_offsets(int32_t B, int32_t h, int32_t w, int64_t *offsets)
{
    if (!offsets) return fail(REDUCE_ERR_NULL, "reduce_cnn_ws_offsets: NULL argument");
    if (B < 1 || h < 16 || w < 16) return fail(REDUCE_ERR_SHAPE, "reduce_cnn_ws_offsets: bad sizes");
    const CnnLayout L = cnn_layout(B, h, w);
    for (int l = 0; l < 4; ++l) offsets[l] = (int64_t)L.act[l];
    offsets[4] = (int64_t)L.dz[0];
    offsets[5] = (int64_t)L.dz[1];
    return REDUCE_OK;
}

extern "C" int reduce_cnn_forward(const uint16_t *ref, int64_t ref_stride, const uint16_t *img, int32_t B,
                                  int32_t h, int32_t w, const float *params, float *pred, void *ws, size_t ws_bytes,
                                  void *stream)
{
    if (!ref || !img || !params || !pred) return fail(REDUCE_ERR_NULL, "reduce_cnn_forward: NULL buffer");
    if (B < 1 || h < 16 || w < 16) return fail(REDUCE_ERR_SHAPE, "reduce_cnn_forward: B >= 1 and h, w >= 16 needed");
    if (ref_stride < 0) return fail(REDUCE_ERR_RANGE, "reduce_cnn_forward: negative ref_stride");
    if (B > 65535 || h > 65535) return fail(REDUCE_ERR_UNSUPPORTED, "reduce_cnn_forward: B or h above 65535");
    const size_t need = cnn_layout(B, h, w).total;
    if (!ws || ws_bytes < need)
        return fail(REDUCE_ERR_WORKSPACE, "reduce_cnn_forward: workspace needs " + std::to_string(need) + " bytes");
    return cnn_forward_launch(ref, ref_stride, img, B, h, w, params, pred, ws, as_stream(stream));
}

extern "C" int reduce_cnn_backward(const uint16_t *ref, int64_t ref_stride, const uint16_t *img, int32_t B,
                                   int32_t h, int32_t w, const float *params, const float *pred, const float *target,
                                   float huber_delta, float *loss, float *grad, void *ws, size_t ws_bytes,
                                   void *stream)
{
    if (!ref || !img || !params || !pred || !target || !loss || !grad)
        return fail(REDUCE_ERR_NULL, "reduce_cnn_backward: NULL buffer");
    if (B < 1 || h < 16 || w < 16) return fail(REDUCE_ERR_SHAPE, "reduce_cnn_backward: B >= 1 and h, w >= 16 needed");
    if (B > 1024) return fail(REDUCE_ERR_UNSUPPORTED, "reduce_cnn_backward: B above 1024");
    if (!(huber_delta > 0.0f)) return fail(REDUCE_ERR_RANGE, "reduce_cnn_backward: huber_delta must be > 0");
    const size_t need = cnn_layout(B, h, w).total;
    if (!ws || ws_bytes < need)
        return fail(REDUCE_ERR_WORKSPACE, "reduce_cnn_backward: workspace needs " + std::to_string(need) + " bytes");
    return cnn_backward_launch(ref, ref_stride, img, B, h, w, params, pred, target, (double)huber_delta, loss, grad,
                               ws, as_stream(stream));
}

extern "C" int reduce_cnn_adamw(float *params, float *m, float *v, const float *grad, int64_t n, float lr,
                                float beta1, float beta2, float eps, float weight_decay, int32_t step, void *stream)
{
    if (!params || !m || !v || !grad) return fail(REDUCE_ERR_NULL, "reduce_cnn_adamw: NULL buffer");
    if (n < 1 || step < 1) return fail(REDUCE_ERR_RANGE, "reduce_cnn_adamw: n and step must be >= 1");
    if (!(lr >= 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f))
        return fail(REDUCE_ERR_RANGE, "reduce_cnn_adamw: bad hyper-parameters");
    const float c1 = (float)(1.0 - std::pow((double)beta1, (double)step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, (double)step));
    hipLaunchKernelGGL(adamw, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, as_stream(stream), params, m, v, grad, n,
                       lr, beta1, beta2, eps, weight_decay, c1, c2);
    return check_launch("reduce_cnn_adamw");
}
