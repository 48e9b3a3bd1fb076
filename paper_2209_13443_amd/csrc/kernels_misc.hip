// Bandwidth-bound kernels for gfx950: depthwise 3x3, max-pool, the exit head (global average
// pool, FC, softmax top-1 and the exit decision), slot compaction / refill and admission.
// All of them move 16 bytes per lane per access along the channel (NHWC) or sample axis so
// that a wavefront touches whole cache lines.
#include <type_traits>
#include <algorithm>

#include "ee_internal.hpp"
#include "head_device.hpp"

namespace ee {

// The kernels that a lane's next step waits for, a few wavefronts each but for the compaction, whose hundreds of workgroups are short: they issue before the wavefronts of another lane's segment on their SIMD.
// MobileNetV2, two lanes of 64 slots, 4,096 requests, ms, medians of 120 passes, 24 processes of each in turn on two cards, two tables: none 11.75-12.02, 11.87 in the mean, all but the compaction 11.74-11.86, 11.80,
// all 11.58-11.88, 11.70.  ResNet-50 int8, which compacts nothing, level (52.29 / 52.33); single lanes too.
__device__ __forceinline__ void issue_first() { __builtin_amdgcn_s_setprio(3); }

typedef int v4i __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f32_to_bf16_rne_m(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }
__device__ __forceinline__ float bf16_to_f32_m(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ int med3_i32(int v, int lo, int hi)       // lo <= hi: v clamped to [lo, hi]
{
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
    return r;
}
__device__ __forceinline__ int byte_of(int word, int e) { return (int)(signed char)((word >> (8 * e)) & 0xFF); }

// ---- depthwise k x k: one lane = one output pixel x 16 bytes of channels ---------------------------
// weights repacked [k*k][C]; int8: int32 accumulate + bias, round-shift, clamp; bf16: float accumulate.
template <int ES>
__global__ __launch_bounds__(256) void depthwise_kernel(PoolArgs a, int units)
{
    request_args<sizeof(PoolArgs)>();
    const int cchunks = a.C * ES / 16, unit = xcd_unit(blockIdx.x, units);
    const long long idx = (long long)unit * 256 + threadIdx.x;
    if (unit < 0) return;
    if (idx >= (long long)a.B * a.Ho * a.Wo * cchunks) return;
    const int q = (int)(idx % cchunks);
    const long long pix = idx / cchunks;
    const int ox = (int)(pix % a.Wo), oy = (int)((pix / a.Wo) % a.Ho), n = (int)(pix / ((long long)a.Wo * a.Ho));
    const unsigned char* x = (const unsigned char*)a.x;
    if constexpr (ES == 1) {
        int acc[16];
        const int* bias = (const int*)a.bias + q * 16;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = bias[e];
        for (int r = 0; r < a.k; ++r) {
            const int iy = oy * a.stride + r - a.pad;
            if (iy < 0 || iy >= a.H) continue;
            for (int s = 0; s < a.k; ++s) {
                const int ix = ox * a.stride + s - a.pad;
                if (ix < 0 || ix >= a.W) continue;
                const v4i xv = *(const v4i*)(x + (((long long)n * a.H + iy) * a.W + ix) * a.C + q * 16);
                const v4i wv = *(const v4i*)((const unsigned char*)a.w + (long long)(r * a.k + s) * a.C + q * 16);
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[e] += byte_of(xv[e >> 2], e & 3) * byte_of(wv[e >> 2], e & 3);
            }
        }
        v4i out = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            int t = a.shift > 0 ? (acc[e] + (1 << (a.shift - 1))) >> a.shift : acc[e];
            t = min(max(t, a.lo), a.hi);
            out[e >> 2] |= (t & 0xFF) << (8 * (e & 3));
        }
        *(v4i*)((unsigned char*)a.y + pix * a.C + q * 16) = out;
    } else {
        float acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
        for (int r = 0; r < a.k; ++r) {
            const int iy = oy * a.stride + r - a.pad;
            if (iy < 0 || iy >= a.H) continue;
            for (int s = 0; s < a.k; ++s) {
                const int ix = ox * a.stride + s - a.pad;
                if (ix < 0 || ix >= a.W) continue;
                const v4i xv = *(const v4i*)(x + ((((long long)n * a.H + iy) * a.W + ix) * a.C) * 2 + q * 16);
                const v4i wv = *(const v4i*)((const unsigned char*)a.w + ((long long)(r * a.k + s) * a.C) * 2 + q * 16);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint16_t xe = (uint16_t)((unsigned)xv[e >> 1] >> (16 * (e & 1)));
                    const uint16_t we = (uint16_t)((unsigned)wv[e >> 1] >> (16 * (e & 1)));
                    acc[e] = fmaf(bf16_to_f32_m(xe), bf16_to_f32_m(we), acc[e]);
                }
            }
        }
        const float* bias = (const float*)a.bias + q * 8;
        v4i out = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float t = fminf(fmaxf(acc[e] + bias[e], a.f_lo), a.f_hi);
            out[e >> 1] |= (int)((unsigned)f32_to_bf16_rne_m(t) << (16 * (e & 1)));
        }
        *(v4i*)((unsigned char*)a.y + (pix * a.C) * 2 + q * 16) = out;
    }
}

// ---- depthwise 3x3, int8, on the 4-way dot product --------------------------------------------------------
// One lane = 4 output pixels along x times 16 channels.  v_dot4_i32_i8 wants the 4 bytes of a dword to be 4
// taps of one channel, NHWC delivers 4 channels of one tap: per input column the three row dwords (and a
// zero) of a 4-channel group are byte-transposed with 8 v_perm_b32, and one dot product per channel adds the
// column to every output pixel whose window holds it.  A column is transposed once for the up to three windows
// that share it, and the lane loads 18 (stride 1) or 27 (stride 2) times 16 bytes for 4 outputs instead of 36.
// Weights are packed per 16-channel chunk as [column s][4-channel group][channel] dwords
// (w[0][s], w[1][s], w[2][s], 0), 192 bytes per chunk.  Coordinates outside the image are clamped, so every
// load is in range; such taps become zero through the selectors of the first permute level (selector 0x0c
// yields a zero byte).  The rounding constant of the shift is added to the bias once.
template <int STRIDE, bool TABLE_IN_LDS>
__global__ __launch_bounds__(256) void depthwise3x3_i8_kernel(PoolArgs a, int groups_x)
{
    constexpr int PX = 4, COLS = (PX - 1) * STRIDE + 3;
    extern __shared__ __attribute__((aligned(16))) unsigned char dw_lds_raw[];
    v4i* dw_lds = (v4i*)dw_lds_raw;                    // per 16-channel chunk: 12 weight quads, then 4 bias quads
    const int cchunks = a.C / 16;
    const long long total = (long long)a.B * a.Ho * groups_x * cchunks;
    const int unit = xcd_unit(blockIdx.x, (int)((total + 255) / 256));
    if (unit < 0) return;
    const long long idx = min((long long)unit * 256 + threadIdx.x, total - 1);      // lanes past the end redo the last item
    const bool active = (long long)unit * 256 + threadIdx.x < total;
    const int q = (int)(idx % cchunks);
    const int g = (int)(idx / cchunks);
    const int ox0 = (g % groups_x) * PX, oy = (g / groups_x) % a.Ho, n = g / (groups_x * a.Ho);
    const unsigned char* x = (const unsigned char*)a.x;
    const int iy0 = oy * STRIDE - a.pad, ix0 = ox0 * STRIDE - a.pad;
    // byte offsets inside the batch tensor fit 32 bits (checked when the context is created)
    unsigned rowoff[3], coloff[COLS];
    bool rowok[3], colok[COLS];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int iy = iy0 + r;
        rowok[r] = (unsigned)iy < (unsigned)a.H;
        rowoff[r] = (unsigned)((n * a.H + min(max(iy, 0), a.H - 1)) * a.W) * (unsigned)a.C + (unsigned)q * 16u;
    }
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
        const int ix = ix0 + c;
        colok[c] = (unsigned)ix < (unsigned)a.W;
        coloff[c] = (unsigned)(min(max(ix, 0), a.W - 1) * a.C);
    }
    v4i xv[3][COLS];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < COLS; ++c) xv[r][c] = *(const v4i*)(x + (rowoff[r] + coloff[c]));
    // Weights and bias depend on the channel chunk only.  With few channels the workgroup copies the whole table
    // into LDS once (C * 16 bytes) instead of 16 loads of 16 bytes per lane through the vector memory path (the big
    // early layers: -10 %); with many channels and few pixels the copy is most of what a workgroup would read
    // anyway and only adds a step to a short launch, so those layers read the table per lane.
    if constexpr (TABLE_IN_LDS) {
        for (int i = threadIdx.x; i < cchunks * 16; i += 256) {
            const int qq = i >> 4, r = i & 15;
            dw_lds[i] = r < 12 ? ((const v4i*)a.w)[qq * 12 + r] : ((const v4i*)a.bias)[qq * 4 + (r - 12)];
        }
        __syncthreads();
    }
    if (!active) return;
    // first permute level of a column whose three rows are x0, x1, x2:
    //   (x0.b0, x1.b0, x0.b1, x1.b1), (x0.b2, x1.b2, x0.b3, x1.b3), (x2.b0, 0, x2.b1, 0), (x2.b2, 0, x2.b3, 0)
    const unsigned s_lo01 = (rowok[0] ? 0x00010000u : 0x000c000cu) | (rowok[1] ? 0x05000400u : 0x0c000c00u);
    const unsigned s_hi01 = (rowok[0] ? 0x00030002u : 0x000c000cu) | (rowok[1] ? 0x07000600u : 0x0c000c00u);
    const unsigned s_lo2 = rowok[2] ? 0x0c010c00u : 0x0c0c0c0cu, s_hi2 = rowok[2] ? 0x0c030c02u : 0x0c0c0c0cu;
    const int rnd = a.shift > 0 ? 1 << (a.shift - 1) : 0;
    v4i outv[PX];
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) {
        v4i b4, w[3];
        if constexpr (TABLE_IN_LDS) {
            b4 = dw_lds[q * 16 + 12 + cg];
#pragma unroll
            for (int s = 0; s < 3; ++s) w[s] = dw_lds[q * 16 + s * 4 + cg];
        } else {
            b4 = *((const v4i*)a.bias + q * 4 + cg);
#pragma unroll
            for (int s = 0; s < 3; ++s) w[s] = *((const v4i*)a.w + q * 12 + s * 4 + cg);
        }
        int acc[PX][4];
#pragma unroll
        for (int p = 0; p < PX; ++p)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[p][e] = b4[e] + rnd;
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
            const unsigned x0 = (unsigned)xv[0][c][cg], x1 = (unsigned)xv[1][c][cg], x2 = (unsigned)xv[2][c][cg];
            const unsigned lo01 = __builtin_amdgcn_perm(x1, x0, colok[c] ? s_lo01 : 0x0c0c0c0cu), hi01 = __builtin_amdgcn_perm(x1, x0, colok[c] ? s_hi01 : 0x0c0c0c0cu);
            const unsigned lo2 = __builtin_amdgcn_perm(0u, x2, colok[c] ? s_lo2 : 0x0c0c0c0cu), hi2 = __builtin_amdgcn_perm(0u, x2, colok[c] ? s_hi2 : 0x0c0c0c0cu);
            // bytes (x0.c, x1.c, x2.c, 0) for the group's channels c = 0..3
            const unsigned t[4] = {__builtin_amdgcn_perm(lo2, lo01, 0x05040100u), __builtin_amdgcn_perm(lo2, lo01, 0x07060302u),
                                   __builtin_amdgcn_perm(hi2, hi01, 0x05040100u), __builtin_amdgcn_perm(hi2, hi01, 0x07060302u)};
#pragma unroll
            for (int s = 0; s < 3; ++s)
                if ((c - s) >= 0 && (c - s) % STRIDE == 0 && (c - s) / STRIDE < PX) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[(c - s) / STRIDE][e] = __builtin_amdgcn_sdot4((int)t[e], w[s][e], acc[(c - s) / STRIDE][e], false);
                }
        }
#pragma unroll
        for (int p = 0; p < PX; ++p) {
            int t[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = med3_i32(acc[p][e] >> a.shift, a.lo, a.hi);
            const unsigned lo = __builtin_amdgcn_perm((unsigned)t[1], (unsigned)t[0], 0x0c0c0400u), hi = __builtin_amdgcn_perm((unsigned)t[3], (unsigned)t[2], 0x0c0c0400u);
            outv[p][cg] = (int)__builtin_amdgcn_perm(hi, lo, 0x05040100u);
        }
    }
#pragma unroll
    for (int p = 0; p < PX; ++p)
        if (ox0 + p < a.Wo) *(v4i*)((unsigned char*)a.y + ((((long long)n * a.Ho + oy) * a.Wo + ox0 + p) * a.C) + q * 16) = outv[p];
}

hipError_t launch_depthwise(const PoolArgs& a, int dtype, hipStream_t s)
{
    const int es = dtype == EE_I8 ? 1 : 2;
    if (dtype == EE_I8 && a.k == 3 && a.w3 && (a.stride == 1 || a.stride == 2)) {
        const int groups_x = (a.Wo + 3) / 4;
        const long long total = (long long)a.B * a.Ho * groups_x * (a.C / 16);
        if (total <= 0) return hipSuccess;
        PoolArgs b = a;
        b.w = a.w3;
        const dim3 grid(xcd_grid((total + 255) / 256));
        if (a.C <= 192) {                   // the table in LDS: measured to pay up to 192 channels (see the kernel)
            const size_t lds_bytes = (size_t)a.C * 16;
            if (a.stride == 1) EE_LAUNCH((depthwise3x3_i8_kernel<1, true>), grid, dim3(256), lds_bytes, s, b, groups_x);
            else EE_LAUNCH((depthwise3x3_i8_kernel<2, true>), grid, dim3(256), lds_bytes, s, b, groups_x);
        } else {
            if (a.stride == 1) EE_LAUNCH((depthwise3x3_i8_kernel<1, false>), grid, dim3(256), 0, s, b, groups_x);
            else EE_LAUNCH((depthwise3x3_i8_kernel<2, false>), grid, dim3(256), 0, s, b, groups_x);
        }
        return hipGetLastError();
    }
    const long long total = (long long)a.B * a.Ho * a.Wo * (a.C * es / 16);
    if (total <= 0) return hipSuccess;
    const int units = (int)((total + 255) / 256);
    if (dtype == EE_I8) EE_LAUNCH(depthwise_kernel<1>, dim3(xcd_grid(units)), dim3(256), 0, s, a, units);
    else EE_LAUNCH(depthwise_kernel<2>, dim3(xcd_grid(units)), dim3(256), 0, s, a, units);
    return hipGetLastError();
}

// ---- max-pool k x k over the in-range taps ---------------------------------------------------------
template <int ES>
__global__ __launch_bounds__(256) void maxpool_kernel(PoolArgs a, int units)
{
    request_args<sizeof(PoolArgs)>();
    const int cchunks = a.C * ES / 16, unit = xcd_unit(blockIdx.x, units);
    const long long idx = (long long)unit * 256 + threadIdx.x;
    if (unit < 0) return;
    if (idx >= (long long)a.B * a.Ho * a.Wo * cchunks) return;
    const int q = (int)(idx % cchunks);
    const long long pix = idx / cchunks;
    const int ox = (int)(pix % a.Wo), oy = (int)((pix / a.Wo) % a.Ho), n = (int)(pix / ((long long)a.Wo * a.Ho));
    const unsigned char* x = (const unsigned char*)a.x;
    constexpr int NE = 16 / ES;
    float bestf[NE];
    int besti[NE];
    bool have = false;
    v4i bits = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < NE; ++e) { besti[e] = -129; bestf[e] = 0.f; }
    for (int r = 0; r < a.k; ++r) {
        const int iy = oy * a.stride + r - a.pad;
        if (iy < 0 || iy >= a.H) continue;
        for (int s = 0; s < a.k; ++s) {
            const int ix = ox * a.stride + s - a.pad;
            if (ix < 0 || ix >= a.W) continue;
            const v4i xv = *(const v4i*)(x + ((((long long)n * a.H + iy) * a.W + ix) * a.C) * ES + q * 16);
            if constexpr (ES == 1) {
#pragma unroll
                for (int e = 0; e < 16; ++e) besti[e] = max(besti[e], byte_of(xv[e >> 2], e & 3));
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint16_t xe = (uint16_t)((unsigned)xv[e >> 1] >> (16 * (e & 1)));
                    const float v = bf16_to_f32_m(xe);
                    if (!have || v > bestf[e]) {
                        bestf[e] = v;
                        bits[e >> 1] = (bits[e >> 1] & ~(0xFFFF << (16 * (e & 1)))) | ((int)xe << (16 * (e & 1)));
                    }
                }
            }
            have = true;
        }
    }
    if constexpr (ES == 1) {
#pragma unroll
        for (int e = 0; e < 16; ++e) bits[e >> 2] |= (besti[e] & 0xFF) << (8 * (e & 3));
    }
    *(v4i*)((unsigned char*)a.y + (pix * a.ldc + a.c_off) * ES + q * 16) = bits;     // a channel slice when ldc > C
}

// ---- average pool k x k: all k*k taps, padding counts as zero, divisor k*k ---------------------------------
// int8: y = floor((2 * sum + k*k) / (2 * k*k)) (round half up); the numerator is made non-negative by adding
// 128 * k*k to the sum (and 128 is taken off the quotient), the division is a multiply-high with
// floor(2^32 / (2 k*k)) and one correction step.  bf16: float sum in tap order / (k*k), rounded to bf16.
template <int ES>
__global__ __launch_bounds__(256) void avgpool_kernel(PoolArgs a, unsigned magic, int units)
{
    request_args<sizeof(PoolArgs)>();
    const int cchunks = a.C * ES / 16, unit = xcd_unit(blockIdx.x, units);
    const long long idx = (long long)unit * 256 + threadIdx.x;
    if (unit < 0) return;
    if (idx >= (long long)a.B * a.Ho * a.Wo * cchunks) return;
    const int q = (int)(idx % cchunks);
    const long long pix = idx / cchunks;
    const int ox = (int)(pix % a.Wo), oy = (int)((pix / a.Wo) % a.Ho), n = (int)(pix / ((long long)a.Wo * a.Ho));
    const unsigned char* x = (const unsigned char*)a.x;
    constexpr int NE = 16 / ES;
    int sumi[NE];
    float sumf[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) { sumi[e] = 0; sumf[e] = 0.f; }
    for (int r = 0; r < a.k; ++r) {
        const int iy = oy * a.stride + r - a.pad;
        if (iy < 0 || iy >= a.H) continue;
        for (int s = 0; s < a.k; ++s) {
            const int ix = ox * a.stride + s - a.pad;
            if (ix < 0 || ix >= a.W) continue;
            const v4i xv = *(const v4i*)(x + ((((long long)n * a.H + iy) * a.W + ix) * a.C) * ES + q * 16);
            if constexpr (ES == 1) {
#pragma unroll
                for (int e = 0; e < 16; ++e) sumi[e] += byte_of(xv[e >> 2], e & 3);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) sumf[e] += bf16_to_f32_m((uint16_t)((unsigned)xv[e >> 1] >> (16 * (e & 1))));
            }
        }
    }
    v4i bits = {0, 0, 0, 0};
    const int kk = a.k * a.k;
    if constexpr (ES == 1) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const unsigned num = (unsigned)(2 * (sumi[e] + 128 * kk) + kk);        // < 2 * 255 * 225 + 225 < 2^17
            unsigned qv = __umulhi(num, magic);                                        // floor(num / (2 kk)), corrected below
            if ((qv + 1) * (unsigned)(2 * kk) <= num) ++qv;
            if (qv * (unsigned)(2 * kk) > num) --qv;
            bits[e >> 2] |= (((int)qv - 128) & 0xFF) << (8 * (e & 3));
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) bits[e >> 1] |= (int)((unsigned)f32_to_bf16_rne_m(sumf[e] / (float)kk) << (16 * (e & 1)));
    }
    *(v4i*)((unsigned char*)a.y + (pix * a.ldc + a.c_off) * ES + q * 16) = bits;
}

// ---- int8 3x3 max / average pool on 16-bit halves ---------------------------------------------------------------
// One lane = 4 output pixels along x times 16 channels; the three rows of every input column are reduced
// first and shared by the windows that overlap it, so a lane issues 18 (stride 1) or 27 (stride 2) 16-byte
// loads for 4 outputs instead of 36, and works on two channels per instruction.  Coordinates outside the
// image are clamped to the nearest pixel inside, so every load is in range and needs no select.
//  max: the clamped pixel belongs to the window (pad < 3), so it changes nothing.  A 16-bit signed max of the
//       halves (b1:b0), (b3:b2) of a dword is decided by the high byte: the raw dword yields channels 1 and 3,
//       the dword shifted left by 8 channels 0 and 2 (the low bytes are don't-cares).
//  avg: v_perm_b32 sign-extends bytes 1 and 3 of a dword into 16-bit lanes (again of the dword and of the
//       dword shifted left by 8); a tap outside the image uses the selector that yields zero instead.  The
//       lanes add with v_pk_add_i16 (|sum| <= 1152).  With S = sum + 1152 >= 0,
//       floor((2 S + 9) / 18) = ((2 S + 9) * 3641) >> 16 exactly for all S <= 2295 (3641 * 18 = 2^16 + 2 and
//       4599 * 2 < 2^16); the product stays below 2^24, so the quotient is byte 2 of it, and it carries the
//       bias 128 = 1152 / 9 that the last xor removes.
typedef short v2s __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pk_max_i16(unsigned a, unsigned b)
{
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(v2s, a), __builtin_bit_cast(v2s, b)));
}
__device__ __forceinline__ unsigned pk_add_i16(unsigned a, unsigned b)
{
    return __builtin_bit_cast(unsigned, __builtin_bit_cast(v2s, a) + __builtin_bit_cast(v2s, b));
}

template <int STRIDE, bool AVG>
__global__ __launch_bounds__(256) void pool3x3_i8_kernel(PoolArgs a, int groups_x, int units)
{
    request_args<sizeof(PoolArgs)>();
    constexpr int PX = 4, COLS = (PX - 1) * STRIDE + 3;
    const int cchunks = a.C / 16, unit = xcd_unit(blockIdx.x, units);
    const long long idx = (long long)unit * 256 + threadIdx.x;
    if (unit < 0) return;
    if (idx >= (long long)a.B * a.Ho * groups_x * cchunks) return;
    const int q = (int)(idx % cchunks);
    const int g = (int)(idx / cchunks);
    const int ox0 = (g % groups_x) * PX, oy = (g / groups_x) % a.Ho, n = g / (groups_x * a.Ho);
    const unsigned char* x = (const unsigned char*)a.x;
    const int iy0 = oy * STRIDE - a.pad, ix0 = ox0 * STRIDE - a.pad;
    // byte offsets inside the batch tensor fit 32 bits (checked when the context is created)
    unsigned rowoff[3], coloff[COLS];
    bool rowok[3], colok[COLS];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int iy = iy0 + r;
        rowok[r] = (unsigned)iy < (unsigned)a.H;
        rowoff[r] = (unsigned)((n * a.H + min(max(iy, 0), a.H - 1)) * a.W) * (unsigned)a.C + (unsigned)q * 16u;
    }
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
        const int ix = ix0 + c;
        colok[c] = (unsigned)ix < (unsigned)a.W;
        coloff[c] = (unsigned)(min(max(ix, 0), a.W - 1) * a.C);
    }
    v4i xv[3][COLS];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < COLS; ++c) xv[r][c] = *(const v4i*)(x + (rowoff[r] + coloff[c]));
    unsigned co[COLS][4], ce[COLS][4];         // per column and dword: channels 1, 3 and channels 0, 2 as 16-bit lanes
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
        unsigned sel[3];                       // avg: bytes (b1, sign b1, b3, sign b3) of the second operand, or four zero bytes
#pragma unroll
        for (int r = 0; r < 3; ++r) sel[r] = rowok[r] && colok[c] ? 0x09030801u : 0x0c0c0c0cu;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const unsigned x0 = (unsigned)xv[0][c][d], x1 = (unsigned)xv[1][c][d], x2 = (unsigned)xv[2][c][d];
            if constexpr (AVG) {
                co[c][d] = pk_add_i16(pk_add_i16(__builtin_amdgcn_perm(0u, x0, sel[0]), __builtin_amdgcn_perm(0u, x1, sel[1])), __builtin_amdgcn_perm(0u, x2, sel[2]));
                ce[c][d] = pk_add_i16(pk_add_i16(__builtin_amdgcn_perm(0u, x0 << 8, sel[0]), __builtin_amdgcn_perm(0u, x1 << 8, sel[1])),
                                      __builtin_amdgcn_perm(0u, x2 << 8, sel[2]));
            } else {
                co[c][d] = pk_max_i16(pk_max_i16(x0, x1), x2);
                ce[c][d] = pk_max_i16(pk_max_i16(x0 << 8, x1 << 8), x2 << 8);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < PX; ++p) {
        if (ox0 + p >= a.Wo) break;
        v4i out;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const unsigned o0 = co[p * STRIDE][d], o1 = co[p * STRIDE + 1][d], o2 = co[p * STRIDE + 2][d];
            const unsigned e0 = ce[p * STRIDE][d], e1 = ce[p * STRIDE + 1][d], e2 = ce[p * STRIDE + 2][d];
            if constexpr (AVG) {
                const unsigned so = pk_add_i16(pk_add_i16(o0, o1), pk_add_i16(o2, 0x04800480u));
                const unsigned se = pk_add_i16(pk_add_i16(e0, e1), pk_add_i16(e2, 0x04800480u));
                const unsigned t0 = (se & 0xFFFFu) * 7282u + 32769u, t2 = (se >> 16) * 7282u + 32769u;
                const unsigned t1 = (so & 0xFFFFu) * 7282u + 32769u, t3 = (so >> 16) * 7282u + 32769u;
                const unsigned lo = __builtin_amdgcn_perm(t1, t0, 0x0c0c0602u), hi = __builtin_amdgcn_perm(t3, t2, 0x06020c0cu);
                out[d] = (int)((lo | hi) ^ 0x80808080u);
            } else {
                const unsigned mo = pk_max_i16(pk_max_i16(o0, o1), o2), me = pk_max_i16(pk_max_i16(e0, e1), e2);
                out[d] = (int)__builtin_amdgcn_perm(mo, me, 0x07030501u);
            }
        }
        *(v4i*)((unsigned char*)a.y + ((((long long)n * a.Ho + oy) * a.Wo + ox0 + p) * a.ldc + a.c_off) + q * 16) = out;
    }
}

template <bool AVG>
static hipError_t launch_pool3x3_i8(const PoolArgs& a, hipStream_t s)
{
    const int groups_x = (a.Wo + 3) / 4;
    const long long total = (long long)a.B * a.Ho * groups_x * (a.C / 16);
    if (total <= 0) return hipSuccess;
    const int units = (int)((total + 255) / 256);
    if (a.stride == 1) EE_LAUNCH((pool3x3_i8_kernel<1, AVG>), dim3(xcd_grid(units)), dim3(256), 0, s, a, groups_x, units);
    else EE_LAUNCH((pool3x3_i8_kernel<2, AVG>), dim3(xcd_grid(units)), dim3(256), 0, s, a, groups_x, units);
    return hipGetLastError();
}

hipError_t launch_maxpool(const PoolArgs& a, int dtype, hipStream_t s)
{
    if (dtype == EE_I8 && a.k == 3 && (a.stride == 1 || a.stride == 2) && a.C % 16 == 0) return launch_pool3x3_i8<false>(a, s);
    const int es = dtype == EE_I8 ? 1 : 2;
    const long long total = (long long)a.B * a.Ho * a.Wo * (a.C * es / 16);
    if (total <= 0) return hipSuccess;
    const int units = (int)((total + 255) / 256);
    if (dtype == EE_I8) EE_LAUNCH(maxpool_kernel<1>, dim3(xcd_grid(units)), dim3(256), 0, s, a, units);
    else EE_LAUNCH(maxpool_kernel<2>, dim3(xcd_grid(units)), dim3(256), 0, s, a, units);
    return hipGetLastError();
}

hipError_t launch_avgpool(const PoolArgs& a, int dtype, hipStream_t s)
{
    if (dtype == EE_I8 && a.k == 3 && (a.stride == 1 || a.stride == 2) && a.C % 16 == 0) return launch_pool3x3_i8<true>(a, s);
    const int es = dtype == EE_I8 ? 1 : 2;
    const long long total = (long long)a.B * a.Ho * a.Wo * (a.C * es / 16);
    if (total <= 0) return hipSuccess;
    if (a.k < 1 || a.k > 15) return hipErrorInvalidValue;
    const int units = (int)((total + 255) / 256);
    const unsigned magic = (unsigned)(0x100000000ull / (unsigned)(2 * a.k * a.k));
    if (dtype == EE_I8) EE_LAUNCH(avgpool_kernel<1>, dim3(xcd_grid(units)), dim3(256), 0, s, a, magic, units);
    else EE_LAUNCH(avgpool_kernel<2>, dim3(xcd_grid(units)), dim3(256), 0, s, a, magic, units);
    return hipGetLastError();
}

// ---- exit head, step 1: global average pool ----------------------------------------------------------
// One workgroup per (sample, one of S pixel splits).  Lane = (pixel lane pl, 16-byte channel chunk q); the pixel lanes are reduced
// through LDS into one partial row per workgroup.  int8: the row is added into sums[B][C] with one
// atomic per channel (int32 addition is exact in any order; the buffer is zero on entry, the softmax
// kernel of every head clears what it used).  bf16: the S partial rows of a sample are stored and a
// second small kernel adds them in split order, so the float means never depend on the order in which
// workgroups ran.  (Handing the rows to the last-arriving workgroup of the same kernel was measured with a device-scope
// release per workgroup, which writes back the whole L2 of its XCD, and with agent-scope stores that need none: either way the
// hand-over takes some 4 us longer than the second launch.)
// Bound by HBM on large batches, by latency on small ones; eight loads in flight per lane, also for the last rows.
// Needs C * ES / 16 <= 256.
template <int ES>
__global__ __launch_bounds__(256) void gap_kernel(HeadArgs a, int pix_per_block, int S)
{
    request_args<sizeof(HeadArgs)>();
    constexpr int NE = 16 / ES, U = 8;
    __shared__ int red[256 * NE];
    const int cchunks = a.C * ES / 16;
    const int npl = 256 / cchunks;
    const int unit = xcd_unit(blockIdx.x, a.B * S);
    if (unit < 0) return;
    const int b = unit / S, split = unit - b * S;
    const int q = (int)threadIdx.x % cchunks, pl = (int)threadIdx.x / cchunks;
    const bool active = pl < npl;
    const int p0 = split * pix_per_block, p1 = min(a.HW, p0 + pix_per_block);
    const long long bs = a.slots ? (long long)a.slots[b] : (long long)b;      // zero-copy compaction: sample b of the batch is slot slots[b] of act
    const unsigned char* x = (const unsigned char*)a.act + bs * a.HW * a.C * ES;
    int acci[NE];
    float accf[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) { acci[e] = 0; accf[e] = 0.f; }
    auto add = [&](const v4i& xv) {
        if constexpr (ES == 1) {
#pragma unroll
            for (int e = 0; e < 16; ++e) acci[e] += __builtin_amdgcn_sbfe(xv[e >> 2], 8 * (e & 3), 8);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) accf[e] += bf16_to_f32_m((uint16_t)((unsigned)xv[e >> 1] >> (16 * (e & 1))));
        }
    };
    if (active) {
        const v4i* row = (const v4i*)(x + q * 16);
        const long long pitch = cchunks;                       // 16-byte chunks per pixel
        int p = p0 + pl;
        for (; p + (U - 1) * npl < p1; p += U * npl) {
            v4i xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) xv[u] = row[(p + u * npl) * pitch];
#pragma unroll
            for (int u = 0; u < U; ++u) add(xv[u]);
        }
        for (; p < p1; p += 4 * npl) {                         // what is left, four at a time: rows past the end read the last one and count nothing
            v4i xv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) xv[u] = row[min(p + u * npl, p1 - 1) * pitch];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (p + u * npl < p1) add(xv[u]);
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            if constexpr (ES == 1) red[pl * a.C + q * NE + e] = acci[e];
            else red[pl * a.C + q * NE + e] = __float_as_int(accf[e]);
        }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < a.C; c += 256) {
        if constexpr (ES == 1) {
            int s = 0;
            for (int l = 0; l < npl; ++l) s += red[l * a.C + c];
            atomicAdd(&a.sums[(long long)b * a.C + c], s);
        } else {
            float s = 0.f;
            for (int l = 0; l < npl; ++l) s += __int_as_float(red[l * a.C + c]);
            if (S == 1) a.sums[(long long)b * a.C + c] = __float_as_int(s / (float)a.HW);
            else a.gap_partial[((long long)b * S + split) * a.C + c] = __float_as_int(s);
        }
    }
}

// Images of up to GAP_SLICE_PIXELS pixels: a workgroup per (sample, SCH chunks of 16 bytes of its channels) adds up every pixel, so that nothing is left to a second launch (bf16) or to atomics (int8).  Sums in a
// fixed order: 1024 / SCH lanes per chunk take every pixel of their turn, a tree over the wavefront, then the 16 wavefronts in turn.
template <int ES, int SCH>
__global__ __launch_bounds__(1024) void gap_slice_kernel(HeadArgs a, int slices)
{
    request_args<sizeof(HeadArgs)>();
    using T = std::conditional_t<ES == 1, int, float>;
    constexpr int NE = 16 / ES, NPL = 1024 / SCH, U = 8;
    __shared__ T red[16][SCH * NE];
    const int unit = xcd_unit(blockIdx.x, a.B * slices);
    if (unit < 0) return;
    const int b = unit / slices, tid = threadIdx.x, q = tid % SCH, pl = tid / SCH;
    const int cchunks = a.C / NE, chunk = (unit - b * slices) * SCH + q;
    const long long bs = a.slots ? (long long)a.slots[b] : (long long)b;
    const v4i* row = (const v4i*)((const unsigned char*)a.act + bs * a.HW * a.C * ES) + min(chunk, cchunks - 1);
    T acc[NE] = {};
    for (int p = pl; p < a.HW; p += U * NPL) {
        v4i xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = row[(long long)min(p + u * NPL, a.HW - 1) * cchunks];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (p + u * NPL < a.HW)
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    if constexpr (ES == 1) acc[e] += __builtin_amdgcn_sbfe(xv[u][e >> 2], 8 * (e & 3), 8);
                    else acc[e] += bf16_to_f32_m((uint16_t)((unsigned)xv[u][e >> 1] >> (16 * (e & 1))));
                }
    }
#pragma unroll
    for (int o = SCH; o < 64; o <<= 1)
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
    if ((tid & 63) < SCH)
#pragma unroll
        for (int e = 0; e < NE; ++e) red[tid >> 6][q * NE + e] = acc[e];
    __syncthreads();
    const int c = (unit - b * slices) * SCH * NE + tid;
    if (tid >= SCH * NE || c >= a.C) return;
    T s = red[0][tid];
#pragma unroll
    for (int w = 1; w < 16; ++w) s += red[w][tid];
    if constexpr (ES == 1) a.sums[(long long)b * a.C + c] = s;
    else a.sums[(long long)b * a.C + c] = __float_as_int(s / (float)a.HW);
}

// bf16: sums[b][c] = (partial[b][0][c] + ... + partial[b][S-1][c]) / HW, 4 channels per lane
__global__ __launch_bounds__(256) void gap_reduce_kernel(HeadArgs a, int S)
{
    issue_first();
    request_args<sizeof(HeadArgs)>();
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;       // (b, c / 4)
    const int c4 = a.C / 4;
    if (idx >= (long long)a.B * c4) return;
    const long long b = idx / c4;
    const int c = (int)(idx - b * c4) * 4;
    const int* rows = a.gap_partial + b * S * a.C + c;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    constexpr int U = 8;                                                    // rows in flight
    for (int k0 = 0; k0 < S; k0 += U) {
        v4i v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = *(const v4i*)(rows + (long long)min(k0 + u, S - 1) * a.C);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + u < S) { s0 += __int_as_float(v[u][0]); s1 += __int_as_float(v[u][1]); s2 += __int_as_float(v[u][2]); s3 += __int_as_float(v[u][3]); }
    }
    // the same rounding as the single-split path: one division per channel
    v4i out = {__float_as_int(s0 / (float)a.HW), __float_as_int(s1 / (float)a.HW), __float_as_int(s2 / (float)a.HW), __float_as_int(s3 / (float)a.HW)};
    *(v4i*)(a.sums + b * a.C + c) = out;
}

// Workgroups: 512 where the pixels allow it (256-512 measured equal, 1024 and more slower: every workgroup ends with one atomic
// or a partial row per channel), at most 32 per sample (on a batch of 5, adding up 103 partial rows per sample took 13.7 us) and
// at least 16 pixels each.
static int gap_pixels_per_block(int B, int HW)
{
    const int splits = std::min(32, (512 + B - 1) / B);      // B * splits <= B + 511
    int ppb = (HW + splits - 1) / splits;
    if (ppb < 16) ppb = HW < 16 ? HW : 16;
    return ppb;
}

static int gap_pixel_splits(int B, int HW)
{
    const int ppb = gap_pixels_per_block(B, HW);
    return (HW + ppb - 1) / ppb;
}

// bf16: what the pooling by pixels would share out goes by slices of channels (gap_slice_kernel), which keep no partial rows
static bool gap_slices_bf16(int B, int HW) { return HW <= GAP_SLICE_PIXELS && gap_pixel_splits(B, HW) > 1; }

int head_gap_splits(int B, int HW)
{
    if (B <= 0 || HW <= 0) return 0;
    return gap_slices_bf16(B, HW) ? 1 : gap_pixel_splits(B, HW);
}

// Slices of channels while a workgroup's pixels are no more than it reads in about the time of a launch: the widest of up to 128 KB, and up to 256 bytes of a pixel rather than more than a workgroup
// per CU.  bf16, the two kernels / this one, us: 56x56x256, 5 samples 7.3 / 5.8 (in slices of 64 bytes; 7.2 in 128, 11.0 in 256), 64 22.1 / 18.1, 256 76.9 / 72.9; 28x28x512, 5 samples
// 7.8 / 4.5, 256 35.9 / 31.1; 14x14x1024, 5 samples 7.2 / 4.2, 64 10.0 / 6.4; 7x7x2048, 5 samples 7.3 / 3.7.  Where the batch is some 400 MB and more both are at the rate of HBM and within 4 %, the
// slices mostly ahead (64x64x384, 200 samples 123.8 / 115.5; behind at 64x64x512, 128 samples 98.8 / 102.7).
template <int ES>
static void launch_gap_slices(const HeadArgs& a, hipStream_t s)
{
    const int cchunks = a.C * ES / 16;
    int sch = 64;                                                       // chunks of 16 bytes per workgroup
    while (sch > 4 && (a.HW * sch * 16 > 128 * 1024 || sch / 2 >= cchunks)) sch /= 2;
    auto slices = [&] { return (cchunks + sch - 1) / sch; };
    while (sch < 16 && a.B * slices() > 256) sch *= 2;
#define EE_SLICE(SCH) if (sch == SCH) EE_LAUNCH((gap_slice_kernel<ES, SCH>), dim3(xcd_grid(a.B * slices())), dim3(1024), 0, s, a, slices())
    EE_SLICE(4);
    EE_SLICE(8);
    EE_SLICE(16);
    EE_SLICE(32);
    EE_SLICE(64);
#undef EE_SLICE
}

hipError_t launch_head_gap(const HeadArgs& a, int dtype, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    const int ppb = gap_pixels_per_block(a.B, a.HW);
    if (dtype == EE_I8) {
        // few pixels of many channels: us with atomics / by slices, 7x7x2048 1 to 64 samples 4.9-5.2 / 4.0-4.3, 256 8.9 / 6.7; 14x14x1024, 5 samples 4.7 / 4.5, 64 6.4 / 4.8; but 14x14x96 3.7 / 5.3,
        // 17x17x768 4.6 / 5.2 (37 samples and more 6.0 / 5.3), 28x28x512 4.3 / 5.8
        if (a.C >= 1024 && a.HW <= 256) {
            launch_gap_slices<1>(a, s);
            return hipGetLastError();
        }
        const int splits = gap_pixel_splits(a.B, a.HW);
        EE_LAUNCH(gap_kernel<1>, dim3(xcd_grid(a.B * splits)), dim3(256), 0, s, a, ppb, splits);
    } else {
        if (gap_slices_bf16(a.B, a.HW)) {
            launch_gap_slices<2>(a, s);
            return hipGetLastError();
        }
        const int splits = head_gap_splits(a.B, a.HW);
        // two kernels when the pooling is split: a timed launch takes the first one's begin and the second one's end
        const hipEvent_t t0 = g_launch_start, t1 = g_launch_stop;
        if (splits > 1) g_launch_stop = nullptr;
        EE_LAUNCH(gap_kernel<2>, dim3(xcd_grid(a.B * splits)), dim3(256), 0, s, a, ppb, splits);
        if (splits > 1) {
            const long long total = (long long)a.B * (a.C / 4);
            g_launch_start = nullptr;
            g_launch_stop = t1;
            EE_LAUNCH(gap_reduce_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a, splits);
            g_launch_start = t0;
        }
    }
    return hipGetLastError();
}

// ---- exit head, step 2: FC ------------------------------------------------------------------------------
// logits[b][j] = b_j + sum_c g[b][c] * W[j][c] as a 16 x 16 matrix-core tile per workgroup: rows = 16
// classes (A operand, ready operands of 1 KB a step: with rows read 64 bytes at a time the 2048-channel bf16 head of 16 samples took 9.7 us, now 6.8), columns = 16
// samples (B operand, the pooled features: requantised on the fly for int8; split into a bf16 head and
// a bf16 remainder for bf16 so that the float mean loses nothing that matters).  The NW wavefronts take
// every NWth 64-byte step of the reduction and add their partial tiles through LDS.  Bound by latency: a wavefront
// has the loads of four steps in flight with one tile of classes, of two with more, and NW is chosen so that one tile's reductions of up to 2 KB are all in flight at once.
//   v_mfma_i32_16x16x64_i8 / v_mfma_f32_16x16x32_bf16, lane l: row l%16, k-bytes [16*(l/16), +16);
//   D: column l%16, rows 4*(l/16) + v for accumulator register v = 0..3.
typedef float v4f_m __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf_m __attribute__((ext_vector_type(8)));

// TC: tiles of 16 classes per workgroup
template <int ES, int NW, int TC>
__global__ __launch_bounds__(64 * NW, 2) void fc_kernel(HeadArgs a)
{
    issue_first();
    request_args<sizeof(HeadArgs)>();
    constexpr int U = TC == 1 ? 4 : 2;                          // steps in flight per wavefront
    constexpr int Q = ES == 1 ? 4 : 2;                          // loads of a lane's features per step
    constexpr unsigned NOWHERE = 0x80000000u;                   // an offset past every buffer: reads zeros
    __shared__ int part[NW][TC * 256];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j0 = blockIdx.x * 16 * TC, b0 = blockIdx.y * 16;
    const int r = lane & 15, kq = lane >> 4;
    const int b = b0 + r;
    const int CB = a.C * ES;                                   // bytes per weight row (a multiple of 16, at most 4096)
    const int nsteps = (CB + 63) / 64, last_tile = (a.n_cls + 15) / 16 - 1;
    const bool bin = b < a.B;
    // Operands through buffers: a step past the last, a channel past the last and a sample past the batch read zeros, with no condition in front of a load; behind conditions the sixteen loads of
    // features went out one branch at a time.  Weights of zero past the last step as well, as an infinite one times zero is no number.  With the features requantised two at a time (32 instructions a
    // step instead of 84): 1000 classes, 256 samples, 2048 channels int8 8.4 -> 7.4 us, bf16 8.9 -> 8.4; 1024 channels 6.1 -> 5.1, 5.8 -> 5.4; 8x8 pixels and 64 samples 6.9 -> 6.0.
    const auto w_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.wfo), (short)0, (last_tile + 1) * nsteps * 1024, 0x00020000);
    const auto g_buf = __builtin_amdgcn_make_buffer_rsrc(a.sums + (long long)b0 * a.C, (short)0, min(16, a.B - b0) * a.C * 4, 0x00020000);
    const auto bias_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.bfc), (short)0, a.n_cls * 4, 0x00020000);
    constexpr int NB = (TC * 256 + 64 * NW - 1) / (64 * NW);    // results per lane
    int bias[NB];
    auto cls_of = [&](int i) { return j0 + i / 256 * 16 + 4 * kq + (i / 64) % 4; };      // element i of the partial tiles: this class of sample r
#pragma unroll
    for (int n = 0; n < NB; ++n) bias[n] = __builtin_amdgcn_raw_buffer_load_b32(bias_buf, cls_of(threadIdx.x + 64 * NW * n) * 4, 0, 0);
    const v4i zero4 = {0, 0, 0, 0};
    v4i acci[TC];
    v4f_m accf[TC];
#pragma unroll
    for (int t = 0; t < TC; ++t) { acci[t] = zero4; accf[t] = v4f_m{0.f, 0.f, 0.f, 0.f}; }
    const int shift = max(a.gap_shift, 0), rnd = shift > 0 ? 1 << (shift - 1) : 0;
    for (int s0 = wave; s0 < nsteps; s0 += U * NW) {
        v4i wv[U][TC], gv[U][Q];
#pragma unroll
        for (int u = 0; u < U; ++u) {                           // all loads of U steps first
            const int step = s0 + NW * u;
            const unsigned g_at = step * 64 + kq * 16 < CB ? (unsigned)(r * a.C + (step * 64 + kq * 16) / ES) * 4u : NOWHERE;
#pragma unroll
            for (int t = 0; t < TC; ++t) {
                const unsigned w_at = step < nsteps ? (unsigned)((min((int)blockIdx.x * TC + t, last_tile) * nsteps + step) * 1024) : NOWHERE;
                wv[u][t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w_buf, w_at + lane * 16, 0, 0));
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) gv[u][q] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(g_buf, g_at + 16 * q, 0, 0));
        }
        __builtin_amdgcn_sched_barrier(0);                      // (left to itself the compiler spreads them over the conversions)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (ES == 1) {
                v4i g8;
#pragma unroll
                for (int q = 0; q < 4; ++q) {                   // v_ashr_pk_i8_i32 shifts and saturates two sums at a time
                    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
                    g8[q] = __builtin_bit_cast(int, (u16x2{(unsigned short)__builtin_amdgcn_ashr_pk_i8_i32(gv[u][q][0] + rnd, gv[u][q][1] + rnd, shift),
                                                           (unsigned short)__builtin_amdgcn_ashr_pk_i8_i32(gv[u][q][2] + rnd, gv[u][q][3] + rnd, shift)}));
                }
#pragma unroll
                for (int t = 0; t < TC; ++t) acci[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wv[u][t], g8, acci[t], 0, 0, 0);
            } else {
                v4i hi = zero4, lo = zero4;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float g = __int_as_float(gv[u][e >> 2][e & 3]);
                    const uint16_t h = f32_to_bf16_rne_m(g);
                    const uint16_t l = f32_to_bf16_rne_m(g - bf16_to_f32_m(h));
                    hi[e >> 1] |= (int)((unsigned)h << (16 * (e & 1)));
                    lo[e >> 1] |= (int)((unsigned)l << (16 * (e & 1)));
                }
#pragma unroll
                for (int t = 0; t < TC; ++t) {
                    accf[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf_m, wv[u][t]), __builtin_bit_cast(v8bf_m, hi), accf[t], 0, 0, 0);
                    accf[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf_m, wv[u][t]), __builtin_bit_cast(v8bf_m, lo), accf[t], 0, 0, 0);
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < TC; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave][t * 256 + v * 64 + lane] = ES == 1 ? acci[t][v] : __float_as_int(accf[t][v]);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int i = threadIdx.x + 64 * NW * n, jj = cls_of(i);
        if (i >= TC * 256 || jj >= a.n_cls || !bin) continue;
        if constexpr (ES == 1) {
            int t = bias[n];
#pragma unroll
            for (int w = 0; w < NW; ++w) t += part[w][i];
            ((int*)a.logits)[(long long)b * a.n_cls + jj] = t;
        } else {
            float t = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) t += __int_as_float(part[w][i]);
            ((float*)a.logits)[(long long)b * a.n_cls + jj] = a.logit_scale * (t + __int_as_float(bias[n]));
        }
    }
}

template <int ES, int NW>
static void launch_fc(const HeadArgs& a, hipStream_t s)
{
    const int tiles = (a.n_cls + 15) / 16, rows = (a.B + 15) / 16;
    // As many tiles per workgroup as leave a workgroup for every CU: a workgroup reads its samples' features whatever the number of its tiles.  1000 classes, us with 1 / 2 / 4 tiles:
    // 2048 channels, 64 samples (252 workgroups of one tile) int8 7.0 / 8.1 / 9.7, bf16 8.7 / 7.7 / 10.4; 128 (504) 11.0 / 7.8 / 9.2, 12.2 / 8.8 / 9.9; 256 (1008) 18.9 / 11.4 / 8.8,
    // 19.4 / 12.2 / 10.0; 256 channels, 256 samples 6.1 / 4.8 / 4.8, 5.8 / 5.0 / 5.0.
    const int tc = tiles * rows <= 256 ? 1 : (tiles + 1) / 2 * rows <= 256 ? 2 : 4;
    if (tc == 1) EE_LAUNCH((fc_kernel<ES, NW, 1>), dim3(tiles, rows), dim3(64 * NW), 0, s, a);
    else if (tc == 2) EE_LAUNCH((fc_kernel<ES, NW, 2>), dim3((tiles + 1) / 2, rows), dim3(64 * NW), 0, s, a);
    else EE_LAUNCH((fc_kernel<ES, NW, 4>), dim3((tiles + 3) / 4, rows), dim3(64 * NW), 0, s, a);
}

hipError_t launch_head_fc(const HeadArgs& a, int dtype, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    const bool wide = a.C * (dtype == EE_I8 ? 1 : 2) > 1024;      // more than the 16 steps four wavefronts have in flight with one tile of classes
    if (dtype == EE_I8) {
        if (wide) launch_fc<1, 8>(a, s);
        else launch_fc<1, 4>(a, s);
    } else {
        if (wide) launch_fc<2, 8>(a, s);
        else launch_fc<2, 4>(a, s);
    }
    return hipGetLastError();
}

// ---- exit head, step 3: softmax top-1 and the exit decision --------------------------------------------------
// 2^30 * 2^(-i/256), i = 0..255, rounded to nearest.
__constant__ uint32_t kExp2[256] = {
#include "exp2_table.inc"
};
static const uint32_t kExp2Host[256] = {
#include "exp2_table.inc"
};
const uint32_t* exp2_table_host() { return kExp2Host; }

// one workgroup per sample.  int8: m = max logit, label = lowest arg-max, S = sum_j T[frac(d_j)] >> (d_j >> f)
// with d_j = m - a_j (a base-2 softmax denominator in Q30); exits iff S <= s_thr.  bf16: float softmax.
// The sample's logits are read once into registers (PER per lane: n_cls <= 256 PER, the smallest of 1, 4 and 8, as every one costs a table lookup or an exponential also where it is no class); the
// arg-max and the denominator travel through one combined reduction.  Bound by latency: a chain of loads, two barriers and the decision.  Exchanges between lanes without the LDS unit (wave_all), all
// lookups in flight together and one barrier per reduction instead of two: with the FC's loads above, an exit step of 37 samples went from 436 to 429 us (four heads), one of a single sample on the
// mobile network from 155 to 151 (three).
template <int ES, int PER>
__global__ __launch_bounds__(256) void softmax_kernel(HeadArgs a)
{
    issue_first();
    request_args<sizeof(HeadArgs)>();
    __shared__ int all[4][4];
    __shared__ uint32_t exp2_lds[256];
    const int b = blockIdx.x, wave = threadIdx.x >> 6;
    uint32_t exp2_mine = 0;
    if constexpr (ES == 1) exp2_mine = kExp2[threadIdx.x];       // on its way with the logits: the terms then look it up in LDS
    const auto lg_buf = __builtin_amdgcn_make_buffer_rsrc((int*)a.logits + (long long)b * a.n_cls, (short)0, a.n_cls * 4, 0x00020000);
    int vi[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) vi[i] = __builtin_amdgcn_raw_buffer_load_b32(lg_buf, (threadIdx.x + 256 * i) * 4, 0, 0);
    auto is = [&](int i) { return (int)threadIdx.x + 256 * i < a.n_cls; };
    if constexpr (ES == 1) {
        // the pooled sums of this sample have been consumed by the FC: leave them zero for the next head
        for (int c = threadIdx.x; c < a.C; c += 256) a.sums[(long long)b * a.C + c] = 0;
        exp2_lds[threadIdx.x] = exp2_mine;                      // complete behind the barrier of the reduction
        int m = INT32_MIN;
#pragma unroll
        for (int i = 0; i < PER; ++i) m = is(i) ? max(m, vi[i]) : m;
        m = wave_all(m, [](int x, int y) { return max(x, y); });
        all[0][wave] = m;                                       // (every lane the same)
        __syncthreads();
        m = max(max(all[0][0], all[0][1]), max(all[0][2], all[0][3]));
        int arg = INT32_MAX;
        unsigned lo = 0, up = 0;                                // the terms' sum in two parts of 16 bits and more: each stays below 2^32 over the workgroup
        const int f = a.frac_bits;                              // 0 .. 30
        unsigned long long S = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const unsigned t = softmax_term_i8(m, vi[i], f, exp2_lds);
            S += is(i) ? t : 0u;
            arg = is(i) && vi[i] == m ? min(arg, (int)threadIdx.x + 256 * i) : arg;
        }
        lo = (unsigned)S & 0xFFFFu;
        up = (unsigned)(S >> 16);                               // S <= 8 * 2^30
        const auto sum = [](int x, int y) { return (int)((unsigned)x + (unsigned)y); };
        lo = wave_all((int)lo, sum);                            // integer sums and minima: exact in any order
        up = wave_all((int)up, sum);
        arg = wave_all(arg, [](int x, int y) { return min(x, y); });
        all[1][wave] = lo;
        all[2][wave] = up;
        all[3][wave] = arg;
        __syncthreads();
        if (threadIdx.x == 0) {
            arg = min(min(all[3][0], all[3][1]), min(all[3][2], all[3][3]));
            lo = all[1][0] + all[1][1] + all[1][2] + all[1][3];
            up = all[2][0] + all[2][1] + all[2][2] + all[2][3];
            head_decide_i8(a, b, arg, (long long)(((unsigned long long)up << 16) + lo));
        }
    } else {
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < PER; ++i) m = is(i) ? fmaxf(m, __int_as_float(vi[i])) : m;
        m = __int_as_float(wave_all(__float_as_int(m), [](int x, int y) { return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(y))); }));
        all[0][wave] = __float_as_int(m);
        __syncthreads();
        m = __int_as_float(all[0][0]);
#pragma unroll
        for (int w = 1; w < 4; ++w) m = fmaxf(m, __int_as_float(all[0][w]));
        int arg = INT32_MAX;
        float den = 0.f;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const float z = __int_as_float(vi[i]);
            const float t = expf(z - m);
            den = is(i) ? den + t : den;
            arg = is(i) && z == m ? min(arg, (int)threadIdx.x + 256 * i) : arg;
        }
        // a fixed tree: the float sum is reproducible
        den = __int_as_float(wave_all(__float_as_int(den), [](int x, int y) { return __float_as_int(__int_as_float(x) + __int_as_float(y)); }));
        arg = wave_all(arg, [](int x, int y) { return min(x, y); });
        all[1][wave] = __float_as_int(den);
        all[3][wave] = arg;
        __syncthreads();
        if (threadIdx.x == 0) {
            den = ((__int_as_float(all[1][0]) + __int_as_float(all[1][1])) + __int_as_float(all[1][2])) + __int_as_float(all[1][3]);
            arg = min(min(all[3][0], all[3][1]), min(all[3][2], all[3][3]));
            head_decide_bf16(a, b, arg, den);
        }
    }
}

template <int ES>
static void launch_softmax(const HeadArgs& a, hipStream_t s)
{
    if (a.n_cls <= 256) EE_LAUNCH((softmax_kernel<ES, 1>), dim3(a.B), dim3(256), 0, s, a);
    else if (a.n_cls <= 1024) EE_LAUNCH((softmax_kernel<ES, 4>), dim3(a.B), dim3(256), 0, s, a);
    else EE_LAUNCH((softmax_kernel<ES, 8>), dim3(a.B), dim3(256), 0, s, a);
}

hipError_t launch_head_softmax(const HeadArgs& a, int dtype, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    if (dtype == EE_I8) launch_softmax<1>(a, s);
    else launch_softmax<2>(a, s);
    return hipGetLastError();
}

// ---- the whole exit head in one launch, for small heads -----------------------------------------------------------
// A head over a few KiB of activations and few classes is three launches of 3-6 us whose work one workgroup does in one memory round trip
// or two: one workgroup per sample pools (or takes the sums the segment's last layer left), keeps the features in LDS, computes every
// logit (16 lanes share a weight row) and decides.  Bound by latency; the first weights are requested in front of the pooling.
// For heads of up to 32 KiB of activations and of weights (one CU then reads in less time than two more launches take) and 256 classes.
// Same integers as the three kernels; bf16: float features times bf16 weights in float.
// Measured: int8, 16x16x16 and 10 classes, 8 samples, the three kernels take 5.9 + 2.6 + 3.6 us; with this one launch and none for slot
// tables a stream of 64 requests in 8 slots (24 exit boundaries) went from 824 to 586 us.
template <int ES>
__global__ __launch_bounds__(256) void head_small_kernel(HeadArgs a, int pooled)
{
    request_args<sizeof(HeadArgs)>();
    constexpr int NE = 16 / ES, U = 4;
    __shared__ __attribute__((aligned(16))) int red[256 * NE];
    __shared__ __attribute__((aligned(16))) unsigned char feat[ES == 1 ? HEAD_SMALL_C : 2 * HEAD_SMALL_C];    // int8 features, or floats (C <= HEAD_SMALL_C / ES)
    __shared__ int lg[HEAD_SMALL_CLS];
    __shared__ uint32_t exp2_lds[256];
    const int tid = threadIdx.x, b = xcd_unit(blockIdx.x, a.B);
    if (b < 0) return;
    const int cchunks = a.C * ES / 16, CB = a.C * ES;
    const v4i w_first = head_weight(a, tid >> 4, tid & 15);
    const int b_first = head_bias(a, tid >> 4);
    if constexpr (ES == 1) exp2_lds[tid] = kExp2[tid];
    if (pooled) {
        for (int c = tid; c < a.C; c += 256) {
            int* sp = a.sums + (long long)b * a.C + c;          // int8 only
            const int s = *sp;
            *sp = 0;                                            // left zero for the next head
            feat[c] = head_feature_i8(a, s);
        }
    } else {
        const int npl = 256 / cchunks, q = tid % cchunks, pl = tid / cchunks;
        if (pl < npl) {
            const long long bs = a.slots ? (long long)a.slots[b] : (long long)b;
            const v4i* row = (const v4i*)((const unsigned char*)a.act + bs * a.HW * CB) + q;
            int acci[NE];
            float accf[NE];
#pragma unroll
            for (int e = 0; e < NE; ++e) { acci[e] = 0; accf[e] = 0.f; }
            for (int p = pl; p < a.HW; p += U * npl) {
                v4i xv[U];
#pragma unroll
                for (int u = 0; u < U; ++u) xv[u] = row[(long long)min(p + u * npl, a.HW - 1) * cchunks];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (p + u * npl < a.HW) {
                        if constexpr (ES == 1) {
#pragma unroll
                            for (int e = 0; e < 16; ++e) acci[e] += __builtin_amdgcn_sbfe(xv[u][e >> 2], 8 * (e & 3), 8);
                        } else {
#pragma unroll
                            for (int e = 0; e < 8; ++e) accf[e] += bf16_to_f32_m((uint16_t)((unsigned)xv[u][e >> 1] >> (16 * (e & 1))));
                        }
                    }
            }
#pragma unroll
            for (int e = 0; e < NE; ++e) red[pl * a.C + q * NE + e] = ES == 1 ? acci[e] : __float_as_int(accf[e]);
        }
        __syncthreads();
        for (int c = tid; c < a.C; c += 256) {
            if constexpr (ES == 1) {
                int s = 0;
                for (int l = 0; l < npl; ++l) s += red[l * a.C + c];
                feat[c] = head_feature_i8(a, s);
            } else {
                float s = 0.f;
                for (int l = 0; l < npl; ++l) s += __int_as_float(red[l * a.C + c]);
                ((float*)feat)[c] = s / (float)a.HW;
            }
        }
    }
    __syncthreads();
    head_logits_decide<ES, 256>(a, b, feat, lg, exp2_lds, tid, w_first, b_first);
}

bool head_small_weights(long long row, int n_cls) { return n_cls <= HEAD_SMALL_CLS && row <= HEAD_SMALL_C && row * n_cls <= 32 * 1024; }

bool head_small(const HeadArgs& a, int dtype, bool pooled)
{
    const long long es = dtype == EE_I8 ? 1 : 2, row = a.C * es;
    return head_small_weights(row, a.n_cls) && (pooled ? dtype == EE_I8 : row * a.HW <= 32 * 1024);
}

hipError_t launch_head_small(const HeadArgs& a, int dtype, bool pooled, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    if (dtype == EE_I8) EE_LAUNCH(head_small_kernel<1>, dim3(xcd_grid(a.B)), dim3(256), 0, s, a, (int)pooled);
    else EE_LAUNCH(head_small_kernel<2>, dim3(xcd_grid(a.B)), dim3(256), 0, s, a, (int)pooled);
    return hipGetLastError();
}

// ---- scratch memory that is part of the library image --------------------------------------------------------
// The exit head needs device memory beyond its inputs and outputs: the pooled sums, the partial rows of the
// float pooling and the logits.  ee_exit_head takes them from the context's workspace; ee_exit_head_static
// takes them from this array, so that the call allocates nothing.  Every GPU holds its own copy of the array
// at its own address: the address is looked up once per device, with that device current, and host code only
// ever uses the looked-up pointer (the array's name is not a device address on the host side).
static __device__ __align__(256) unsigned char scratch[EE_STATIC_SCRATCH_BYTES];

hipError_t static_scratch(void** out)
{
    static void* ptr_of_device[64] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    void* p = __atomic_load_n(&ptr_of_device[dev], __ATOMIC_ACQUIRE);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        __atomic_store_n(&ptr_of_device[dev], p, __ATOMIC_RELEASE);      // the same value from every thread that races here
    }
    *out = p;
    return hipSuccess;
}

__global__ __launch_bounds__(256) void fill_zero_kernel(v4i* p, long long n16)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    const v4i z = {0, 0, 0, 0};
    if (i < n16) p[i] = z;
}

// ---- slot tables of a step: kernel arguments -> device memory ---------------------------------------------
// It stands between the host's decision at an exit and the next segment's first layer.  1 KB of arguments costs the host 1.5 us more per launch than a few words and the kernel 1 us to fetch, so batches of up to 64
// samples bring a quarter of them.
struct SlotPair64 { uint16_t in[64], out[64]; };
__global__ __launch_bounds__(64) void upload_slots_kernel(SlotPair64 t, uint16_t* dst)
{
    issue_first();
    dst[threadIdx.x] = t.in[threadIdx.x];
    dst[EE_ZC_MAX_B + threadIdx.x] = t.out[threadIdx.x];
}
__global__ __launch_bounds__(256) void upload_slots_kernel(SlotTab in, SlotTab out, uint16_t* dst)
{
    issue_first();
    dst[threadIdx.x] = in.s[threadIdx.x];
    dst[EE_ZC_MAX_B + threadIdx.x] = out.s[threadIdx.x];
}

hipError_t launch_upload_slots(const SlotTab& in, const SlotTab& out, int b, uint16_t* dst, hipStream_t s)
{
    if (b <= 64) {
        SlotPair64 t;
        std::memcpy(t.in, in.s, sizeof t.in);
        std::memcpy(t.out, out.s, sizeof t.out);
        EE_LAUNCH(static_cast<void (*)(SlotPair64, uint16_t*)>(upload_slots_kernel), dim3(1), dim3(64), 0, s, t, dst);
    } else EE_LAUNCH(static_cast<void (*)(SlotTab, SlotTab, uint16_t*)>(upload_slots_kernel), dim3(1), dim3(EE_ZC_MAX_B), 0, s, in, out, dst);
    return hipGetLastError();
}

// bytes [0, round-up-to-16(bytes)) of p become zero; a kernel, not a memset node, so that it may be captured
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s)
{
    const long long n16 = (long long)((bytes + 15) / 16);
    if (n16 == 0) return hipSuccess;
    EE_LAUNCH(fill_zero_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, s, (v4i*)p, n16);
    return hipGetLastError();
}

// ---- compaction and refill: survivors keep their order, newcomers follow behind them ------------------------
// A workgroup per (row, chunk of 16 KiB), b_act + b_incr rows: row b < b_act is a slot of the batch, the rows behind are the newcomers.  Bound by
// HBM: every sample that stays is read and written once.  A workgroup's four 16-byte loads per lane are on their way before it
// works out where its sample goes (each wavefront by itself: number of survivors in front of the slot by ballots over the
// flags, no barrier), and the stores are non-temporal: a line that is only written does not displace the sources in L2.
// 144 of 200 samples of 1.6 MB: 99 us (4 loads behind two barriers, plain stores) -> 69 us = 6.7 TB/s, with 56 newcomers behind them 108 us =
// 6.0 TB/s (torch's copy of 1 GiB: 5.2 TB/s); eight loads per lane and non-temporal loads were 4 and 13 % slower.  ring_rows > 0: dst is
// a ring of that many sample rows and the destination row wraps around its end.
__global__ __launch_bounds__(256) void compact_kernel(const uint8_t* flag, const unsigned char* src, unsigned char* dst,
                                                      const int32_t* ids_src, int32_t* ids_dst, int b_act, const unsigned char* refill,
                                                      const int32_t* refill_ids, int b_incr, long long sample_bytes, int dst_off, int ring_rows,
                                                      int* b_rem_out, int* b_merged_out)
{
    issue_first();
    const int chunks = (int)((sample_bytes + 16383) / 16384), unit = xcd_unit(blockIdx.x, (b_act + b_incr) * chunks);
    if (unit < 0) return;
    const int b = unit / chunks, chunk = unit - b * chunks, lane = threadIdx.x & 63;
    const bool fresh = b >= b_act;
    const bool books = chunk == 0 && b == 0 && (b_rem_out || b_merged_out);      // this workgroup also reports the counts
    const bool gone = !fresh && flag[b] != 0;
    if (gone && !books) return;
    const long long c0 = (long long)chunk * 16384;
    const v4i* s4 = (const v4i*)((fresh ? refill + (long long)(b - b_act) * sample_bytes : src + (long long)b * sample_bytes) + c0) + threadIdx.x;
    const long long n16 = (sample_bytes - c0) / 16;
    v4i v[4];
    if (n16 >= 1024 && !gone) {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = s4[256 * u];
    }
    const int upto = books || fresh ? b_act : b;
    int before = 0, total = 0;
    for (int t0 = 0; t0 < upto; t0 += 64) {
        const int t = t0 + lane;
        const bool alive = t < upto && flag[t] == 0;
        total += __popcll(__ballot(alive));
        before += __popcll(__ballot(alive && t < b));
    }
    if (books && threadIdx.x == 0) {
        if (b_rem_out) *b_rem_out = total;
        if (b_merged_out) *b_merged_out = total + b_incr;
    }
    if (gone) return;
    int d = dst_off + before + (fresh ? b - b_act : 0);
    if (ring_rows > 0 && d >= ring_rows) d -= ring_rows;
    if (chunk == 0 && threadIdx.x == 0 && ids_dst) {
        if (fresh ? refill_ids != nullptr : ids_src != nullptr) ids_dst[d] = fresh ? refill_ids[b - b_act] : ids_src[b];
    }
    v4i* d4 = (v4i*)(dst + (long long)d * sample_bytes + c0) + threadIdx.x;
    if (n16 >= 1024) {
#pragma unroll
        for (int u = 0; u < 4; ++u) __builtin_nontemporal_store(v[u], d4 + 256 * u);
    } else {
        for (int i = 0; i + (int)threadIdx.x < n16; i += 256) d4[i] = s4[i];
    }
}

// the counts of an empty batch (a kernel, not a memset node, so that it may be captured)
__global__ void zero_counts_kernel(int* b_rem_out, int* b_merged_out)
{
    if (b_rem_out) *b_rem_out = 0;
    if (b_merged_out) *b_merged_out = 0;
}

hipError_t launch_compact(const uint8_t* flag, const void* src, void* dst, const int32_t* ids_src, int32_t* ids_dst, int b_act,
                          const void* refill, const int32_t* refill_ids, int b_incr, int64_t sample_bytes, int dst_off, int ring_rows,
                          int* b_rem_out, int* b_merged_out, hipStream_t s)
{
    if (b_act + b_incr <= 0) {
        if (!b_rem_out && !b_merged_out) return hipSuccess;
        EE_LAUNCH(zero_counts_kernel, dim3(1), dim3(1), 0, s, b_rem_out, b_merged_out);
        return hipGetLastError();
    }
    const dim3 grid(xcd_grid((sample_bytes + 16383) / 16384 * (b_act + b_incr)));
    EE_LAUNCH(compact_kernel, grid, dim3(256), 0, s, flag, (const unsigned char*)src, (unsigned char*)dst, ids_src, ids_dst, b_act,
              (const unsigned char*)refill, refill_ids, b_incr, (long long)sample_bytes, dst_off, ring_rows, b_rem_out, b_merged_out);
    return hipGetLastError();
}

// ---- admission: whole samples copied to given slots ------------------------------------------------------------
// slot k = pool row ids[k]
__global__ __launch_bounds__(256) void copy_rows_kernel(const unsigned char* src, unsigned char* dst, const int32_t* gather_ids, int rows, long long sample_bytes)
{
    const int chunks = (int)((sample_bytes + 16383) / 16384), unit = xcd_unit(blockIdx.x, rows * chunks);
    if (unit < 0) return;
    const int k = unit / chunks;
    const long long row = gather_ids[k];
    const long long c0 = (long long)(unit - k * chunks) * 16384;
    const v4i* s4 = (const v4i*)(src + row * sample_bytes + c0);
    v4i* d4 = (v4i*)(dst + (long long)k * sample_bytes + c0);
    const long long n16 = min((long long)1024, (sample_bytes - c0) / 16);
    for (long long i = threadIdx.x; i < n16; i += 256) d4[i] = s4[i];
}

hipError_t launch_admit(const void* pool, void* dst, const int32_t* ids, int b, int64_t sample_bytes, hipStream_t s)
{
    if (b <= 0) return hipSuccess;
    const dim3 grid(xcd_grid((sample_bytes + 16383) / 16384 * b));
    EE_LAUNCH(copy_rows_kernel, grid, dim3(256), 0, s, (const unsigned char*)pool, (unsigned char*)dst, ids, b, (long long)sample_bytes);
    return hipGetLastError();
}

}  // namespace ee
