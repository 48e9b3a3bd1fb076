// Matrix-core convolution for few output pixels (gfx950): the reduction of a 32-pixel tile split over the wavefronts of a workgroup,
// operands straight from global memory.
//
// With few pixels (small batches, and the deep layers of any batch) a layer is a handful of tiles whose reduction is
// long: in the staged kernel (kernels_igemm.hip) a workgroup then walks through its steps one copy round trip and one barrier after the
// other, 20-70 times, on a chip that is mostly idle.  What bounds such a launch is the length of that chain.  Here a workgroup
// owns 32 pixels x 32 TN channels and its NW wavefronts share the reduction axis: each reads its part of both operands into registers,
// several 32-byte steps at a time with the next ones in flight, multiplies, and the partial sums meet in LDS once.  No
// staging, no barrier inside the loop; the chain is one or two memory round trips long.  Weights are packed as ready operands
// ([32 channels][step][lane][16 bytes]: a wavefront's load is one contiguous KiB).  Every operand byte is used by one instruction only,
// so this is for launches that latency bounds: with many pixels the staged kernel's reuse wins (the tables and the rule in
// launch_conv_skinny's caller decide).
// Measured, launches back to back, best staged configuration -> this kernel: 7x7, 3x3, 512 -> 512 int8, 1 sample 10.1 -> 7.0 us (T = 32),
// 8 samples 10.2 -> 7.4 us; bf16, 5 samples 17.7 -> 11.7 us; 14x14, 1x1, 1024 -> 256 int8, 1 sample 4.6 -> 3.5 us.
#pragma once
#include "ee_internal.hpp"
#include "igemm_device.hpp"

namespace ee {
namespace {

constexpr unsigned SKINNY_NOWHERE = 0xffffff00u;         // bytes a buffer of operands reaches; offsets from there on read zeros

typedef float v4f_s __attribute__((ext_vector_type(4)));

// T: 32 (v_mfma 32x32, 32 bytes of the reduction per step) or 16 (16x16, 64 bytes; D: column l%16, rows 4*(l/16) + v).  NW:
// wavefronts sharing the reduction; TN: blocks of T channels
// MODE: a 1x1 kernel without padding (SKINNY_PLAIN) or taps (SKINNY_TAPS) of whole steps: all lanes of a step are inside one tap, so its place is kept in scalar registers, and both operands are read through
// buffers at (lane's offset + scalar offset).  A tap outside the image costs a lane three instructions then, an operand of weights none; in the general form, which keeps a lane's place in its own
// registers, a step is some twenty, half of a short launch's time (14x14, 3x3, 256 -> 256, one sample: 2,200 of 6,000 cycles before the last request was out).  All segments, us: ResNet-50 int8, one sample 174.0 -> 170.1 (22 of its launches), bf16, 5 samples
// 328.6 -> 323.2, Inception-style, 4 samples 315.9 -> 312.3.
// block: the workgroup's number among those of this layer
enum { SKINNY_ANY = 0, SKINNY_PLAIN = 1, SKINNY_TAPS = 2 };
template <int ES, int T, int NW, int TN, int MODE>
__device__ __forceinline__ void skinny_tile(const ConvArgs& a, int gn, unsigned magic_gn, int nk, int pitch, unsigned block)
{
    constexpr int U = 4;                                    // steps per group of loads; two groups in flight
    constexpr int G = T / 8 * (T == 32) + (T == 16);        // accumulator quads per block and lane: 4, or 1
    constexpr int QB = 64 * G;                              // quads (pixel, 4 channels) per block of T x T results
    constexpr int QPT = G * TN >= NW ? G * TN / NW : 1;     // quads a lane finishes
    constexpr int KB = 1024 / T;                            // bytes of the reduction per step
    using acc_t = typename std::conditional<T == 32, typename std::conditional<ES == 1, v16i, v16f>::type, typename std::conditional<ES == 1, v4i, v4f_s>::type>::type;
    __shared__ v4i part[NW > 1 ? NW : 1][NW > 1 ? TN * QB : 1];
    const int tid = threadIdx.x, lane = tid & 63, mrow = lane & (T - 1), hi = lane / T;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mt = (int)fast_div(block, (unsigned)gn, magic_gn), nt = (int)block - mt * gn;
    const int m0 = mt * T, n0 = nt * T * TN;
    const int CiB = a.Ci * ES;

    // ---- the lane's pixel as an operand row ------------------------------------------------------------------
    const int m = min(m0 + mrow, a.M - 1);
    const unsigned howo = (unsigned)(a.Ho * a.Wo);
    const unsigned n = fast_div((unsigned)m, howo, a.magic_howo), rem = (unsigned)m - n * howo;
    const unsigned oy = fast_div(rem, (unsigned)a.Wo, a.magic_wo), ox = rem - oy * a.Wo;
    const int iy0 = (int)oy * a.stride - a.pad, ix0 = (int)ox * a.stride - a.pad_w;
    unsigned nx = n;
    if (a.xs) {                                             // zero-copy compaction: sample n is slot xs[n] of x
        nx = a.xs[n];
        asm volatile("" : "+v"(nx));                        // waited for in here: else every launch waits at this point, for whatever it has in flight
    }
    const int ntaps = a.kh * a.kw;
    unsigned mask = 0;                                      // bit r * kw + s: that tap is inside the image
    if (MODE != SKINNY_PLAIN) {
        const int s_lo = max(0, -ix0), s_hi = min(a.kw, a.W - ix0), r_lo = max(0, -iy0), r_hi = min(a.kh, a.H - iy0);
        const unsigned colmask = s_hi > s_lo ? ((1u << s_hi) - 1u) & ~((1u << s_lo) - 1u) : 0u;
        const unsigned rowsel = r_hi > r_lo ? a.tap_rows & ((1u << (r_hi * a.kw)) - 1u) & ~((1u << (r_lo * a.kw)) - 1u) : 0u;
        mask = colmask * rowsel;
    }
    const int per = (nk + NW - 1) / NW, k0 = wave * per, k1 = min(nk, k0 + per);      // this wavefront's steps

    // ---- the reduction -----------------------------------------------------------------------------------------
    // operands are packed for T = 32: [32 rows][32 bytes][row + 32 * half][16]; a 16-row operand of 64 bytes is half of the rows of two of them
    const int row0 = nt * TN * T;                           // first weight row, a multiple of T
    const auto w_buf = __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(a.wo) + (long long)(row0 >> 5) * pitch * 1024, (short)0, SKINNY_NOWHERE, 0x00020000);      // begins with the tile's rows
    const int w_lane = T == 32 ? lane * 16 : (hi >> 1) * 1024 + (mrow + 32 * (hi & 1)) * 16;
    auto weight = [&](int j, int k) {
        const int r = (row0 & 31) + T * j;
        const int at = T == 32 ? ((r >> 5) * pitch + k) * 1024 : ((r >> 5) * pitch + 2 * k) * 1024 + (r & 16) * 16;
        return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w_buf, w_lane, at, 0));
    };
    const unsigned char* zp = (const unsigned char*)a.zeros;
    // the position inside the patch: the lane's (general form), or the wavefront's.  The buffer of the input begins where the first pixel's patch would, so that every lane's offset is positive; no tap
    // inside the image lies in front of x.
    const unsigned back = (unsigned)((a.pad * a.W + a.pad_w) * CiB);
    const auto x_buf = __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(a.x) - back, (short)0, SKINNY_NOWHERE, 0x00020000);
    const unsigned x_lane = (unsigned)((((int)nx * a.H + iy0) * a.W + ix0) * CiB) + back + 16 * hi;
    const unsigned char* xrow = (const unsigned char*)a.x + (long long)(((int)nx * a.H + iy0) * a.W + ix0) * CiB;
    int tap = 0, ts = 0, tc = 0, toff = 0;
    const int row_jump = (a.W - a.kw) * CiB;
    if (MODE == SKINNY_PLAIN) toff = KB * k0;
    else if (MODE == SKINNY_TAPS) {
        const int spt = CiB / KB;                           // steps of a tap
        tap = (int)fast_div((unsigned)k0, (unsigned)spt, a.magic_spt);
        tc = (k0 - tap * spt) * KB;
        const int r = (int)fast_div((unsigned)tap, (unsigned)a.kw, a.magic_kw);
        ts = tap - r * a.kw;
        toff = (r * a.W + ts) * CiB + tc;
    } else if (k0 < k1) {
        const int at = KB * k0 + 16 * hi;
        tap = at / CiB;
        tc = at - tap * CiB;
        const int r = tap / a.kw;
        ts = tap - r * a.kw;
        toff = (r * a.W + ts) * CiB + tc;
    }
    v4i fx[2][U], fw[2][U][TN];
    auto request = [&](int buf, int k) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = k + u < k1;
            if constexpr (MODE == SKINNY_ANY) {
                const bool ok = in && tap < ntaps && (mask >> tap) & 1u;
                fx[buf][u] = *(const v4i*)(ok ? xrow + toff : zp);
            } else {
                // in is uniform: as a condition of the address it would become a branch with a load on either side
                unsigned at = x_lane | (MODE == SKINNY_PLAIN && !in ? SKINNY_NOWHERE : 0u);
                if constexpr (MODE == SKINNY_TAPS) at = mask & (in ? 1u << tap : 0u) ? x_lane : SKINNY_NOWHERE;
                fx[buf][u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(x_buf, (int)at, toff, 0));
            }
            const int kc = in ? k + u : k1 - 1;
#pragma unroll
            for (int j = 0; j < TN; ++j) fw[buf][u][j] = weight(j, kc);
            toff += KB;
            if constexpr (MODE != SKINNY_PLAIN) {
                tc += KB;
                auto next_tap = [&] {
                    tc -= CiB;
                    ++tap;
                    if (++ts == a.kw) { ts = 0; toff += row_jump; }
                };
                if constexpr (MODE == SKINNY_TAPS) { if (tc >= CiB) next_tap(); }
                else
                    while (tc >= CiB) next_tap();           // at most four times: a pixel is at least 16 bytes
            }
        }
    };
    acc_t acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4 * G; ++v) acc[j][v] = 0;
    auto multiply = [&](int buf) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (T == 16 && ES == 1) acc[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[buf][u][j], fx[buf][u], acc[j], 0, 0, 0);
                else if constexpr (T == 16) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, fw[buf][u][j]), __builtin_bit_cast(v8bf, fx[buf][u]), acc[j], 0, 0, 0);
                else if constexpr (ES == 1) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw[buf][u][j], fx[buf][u], acc[j], 0, 0, 0);
                else acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, fw[buf][u][j]), __builtin_bit_cast(v8bf, fx[buf][u]), acc[j], 0, 0, 0);
            }
    };
    // bias and residual of the results this lane finishes (results past the layer's ends read its last ones)
    const bool finisher = NW == 1 || tid < QB * TN;
    v4i bias[QPT];
    uint2 resv[QPT];
    int fm[QPT], fc[QPT];
    bool fin[QPT];
    auto request_epilogue = [&] {
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            const int q = tid + 64 * NW * i, l = q & 63;    // accumulator quad q: block q / QB, register group (q / 64) % G, lane l
            fm[i] = m0 + (l & (T - 1));
            fc[i] = n0 + (q / QB) * T + (T == 32 ? ((q >> 6) & 3) * 8 : 0) + 4 * (l / T);
            fin[i] = finisher && fm[i] < a.M && fc[i] < a.Co;
            const int c = min(fc[i], (a.Co - 1) & ~3);
            bias[i] = *(const v4i*)((const int*)a.bias + c);
            // without a residual the bias again: one load on every path
            const unsigned char* const r = a.res ? (const unsigned char*)a.res : (const unsigned char*)a.bias;
            const long long o = a.res ? ((long long)min(fm[i], a.M - 1) * a.Co + c) * ES : 0;
            if constexpr (ES == 1) resv[i].x = *(const unsigned*)(r + o);
            else resv[i] = *(const uint2*)(r + o);
        }
    };
    // Two groups of steps in flight, those of the first group requested in front of anything else the tile reads.  The compiler counts the requests in flight on every path and takes the smaller number where
    // paths meet: with requests behind conditions, and bias and residual in front, a launch waited for the latter before its first operand was requested and for both groups before it multiplied one.
    if (k0 + U < k1) {
        request(0, k0);
        request(1, k0 + U);
        request_epilogue();
        int k = k0 + 2 * U;
        for (; k + U < k1; k += 2 * U) {
            multiply(0);
            request(0, k);
            multiply(1);
            request(1, k + U);
        }
        if (k < k1) {
            multiply(0);
            request(0, k);
            multiply(1);
            multiply(0);
        } else {
            multiply(0);
            multiply(1);
        }
    } else if (k0 < k1) {
        request(0, k0);
        request_epilogue();
        multiply(0);
    } else request_epilogue();

    // ---- partial sums meet; every lane finishes QPT quads ------------------------------------------------------------
    if constexpr (NW > 1) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                v4i v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = ES == 1 ? (int)acc[j][4 * g + e] : __float_as_int((float)acc[j][4 * g + e]);
                part[wave][(j * G + g) * 64 + lane] = v;
            }
        __syncthreads();
        if (!finisher) return;                              // whole wavefronts
    }
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        v4i t;
        if constexpr (NW > 1) {
            const int q = tid + 64 * NW * i;
            t = part[0][q];
#pragma unroll
            for (int w = 1; w < NW; ++w) {
                const v4i p = part[w][q];
#pragma unroll
                for (int e = 0; e < 4; ++e) t[e] = ES == 1 ? t[e] + p[e] : __float_as_int(__int_as_float(t[e]) + __int_as_float(p[e]));
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = ES == 1 ? (int)acc[i / G][4 * (i % G) + e] : __float_as_int((float)acc[i / G][4 * (i % G) + e]);
        }
        long long orow = fm[i];
        unsigned fn = 0;
        if (a.ys || a.gap_sums) fn = fast_div((unsigned)min(fm[i], a.M - 1), howo, a.magic_howo);
        if (a.ys && fin[i]) orow = (long long)a.ys[fn] * howo + ((unsigned)fm[i] - fn * howo);      // zero-copy compaction: sample n goes to slot ys[n]
        const long long o = orow * a.ldc + a.c_off + fc[i];
        if constexpr (ES == 1) {
            int q[4] = {0, 0, 0, 0};
            if (fin[i]) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    int v = t[e] + bias[i][e];              // the rounding constant is part of the bias
                    if (a.res) v += __builtin_amdgcn_sbfe((int)resv[i].x, 8 * e, 8) << a.res_shift;
                    q[e] = clamp_i32(v >> a.shift, a.lo, a.hi);
                }
                *(unsigned*)((signed char*)a.y + o) = pack4_i8(q[0], q[1], q[2], q[3]);
            }
            if (a.gap_sums) {
                // the exit head's pooling: T lanes hold the pixels of the same 4 channels; per sample among them they
                // add up and one lane adds to the sums (integers: exact in any order)
                const int n_first = (int)fast_div((unsigned)min(m0, a.M - 1), howo, a.magic_howo), n_last = (int)fast_div((unsigned)min(m0 + T - 1, a.M - 1), howo, a.magic_howo);
                for (int s = n_first; s <= n_last; ++s) {
                    int v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = (int)fn == s ? q[e] : 0;
#pragma unroll
                    for (int d = T / 2; d > 0; d >>= 1)
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += __shfl_xor(v[e], d, 64);
                    if (mrow == 0 && fc[i] < a.Co) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) atomicAdd(a.gap_sums + (long long)s * a.Co + fc[i] + e, v[e]);
                    }
                }
            }
        } else if (fin[i]) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __int_as_float(t[e]) + __int_as_float(bias[i][e]);
            if (a.res) {
                v[0] += __uint_as_float(resv[i].x << 16); v[1] += __uint_as_float(resv[i].x & 0xFFFF0000u);
                v[2] += __uint_as_float(resv[i].y << 16); v[3] += __uint_as_float(resv[i].y & 0xFFFF0000u);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fminf(fmaxf(v[e], a.f_lo), a.f_hi);
            uint2 out;
            out.x = pack2_bf16(v[0], v[1]);
            out.y = pack2_bf16(v[2], v[3]);
            *(uint2*)((uint16_t*)a.y + o) = out;
        }
    }
}

// whether 32-bit offsets reach the weights of a tile, at most 64 rows
inline bool skinny_reaches(const ConvArgs& a, int es) { return (long long)a.Kp * es * 64 < 1ll << 31; }

// the form a layer runs in, with its divisors set
inline int skinny_mode(ConvArgs& a, int es, int t)
{
    const int kb = 1024 / t, cib = a.Ci * es;
    // the input's buffer reaches 4 GiB (slots of zero-copy compaction lie in less than 2: ee_create); that of the weights begins with the tile's rows (skinny_reaches)
    if (cib % kb != 0 || ((long long)(a.M - 1) / (a.Ho * a.Wo) + 1) * a.H * a.W * cib >= 1ll << 31) return SKINNY_ANY;
    auto magic = [](int d) { return (unsigned)(0x100000000ull / (unsigned)d - (d == 1)); };
    a.magic_spt = magic(cib / kb);
    a.magic_kw = magic(a.kw);
    return a.kh == 1 && a.kw == 1 && a.pad == 0 && a.pad_w == 0 ? SKINNY_PLAIN : SKINNY_TAPS;
}

}  // namespace
}  // namespace ee
