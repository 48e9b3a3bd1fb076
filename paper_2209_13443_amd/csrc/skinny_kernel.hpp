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

typedef float v4f_s __attribute__((ext_vector_type(4)));

// T: 32 (v_mfma 32x32, 32 bytes of the reduction per step) or 16 (16x16, 64 bytes; D: column l%16, rows 4*(l/16) + v).  NW:
// wavefronts sharing the reduction; TN: blocks of T channels; PLAIN: 1x1 kernel without padding
// block: the workgroup's number among those of this layer
template <int ES, int T, int NW, int TN, bool PLAIN>
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
    const unsigned nx = a.xs ? (unsigned)a.xs[n] : n;       // zero-copy compaction: sample n is slot xs[n] of x
    const unsigned char* xrow = (const unsigned char*)a.x + (long long)(((int)nx * a.H + iy0) * a.W + ix0) * CiB;
    const int ntaps = a.kh * a.kw;
    unsigned mask = 0;                                      // bit r * kw + s: that tap is inside the image
    if (!PLAIN) {
        const int s_lo = max(0, -ix0), s_hi = min(a.kw, a.W - ix0), r_lo = max(0, -iy0), r_hi = min(a.kh, a.H - iy0);
        const unsigned colmask = s_hi > s_lo ? ((1u << s_hi) - 1u) & ~((1u << s_lo) - 1u) : 0u;
        const unsigned rowsel = r_hi > r_lo ? a.tap_rows & ((1u << (r_hi * a.kw)) - 1u) & ~((1u << (r_lo * a.kw)) - 1u) : 0u;
        mask = colmask * rowsel;
    }
    const int per = (nk + NW - 1) / NW, k0 = wave * per, k1 = min(nk, k0 + per);      // this wavefront's steps

    // ---- bias and residual of the results this lane finishes, requested first --------------------------------
    const bool finisher = NW == 1 || tid < QB * TN;
    int bias[QPT][4];
    uint2 resv[QPT];
    int fm[QPT], fc[QPT];
    bool fin[QPT];
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        const int q = tid + 64 * NW * i, l = q & 63;        // accumulator quad q: block q / QB, register group (q / 64) % G, lane l
        fm[i] = m0 + (l & (T - 1));
        fc[i] = n0 + (q / QB) * T + (T == 32 ? ((q >> 6) & 3) * 8 : 0) + 4 * (l / T);
        fin[i] = finisher && fm[i] < a.M && fc[i] < a.Co;
        if (fin[i]) {
            const v4i b4 = *(const v4i*)((const int*)a.bias + fc[i]);
#pragma unroll
            for (int e = 0; e < 4; ++e) bias[i][e] = b4[e];
            if (a.res) {
                const long long o = (long long)fm[i] * a.Co + fc[i];
                if constexpr (ES == 1) resv[i].x = *(const unsigned*)((const signed char*)a.res + o);
                else resv[i] = *(const uint2*)((const uint16_t*)a.res + o);
            }
        }
    }

    // ---- the reduction -----------------------------------------------------------------------------------------
    // operands are packed for T = 32: [32 rows][32 bytes][row + 32 * half][16]; a 16-row operand of 64 bytes is half of the rows of two of them
    const int row0 = nt * TN * T;                           // first weight row, a multiple of T
    auto weight = [&](int j, int k) -> const v4i* {
        const unsigned char* wo = (const unsigned char*)a.wo;
        if constexpr (T == 32) return (const v4i*)(wo + (((long long)((row0 >> 5) + j) * pitch + k) * 64 + lane) * 16);
        else {
            const int r = row0 + 16 * j;
            return (const v4i*)(wo + (((long long)(r >> 5) * pitch + 2 * k + (hi >> 1)) * 64 + (r & 16) + mrow + 32 * (hi & 1)) * 16);
        }
    };
    const unsigned char* zp = (const unsigned char*)a.zeros;
    int tap = 0, ts = 0, tc = 0, toff = 0;                  // the lane's position inside the patch
    {
        const int at = KB * k0 + 16 * hi;
        if (PLAIN) toff = at;
        else if (k0 < k1) {
            tap = at / CiB;
            tc = at - tap * CiB;
            const int r = tap / a.kw;
            ts = tap - r * a.kw;
            toff = (r * a.W + ts) * CiB + tc;
        }
    }
    const int row_jump = (a.W - a.kw) * CiB;
    v4i fx[2][U], fw[2][U][TN];
    auto request = [&](int buf, int k) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = k + u < k1;
            const bool ok = in && (PLAIN || (tap < ntaps && (mask >> tap) & 1u));
            fx[buf][u] = *(const v4i*)(ok ? xrow + toff : zp);
            const int kc = in ? k + u : k1 - 1;
#pragma unroll
            for (int j = 0; j < TN; ++j) fw[buf][u][j] = *weight(j, kc);
            toff += KB;
            if (!PLAIN) {
                tc += KB;
                while (tc >= CiB) {                         // at most four times: a pixel is at least 16 bytes
                    tc -= CiB;
                    ++tap;
                    if (++ts == a.kw) { ts = 0; toff += row_jump; }
                }
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
    if (k0 < k1) {
        request(0, k0);
        for (int k = k0; k < k1; k += 2 * U) {
            if (k + U < k1) request(1, k + U);
            multiply(0);
            if (k + U < k1) {
                if (k + 2 * U < k1) request(0, k + 2 * U);
                multiply(1);
            }
        }
    }

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

}  // namespace
}  // namespace ee
