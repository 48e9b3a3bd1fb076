// Device code shared by the kernels that end in an exit decision (gfx950): features, terms of the integer softmax, the decision and its
// record for the host.
#pragma once
#include <type_traits>

#include "ee_internal.hpp"

namespace ee {
namespace {

typedef int v4i_h __attribute__((ext_vector_type(4)));

// A sample's record for the host: one 16-byte store into pinned host memory.  Both 64-bit words carry the launch's tag, so
// the host sees by itself when a record is complete (an aligned 64-bit word arrives whole): no fence, no counter of
// workgroups and no word behind them on the device side, and the host reads a record as soon as it lands.
__device__ __forceinline__ void host_record(HostOutcome* dst, uint64_t payload, int label, unsigned flag, unsigned tag)
{
    const uint64_t w0 = payload | (uint64_t)tag << EE_OUTCOME_TAG_SHIFT;
    const uint64_t w1 = (uint64_t)(unsigned)label | (uint64_t)(flag & 1u) << 32 | (uint64_t)tag << EE_OUTCOME_TAG_SHIFT;
    const v4i_h rec = {(int)(unsigned)w0, (int)(unsigned)(w0 >> 32), (int)(unsigned)w1, (int)(unsigned)(w1 >> 32)};
    *(v4i_h*)dst = rec;
}

// term of the base-2 softmax denominator: T[frac(d)] >> (d >> f), d = m - v
__device__ __forceinline__ unsigned softmax_term_i8(int m, int v, int f, const uint32_t* table)
{
    const unsigned d = (unsigned)m - (unsigned)v;                // 0 .. 2^32 - 1
    const unsigned q = d >> f, frac = d & ((1u << f) - 1u);
    const unsigned r = f >= 8 ? frac >> (f - 8) : frac << (8 - f);
    return table[r] >> min(q, 31u);                              // (the table is below 2^31; no condition the lookup would be behind)
}
// the exit decision of sample b and its outcome (one lane)
__device__ __forceinline__ void head_decide_i8(const HeadArgs& a, int b, int arg, long long S)
{
    const float conf = (float)(1073741824.0 / (double)S);
    const uint8_t flag = (uint8_t)(a.last || S <= a.s_thr);
    a.label[b] = arg;
    a.score[b] = S;
    a.conf[b] = conf;
    a.flag[b] = flag;
    if (a.host_out) host_record(a.host_out + b, (uint64_t)S, arg, flag, a.tag);
}
__device__ __forceinline__ void head_decide_bf16(const HeadArgs& a, int b, int arg, float den)
{
    const float conf = 1.0f / den;
    const uint8_t flag = (uint8_t)(a.last || conf >= a.thr);
    a.label[b] = arg;
    a.score[b] = 0;
    a.conf[b] = conf;
    a.flag[b] = flag;
    if (a.host_out) host_record(a.host_out + b, (uint64_t)__float_as_uint(conf), arg, flag, a.tag);
}

// the int8 feature of a channel's sum
__device__ __forceinline__ unsigned char head_feature_i8(const HeadArgs& a, int s)
{
    return (unsigned char)min(max(a.gap_shift > 0 ? (s + (1 << (a.gap_shift - 1))) >> a.gap_shift : s, -128), 127);
}

// v of the lane n places further round a row of 16 lanes: a reduction over the row takes rotations by 8, 4, 2, 1
template <int N>
__device__ __forceinline__ int row_rotate(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, false); }
__device__ __forceinline__ int row_sum(int v)
{
    v += row_rotate<8>(v);
    v += row_rotate<4>(v);
    v += row_rotate<2>(v);
    return v + row_rotate<1>(v);
}

// op over the 64 lanes, in every lane.  In the order of exchanges over 32, 16, 8, 4, 2 and 1 lanes (a rotation of what is already the same every 2 N lanes is that exchange), so a
// float sum has the bits of that tree; without the round trip through the LDS unit per exchange.
template <typename OP>
__device__ __forceinline__ int wave_all(int v, OP op)
{
    const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = op((int)h[0], (int)h[1]);
    const auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = op((int)q[0], (int)q[1]);
    v = op(v, row_rotate<8>(v));
    v = op(v, row_rotate<4>(v));
    v = op(v, row_rotate<2>(v));
    return op(v, row_rotate<1>(v));
}

__device__ __forceinline__ float head_bf16_f32(uint16_t v) { return __uint_as_float((unsigned)v << 16); }

// ---- what is behind the features of a small head (at most HEAD_SMALL_CLS classes) ---------------------------------------
constexpr int HEAD_SMALL_C = 4096, HEAD_SMALL_CLS = 256;
// chunk k of 16 weight bytes of class j; zeros outside the matrix
__device__ __forceinline__ v4i_h head_weight(const HeadArgs& a, int j, int k)
{
    const int CB = a.C * (a.es == 2 ? 2 : 1);
    return j < a.n_cls && k < CB / 16 ? *(const v4i_h*)((const unsigned char*)a.wfc + (long long)j * CB + k * 16) : v4i_h{0, 0, 0, 0};
}
// the bias of class j (integer or float bits)
__device__ __forceinline__ int head_bias(const HeadArgs& a, int j) { return j < a.n_cls ? ((const int*)a.bfc)[j] : 0; }
// Sample b's logits from its features in LDS (int8 features, or floats), 16 lanes per weight row, NT lanes in all, then the decision by the first
// wavefront: softmax_kernel's arithmetic.  w_first, b_first: the lane's first
// weight chunk (class tid / 16, chunk tid % 16) and that class's bias, requested early.  Contains a barrier.
template <int ES, int NT>
__device__ __forceinline__ void head_logits_decide(const HeadArgs& a, int b, const unsigned char* feat, int* lg, const uint32_t* exp2_lds, int tid, const v4i_h& w_first, int b_first)
{
    constexpr int PC = NT / 16;                                  // classes at a time
    const int lane = tid & 63, cchunks = a.C * ES / 16, part = tid & 15, j0 = tid >> 4;
    for (int j = j0; j < (a.n_cls + PC - 1) / PC * PC; j += PC) {
        int ti = 0;
        float tf = 0.f;
        for (int k = part; k < cchunks; k += 16) {
            const v4i_h w = j == j0 && k == part ? w_first : head_weight(a, j, k);
            if constexpr (ES == 1) {
                const v4i_h g = *(const v4i_h*)(feat + k * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) ti = __builtin_amdgcn_sdot4(w[e], g[e], ti, false);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) tf = fmaf(head_bf16_f32((uint16_t)((unsigned)w[e >> 1] >> (16 * (e & 1)))), ((const float*)feat)[k * 8 + e], tf);
            }
        }
        if constexpr (ES == 1) ti = row_sum(ti);
        else {
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) tf += __shfl_xor(tf, o, 64);
        }
        if (part == 0 && j < a.n_cls) {
            const int bias = j == j0 ? b_first : ((const int*)a.bfc)[j];
            const int v = ES == 1 ? ti + bias : __float_as_int(a.logit_scale * (tf + __int_as_float(bias)));
            lg[j] = v;
            ((int*)a.logits)[(long long)b * a.n_cls + j] = v;
        }
    }
    __syncthreads();
    if (tid >= 64) return;
    constexpr int PER = HEAD_SMALL_CLS / 64;
    int vi[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) vi[i] = lane + 64 * i < a.n_cls ? lg[lane + 64 * i] : (ES == 1 ? INT32_MIN : __float_as_int(-INFINITY));
    int arg = INT32_MAX;
    const auto lesser = [](int x, int y) { return min(x, y); };
    if constexpr (ES == 1) {
        int m = INT32_MIN;
#pragma unroll
        for (int i = 0; i < PER; ++i) m = max(m, vi[i]);
        m = wave_all(m, [](int x, int y) { return max(x, y); });
        unsigned long long S = 0;
        const int f = a.frac_bits;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (64 * i >= a.n_cls) break;
            const bool in = lane + 64 * i < a.n_cls;
            const unsigned t = softmax_term_i8(m, vi[i], f, exp2_lds);
            arg = in && vi[i] == m ? min(arg, lane + 64 * i) : arg;
            S += in ? t : 0u;
        }
        // in two parts, the lower 16 bits and the rest (a lane's sum is at most 4 * 2^30): each stays below 2^32 over the wavefront
        const auto sum = [](int x, int y) { return (int)((unsigned)x + (unsigned)y); };
        const unsigned lo = (unsigned)wave_all((int)((unsigned)S & 0xFFFFu), sum), up = (unsigned)wave_all((int)(unsigned)(S >> 16), sum);
        arg = wave_all(arg, lesser);
        if (lane == 0) head_decide_i8(a, b, arg, (long long)(((unsigned long long)up << 16) + lo));
    } else {
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < PER; ++i) m = fmaxf(m, __int_as_float(vi[i]));
        m = __int_as_float(wave_all(__float_as_int(m), [](int x, int y) { return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(y))); }));
        float den = 0.f;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (64 * i >= a.n_cls) break;
            const bool in = lane + 64 * i < a.n_cls;
            const float z = __int_as_float(vi[i]), t = expf(z - m);
            arg = in && z == m ? min(arg, lane + 64 * i) : arg;
            den = in ? den + t : den;
        }
        den = __int_as_float(wave_all(__float_as_int(den), [](int x, int y) { return __float_as_int(__int_as_float(x) + __int_as_float(y)); }));
        arg = wave_all(arg, lesser);
        if (lane == 0) head_decide_bf16(a, b, arg, den);
    }
}

}  // namespace
}  // namespace ee
