// A whole small segment and its exit head in one launch (int8), for gfx950: networks on small images, whose layers are a few microseconds of
// launch, first load and last store around a few hundred cycles of arithmetic.  Layer by layer a step of such a segment is five launches (folded
// copy or slot tables, the layers, the head) that wait for one another; here one workgroup of eight wavefronts per sample does it all:
//   every layer's weights (ready operands) and biases are requested at once, asynchronously, into LDS, then the sample's input; a folded first
//   layer's super-pixels are built in LDS from the raw image;
//   a layer: (32 output pixels, 32 channels) per wavefront, the operands straight out of LDS (a lane's 16 bytes are one chunk of one tap, found through a
//   table of the layer's chunks; a tap outside the image reads zeros), requantised into the next tensor in LDS; one barrier;
//   the last layer also writes the segment's output and adds up its channel sums (one more matrix instruction with the identity turns a block so
//   that a lane holds one channel; integer sums are exact in any order);
//   the head: features, logits, decision, as head_small_kernel.
// Results are those of the separate kernels bit for bit.
//
// Measured on a network of 32 x 32 images (three segments of two 3x3 layers, 16 / 32 / 64 channels, 10 classes) against the layers' own launches, two
// processes of each in turn: all segments and heads 1 to 256 samples 81-101 us -> 53; streams of 64 requests one by one 2510-2740 -> 1770 us, 64 in 8 slots
// 557-617 -> 399, 2000 in 64 slots on two lanes 1090-1250 -> 700, 5000 in 256 slots 790-870 -> 590.  What bounds it (time stamps, 8.2 us a launch): latency.  0.6 us for the launch's arguments, 1.2 for the requests, 0.7 the folding, 1.5 to 2.5 a
// layer (300 instructions per item in one dependent chain and two wavefronts per SIMD), 1.3 the logits and the decision.
#include "ee_internal.hpp"
#include "head_device.hpp"
#include "igemm_device.hpp"
#include "ir_device.hpp"

namespace ee {

// SegRows (by_value): sample n is row src[n] of the input, row dst[n] of the output.  The kernel's first argument: read through the kernel-argument segment
typedef const __attribute__((address_space(4))) SegPlan* SegPlanPtr;
typedef const __attribute__((address_space(4))) SegLayer* SegLayerPtr;

__global__ __launch_bounds__(512) void segment_small_i8_kernel(SegRows, const SegPlan* plan, const void* x, void* y, int B, int by_value, const int32_t* ids, const uint16_t* xs,
                                                               const uint16_t* ys, int head, HeadArgs h)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char sg_lds[];
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Two round trips to memory in front of the first load of data: the arguments with the table of rows, then a line of every part of the plan that the layers read.  With the count of samples,
    // the other arguments, the row and the plan waited for one after the other a launch took 8.7 us, now 8.2; a stream of 24 such steps moves by less than two of its runs differ.
    request_args<explicit_args<decltype(segment_small_i8_kernel)>::bytes()>();
    const auto& a = *(SegPlanPtr)plan;
    {
        const __attribute__((address_space(4))) int* p = (const __attribute__((address_space(4))) int*)plan;
        const int x = [&]<int... LINE>(std::integer_sequence<int, LINE...>) { return (p[16 * LINE] ^ ...); }(std::make_integer_sequence<int, (int)(__builtin_offsetof(SegPlan, tab) + 63) / 64>{});
        asm volatile("" ::"s"(x));
    }
    const int b = xcd_unit(blockIdx.x, B);
    if (b < 0) return;
    const __attribute__((address_space(4))) int* tab = (const __attribute__((address_space(4))) int*)__builtin_amdgcn_kernarg_segment_ptr();
    const long long src_row = by_value ? tab[b] : ids ? ids[b] : xs ? (int)xs[b] : b;
    const long long dst_row = by_value ? tab[EE_SEG_ROWS + b] : ys ? (int)ys[b] : b;
    const unsigned lds0 = lds_addr(sg_lds);
    int* const l_sums = (int*)(sg_lds + a.sums_off);
    unsigned char* const l_feat = sg_lds + a.feat_off;
    int* const l_logits = (int*)(sg_lds + a.logits_off);
    uint32_t* const l_exp2 = (uint32_t*)(sg_lds + a.exp2_off);

    // ---- requests: input, weights, biases, tables --------------------------------------------------------------------------
    const unsigned char* in = (const unsigned char*)x + src_row * a.in_bytes;
    auto copy = [&](int to, const void* from, int instr) {              // 1 KiB per instruction, shared out over the wavefronts
        for (int i = wave; i < instr; i += 8) dma16(__builtin_amdgcn_readfirstlane(lds0 + (unsigned)(to + i * 1024)), (const unsigned char*)from + i * 1024 + lane * 16);
    };
    if (a.in_pitch == 16 * a.in_cpp) {                                  // pixels without gaps (and the raw image): the lanes past the end repeat the last chunk
        for (int i = wave; i < (a.in_chunks + 63) / 64; i += 8)
            dma16(__builtin_amdgcn_readfirstlane(lds0 + (unsigned)(a.in_off + i * 1024)), in + (long long)min(64 * i + lane, a.in_chunks - 1) * 16);
    } else {
        for (int q = tid; q < a.in_chunks; q += 512) {
            const v4i v = *(const v4i*)(in + (long long)q * 16);
            const int px = (int)fast_div((unsigned)q, (unsigned)a.in_cpp, a.magic_cpp), c = q - px * a.in_cpp;
            *(v4i*)(sg_lds + a.in_off + px * a.in_pitch + c * 16) = v;
        }
    }
    for (int l = 0; l < a.n; ++l) {
        const auto& L = *(SegLayerPtr)&a.layer[l];
        for (int i = wave; i < L.blocks * L.steps; i += 8) {
            const int cb = (int)fast_div((unsigned)i, (unsigned)L.steps, L.magic_steps), k = i - cb * L.steps;
            dma16(__builtin_amdgcn_readfirstlane(lds0 + (unsigned)(L.w_off + i * 1024)), (const unsigned char*)L.wo + ((long long)(cb * L.pitch + k) * 64 + lane) * 16);
        }
        copy(L.bias_off, L.bias, L.bias_kib);
    }
    copy(a.tab_off, plan->tab, a.tab_kib);
    if (head) copy(a.exp2_off, h.exp2, 1);
    const v4i w_first = head ? head_weight(h, tid >> 4, tid & 15) : v4i{0, 0, 0, 0};
    const int b_first = head ? head_bias(h, tid >> 4) : 0;
    if (tid < 4) *(int*)(sg_lds + a.zero_off + tid * 4) = 0;
    for (int i = tid; i < a.layer[a.n - 1].blocks * 32; i += 512) l_sums[i] = 0;
    wait_all_then_barrier<0>();
    if (a.fold) {
        // super-pixels (dy, dx, c) of 2 x 2 pixels x 4 channels of the zero-padded image
        for (int o = tid; o < a.fold_h * a.fold_w; o += 512) {
            const int ys0 = (int)fast_div((unsigned)o, (unsigned)a.fold_w, a.magic_fold_w), xs0 = o - ys0 * a.fold_w;
            unsigned char px[4][4];                                     // every byte requested before the first is used; clamped, then zeroed where there is none
            unsigned d[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int iy = min(max(2 * ys0 + (t >> 1) - a.fold_pad, 0), a.img_h - 1), ix = min(max(2 * xs0 + (t & 1) - a.fold_pad, 0), a.img_w - 1);
                const unsigned char* p = sg_lds + a.in_off + (iy * a.img_w + ix) * a.img_c;
#pragma unroll
                for (int c = 0; c < 4; ++c) px[t][c] = p[min(c, a.img_c - 1)];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int iy = 2 * ys0 + (t >> 1) - a.fold_pad, ix = 2 * xs0 + (t & 1) - a.fold_pad;
                const bool there = (unsigned)iy < (unsigned)a.img_h && (unsigned)ix < (unsigned)a.img_w;
                d[t] = px[t][0] | (a.img_c > 1 ? px[t][1] << 8 : 0) | (a.img_c > 2 ? px[t][2] << 16 : 0) | (a.img_c > 3 ? (unsigned)px[t][3] << 24 : 0);
                d[t] = there ? d[t] : 0;
            }
            *(v4i*)(sg_lds + a.fold_off + o * 16) = v4i{(int)d[0], (int)d[1], (int)d[2], (int)d[3]};
        }
        lds_barrier();
    }
    const v4i unit = ir_unit(m, hi);

    // ---- the layers ------------------------------------------------------------------------------------------------------------
    for (int l = 0; l < a.n; ++l) {
        const auto& D = *(SegLayerPtr)&a.layer[l];
        // the layer's description in scalar registers, requested together: read where they are used they are a scalar round trip each
        struct { int w_off, bias_off, tab, steps, blocks, co, src, src_pitch, dst, dst_pitch, res, res_pitch, H, W, Ho, Wo, kh, kw, stride, pad, pad_w, shift, res_shift, lo, hi; unsigned tap_rows, magic_wo, magic_blocks; } L =
            {D.w_off, D.bias_off, D.tab, D.steps, D.blocks, D.co, D.src, D.src_pitch, D.dst, D.dst_pitch, D.res, D.res_pitch, D.H, D.W, D.Ho, D.Wo, D.kh, D.kw, D.stride, D.pad, D.pad_w, D.shift, D.res_shift, D.lo, D.hi, D.tap_rows, D.magic_wo, D.magic_blocks};
        int zero_off = a.zero_off;
        asm volatile("" : "+s"(L.w_off), "+s"(L.bias_off), "+s"(L.tab), "+s"(L.steps), "+s"(L.blocks), "+s"(L.co), "+s"(L.src), "+s"(L.src_pitch), "+s"(L.dst), "+s"(L.dst_pitch), "+s"(L.res), "+s"(L.res_pitch), "+s"(zero_off));
        asm volatile("" : "+s"(L.H), "+s"(L.W), "+s"(L.Ho), "+s"(L.Wo), "+s"(L.kh), "+s"(L.kw), "+s"(L.stride), "+s"(L.pad), "+s"(L.pad_w), "+s"(L.shift), "+s"(L.res_shift), "+s"(L.lo), "+s"(L.hi), "+s"(L.tap_rows));
        const bool last = l == a.n - 1;
        const int px_n = L.Ho * L.Wo, items = (px_n + 31) / 32 * L.blocks;
        const IrClamp cl = ir_clamp(L.shift, L.lo, L.hi);
        const bool relu = ir_relu(L.shift, L.lo, L.hi);
        for (int it = wave; it < items; it += 8) {
            const int pb = (int)fast_div((unsigned)it, (unsigned)L.blocks, L.magic_blocks), cb = it - pb * L.blocks;
            const int px = 32 * pb + m, pxc = min(px, px_n - 1);
            const bool live = px < px_n;
            const int oy = (int)fast_div((unsigned)pxc, (unsigned)L.Wo, L.magic_wo), ox = pxc - oy * L.Wo;
            const int iy0 = oy * L.stride - L.pad, ix0 = ox * L.stride - L.pad_w;
            // taps s in [s_lo, s_hi) and r in [r_lo, r_hi) fall inside the image; bit r * kw + s of the mask says so (31: no tap)
            const int s_lo = max(0, -ix0), s_hi = min(L.kw, L.W - ix0), r_lo = max(0, -iy0), r_hi = min(L.kh, L.H - iy0);
            const unsigned colmask = s_hi > s_lo ? ((1u << s_hi) - 1u) & ~((1u << s_lo) - 1u) : 0u;
            const unsigned rowsel = r_hi > r_lo ? L.tap_rows & ((1u << (r_hi * L.kw)) - 1u) & ~((1u << (r_lo * L.kw)) - 1u) : 0u;
            const unsigned mask = colmask * rowsel;
            const int base = L.src + (iy0 * L.W + ix0) * L.src_pitch;
            const unsigned char* const tl = sg_lds + L.tab + 8 * hi;      // chunk 2 k + hi of step k: offset from the patch's corner, tap
            v16i acc;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i b4 = *(const v4i*)(sg_lds + L.bias_off + (32 * cb + 8 * q + 4 * hi) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[4 * q + e] = b4[e];
            }
            const unsigned char* wl = sg_lds + L.w_off + cb * L.steps * 1024 + lane * 16;
            // four steps at a time through two sets of registers: the table's entries two batches ahead, the operands one
            v4i w[2][4], xv[2][4];
            int2 t[2][4];
            auto entries = [&](int k0, int2* e) {
#pragma unroll
                for (int u = 0; u < 4; ++u) e[u] = *(const int2*)(tl + 16 * min(k0 + u, L.steps - 1));
            };
            auto operands = [&](int k0, const int2* e, v4i* ww, v4i* xx) {      // steps past the last multiply zeros
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool ok = k0 + u < L.steps && (mask >> e[u].y & 1u);
                    xx[u] = *(const v4i*)(sg_lds + (ok ? base + e[u].x : zero_off));
                    ww[u] = *(const v4i*)(wl + min(k0 + u, L.steps - 1) * 1024);
                }
            };
            auto multiply = [&](const v4i* ww, const v4i* xx) {
#pragma unroll
                for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(ww[u], xx[u], acc, 0, 0, 0);
            };
            entries(0, t[0]);
            entries(4, t[1]);
            operands(0, t[0], w[0], xv[0]);
            for (int k0 = 0; k0 < L.steps; k0 += 8) {
                entries(k0 + 8, t[0]);
                if (k0 + 4 < L.steps) operands(k0 + 4, t[1], w[1], xv[1]);
                __builtin_amdgcn_sched_barrier(0);
                multiply(w[0], xv[0]);
                __builtin_amdgcn_sched_barrier(0);
                entries(k0 + 12, t[1]);
                if (k0 + 8 < L.steps) operands(k0 + 8, t[0], w[0], xv[0]);
                __builtin_amdgcn_sched_barrier(0);
                if (k0 + 4 < L.steps) multiply(w[1], xv[1]);
                __builtin_amdgcn_sched_barrier(0);
            }
            const int ch = 2 * cb + hi, chunks = L.co >> 4;               // this lane's chunk of 16 output channels
            v4i o;
            if (L.res >= 0) {
                const v4i rv = ch < chunks ? *(const v4i*)(sg_lds + L.res + pxc * L.res_pitch + ch * 16) : v4i{0, 0, 0, 0};
                ir_add_residual(acc, rv, L.res_shift, unit);
            }
            o = ir_requant_pack(acc, cl, relu);
            const bool mine = live && ch < chunks;
            if (mine) {
                if (last) *(v4i*)((unsigned char*)y + dst_row * a.out_bytes + px * L.co + ch * 16) = o;
                else *(v4i*)(sg_lds + L.dst + px * L.dst_pitch + ch * 16) = o;
            }
            if (last && head) {
                if (!mine) o = v4i{0, 0, 0, 0};
                v16i t;
#pragma unroll
                for (int i = 0; i < 16; ++i) t[i] = 0;
                t = __builtin_amdgcn_mfma_i32_32x32x32_i8(o, unit, t, 0, 0, 0);
                int sum = 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) sum += t[i];
                const auto both = __builtin_amdgcn_permlane32_swap((unsigned)sum, (unsigned)sum, false, false);      // the other 16 pixels
                sum = (int)(both[0] + both[1]);
                if (hi == 0) __hip_atomic_fetch_add((__attribute__((address_space(3))) int*)l_sums + 32 * cb + m, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        lds_barrier();
    }
    if (!head) return;
    for (int c = tid; c < h.C; c += 512) l_feat[c] = head_feature_i8(h, l_sums[c]);
    lds_barrier();
    head_logits_decide<1, 512>(h, b, l_feat, l_logits, l_exp2, tid, w_first, b_first);
}

hipError_t launch_segment_small(const SegPlan& plan, const SegPlan* dev_plan, const void* x, void* y, int B, const SegRows* rows, const int32_t* ids, const uint16_t* xs, const uint16_t* ys, const HeadArgs* h, hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    if (plan.n < 1 || plan.n > EE_SEG_LAYERS || (rows && B > EE_SEG_ROWS)) return hipErrorInvalidValue;
    static const hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void*>(&segment_small_i8_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (granted != hipSuccess) return granted;
    const SegRows none{};
    const HeadArgs no_head{};
    EE_LAUNCH(segment_small_i8_kernel, dim3(xcd_grid(B)), dim3(512), (size_t)plan.lds_bytes, s, rows ? *rows : none, dev_plan, x, y, B, (int)(rows != nullptr), ids, xs, ys, (int)(h != nullptr), h ? *h : no_head);
    return hipGetLastError();
}

}  // namespace ee
