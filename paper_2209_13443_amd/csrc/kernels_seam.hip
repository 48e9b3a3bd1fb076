// The seam between two bottleneck blocks in one launch, for gfx950 (int8): the 3x3 convolution (C -> C channels, C = 128 or 256), the 1x1 convolution with the residual that ends the
// block (C -> 4 C), and the 1x1 convolution of the next block that reads it (4 C -> C); or the two 1x1 ones alone.
//
// Layer by layer each of them is a launch that starts, fills the chip for a round or two of tiles, and writes a tensor that the next one reads back.  The 1x1 layers are pixel by pixel and
// the 3x3 one needs a frame of one pixel, so a workgroup owns a tile of consecutive pixels and does all three; only the block's output and the next block's first tensor are written, and
// nothing in between is read back.  The weights of the three layers are more than a CU's registers or LDS hold, so they are streamed: each of eight wavefronts owns 32 channels of every layer and
// loads its weights as ready operands (one contiguous KiB per 32 bytes of a reduction, ConvArgs::wo), eight steps ahead, across the layers' boundaries.
//   3x3: the input rows under the tile are one run of the flattened tensor, copied to LDS once (rows padded by 16 bytes); every tap reads it at shifted rows, taps outside the image read
//     zeros (as kernels_taps.hip);
//   1x1 with residual: 256 channels (a piece) at a time, 32 per wavefront, every pixel of the tile; the results replace the residual in LDS;
//   1x1 of the next block: the piece as it stands in LDS is its operand, its accumulators stay in registers over the pieces.  One barrier per piece.
// Four more wavefronts do everything that waits for memory behind the L2: slab, residual and input rows to LDS, finished pieces out of it.  A wavefront's loads and stores come back in order; with
// residuals and stores in the multiplying wavefronts every weight behind one waited for it (14x14, 64 samples: 30.3 us a launch, 24.5 with wavefronts of their own; 23.5 since finished pieces are not waited for).
// Rows in LDS that are not padded are swizzled: chunk c of row r at c ^ f(r), as in the staged kernel.  int32 sums are exact and every tensor is rounded as by its own layer: results are those of the
// separate launches bit for bit.
// What bounds it: one tile per CU at a time, whose weights (275 KB at C = 128, 1.1 MB at C = 256) go through the CU's vector memory path at some 50 bytes/clk, 11 us of 23.5 at C = 256; the
// multiplications are 7.5.  Kernel times of the three launches it replaces and its own, us: 28x28, 40 samples 25.9 / 17.6, 64 (two rounds) 35.5 / 27.4; 14x14, 40 samples 24.0 / 18.5, 64 29.4 / 23.5; and two
// launches fewer, 2.4 us of GPU time and 3 of the host's each.
// int8 only: in bf16 the weights are twice the bytes and the pieces twice the LDS, slower at every size tried (14x14, 256 samples 109 -> 150 us).
#include <algorithm>

#include "ee_internal.hpp"
#include "igemm_device.hpp"
#include "ir_device.hpp"

namespace ee {

// NB: blocks of 32 channels of the narrow tensors (C = 32 NB; 4 or 8); TM: blocks of 32 pixels per wavefront in the layers that write narrow tensors
template <int NB, int TM>
struct SeamShape {
    static constexpr int C = 32 * NB;                                   // channels (bytes) of a narrow pixel
    static constexpr int H = 8 / NB;                                    // groups of wavefronts with pixels of their own in those layers
    static constexpr int PB = TM * H, BM = 32 * PB;                     // blocks of pixels, pixels per tile
    static constexpr int N1 = 4 * C, NP = N1 / 256;                     // channels of the wide tensor, in pieces of 256
    static constexpr int OROW = 256, O_BYTES = BM * OROW;               // a piece in LDS
    static constexpr int NI = O_BYTES / 4096;                           // copies (and stores) of a piece per copying wavefront
    static constexpr int PITCH = C + 16;                                // slab rows
    static constexpr int S0T = C / 32, S0 = 9 * S0T, S1 = S0T, S2 = 8;      // steps: 3x3 layer, one tap of it; per piece: wide layer, next layer
    static constexpr int MID_BYTES = BM * C;
    static int slab_bytes(int W) { return (BM + 2 * W + 2) * PITCH; }
    static int over_bytes(bool front, int W) { return std::max(front ? C + slab_bytes(W) : 0, O_BYTES); }      // zeros and slab, later the last piece
    static int lds_bytes(bool front, int W) { return over_bytes(front, W) + (NP - 1) * O_BYTES + MID_BYTES; }
};

template <int N>
__device__ __forceinline__ void seam_wait_copies() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void seam_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Twelve wavefronts leave 168 registers to each.  The widest form (C = 256, 64 pixels, with the 3x3 layer) keeps four more than that in scratch memory (20 bytes a lane), the others none.
template <int NB, int TM, bool FRONT>
__global__ __launch_bounds__(768, 3) void conv_seam_kernel(SeamArgs a, int over_bytes, unsigned slab_bytes)
{
    request_args<sizeof(SeamArgs)>();
    using Sh = SeamShape<NB, TM>;
    constexpr int CB = Sh::C, PB = Sh::PB, BM = Sh::BM, NP = Sh::NP, NI = Sh::NI, OROW = Sh::OROW, PITCH = Sh::PITCH;
    constexpr int S0 = Sh::S0, S0T = Sh::S0T, S1 = Sh::S1, S2 = Sh::S2, SC = S1 + S2;
    constexpr int R = 8;                                                // weights in flight
    constexpr int XC = CB / 16, XR256 = CB >= 256 ? 1 : 256 / CB, XMASK = XC < 16 ? XC - 1 : 15;      // rows between the 3x3 and the wide layer: chunks, rows per 256 bytes
    constexpr int OC = OROW / 16;
    extern __shared__ __attribute__((aligned(16))) unsigned char seam_lds[];
    // [zeros, slab; later the last piece] [the other pieces] [the tensor between the 3x3 and the wide layer]
    auto buffer = [&](int c) -> int { return c == NP - 1 ? 0 : over_bytes + c * Sh::O_BYTES; };
    const int m_off = over_bytes + (NP - 1) * Sh::O_BYTES;
    const unsigned lds0 = lds_addr(seam_lds);
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int u = xcd_unit(blockIdx.x, (a.M + BM - 1) / BM);
    if (u < 0) return;                                                  // whole workgroup
    const int m0 = u * BM;

    if (wave >= 8) {
        // ==== the copying wavefronts: everything that waits for memory behind the L2.  A wavefront's loads and stores come back in order, so in the others a residual or a store in
        // front of a weight would be waited for with the weight. ==========================================================================================================
        const int io = wave - 8;
        auto residual = [&](int c) {                                    // rows past the end read the last one
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int i = io + 4 * j, p = i * 64 + lane, row = p / OC, chunk = (p % OC) ^ (row & 15);
                dma16(lds0 + (unsigned)(buffer(c) + i * 1024), a.res, (unsigned)min(m0 + row, a.M - 1) * (unsigned)Sh::N1 + c * 256 + chunk * 16);
            }
        };
        if constexpr (FRONT) {
            constexpr int P = PITCH / 16;
            for (unsigned q = tid - 512; q < slab_bytes / 16; q += 256) {
                const unsigned row = q / P, pos = q - row * P;          // divisions by a constant
                const int g = min(max(m0 - a.W - 1 + (int)row, 0), a.M - 1);
                dma16(lds0 + (unsigned)CB + __builtin_amdgcn_readfirstlane(q) * 16u, a.x, (unsigned)g * (unsigned)CB + (pos == P - 1 ? 0u : pos * 16u));
            }
#pragma unroll
            for (int c = 0; c < NP - 1; ++c) residual(c);
            seam_wait_copies<(NP - 1) * NI>();                        // the slab
            seam_barrier();
            seam_wait_copies<0>();
            seam_barrier();                                             // the 3x3 layer is done with the slab
            residual(NP - 1);
        } else {
            constexpr int XI = Sh::MID_BYTES / 1024;                    // the wide layer's input rows as they are in memory
#pragma unroll
            for (int j = 0; j < (XI + 3) / 4; ++j) {
                const int i = (io + 4 * j) % XI, p = i * 64 + lane, row = p / XC, chunk = (p % XC) ^ ((row / XR256) & XMASK);      // fewer instructions than wavefronts: the same bytes once more
                dma16(lds0 + (unsigned)(m_off + i * 1024), a.x, (unsigned)min(m0 + row, a.M - 1) * (unsigned)CB + chunk * 16);
            }
#pragma unroll
            for (int c = 0; c < NP; ++c) residual(c);
            seam_wait_copies<(NP - 1) * NI>();                        // input rows and the first piece's residual
            seam_barrier();
        }
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            // The next piece's residual has to be there behind the barrier.  With the 3x3 layer in front all but the last piece's are since the barrier in the middle; finished pieces on
            // their way out are not waited for except where a residual is (the counter has both, and rows past the end are not stored, so stores cannot be counted off).
            if (FRONT ? c == NP - 2 : c < NP - 1) {
                if (!FRONT && c == 0) seam_wait_copies<(NP - 2) * NI>();
                else seam_wait_copies<0>();
            }
            seam_barrier();                                             // piece c is complete
            const unsigned char* const lo = seam_lds + buffer(c);
#pragma unroll
            for (int j = 0; j < NI; ++j) {                              // out it goes, in the order it has in LDS
                const int i = io + 4 * j, p = i * 64 + lane, row = p / OC, chunk = (p % OC) ^ (row & 15);
                const v4i v = *(const v4i*)(lo + i * 1024 + lane * 16);
                if (m0 + row < a.M) *(v4i*)((unsigned char*)a.y1 + (size_t)(unsigned)(m0 + row) * Sh::N1 + c * 256 + chunk * 16) = v;
            }
        }
        return;
    }

    // ==== the multiplying wavefronts ==================================================================================================================================================
    const int jb = wave % NB, p0 = wave / NB * (32 * TM);               // narrow layers: this wavefront's block of channels, its first pixel
    auto mfma = [](const v4i& w, const v4i& x, const v16i& c) { return __builtin_amdgcn_mfma_i32_32x32x32_i8(w, x, c, 0, 0, 0); };
    // ---- the stream of weights: 3x3 layer (S0 steps), then per piece S1 steps of the wide and S2 of the next layer --------------
    const unsigned char* const w0 = FRONT ? (const unsigned char*)a.w0 + (size_t)jb * a.pitch0 * 1024 + lane * 16 : nullptr;
    const unsigned char* const w1 = (const unsigned char*)a.w1 + (size_t)wave * a.pitch1 * 1024 + lane * 16;
    const unsigned char* const w2 = (const unsigned char*)a.w2 + (size_t)jb * a.pitch2 * 1024 + lane * 16;
    v4i wr[R];
    auto piece_weight = [&](int c, int r) -> const v4i* {               // step r of piece c (r < SC); past the last piece: the last one's
        c = min(c, NP - 1);
        return (const v4i*)(r < S1 ? w1 + (unsigned)(c * 8 * a.pitch1 + r) * 1024u : w2 + (unsigned)(c * S2 + r - S1) * 1024u);
    };
    constexpr int POS = FRONT ? S0 % R : 0;                             // register of the first piece's first step
#pragma unroll
    for (int s = 0; s < R; ++s) {
        const v4i* from = FRONT ? (const v4i*)(w0 + s * 1024) : piece_weight(0, s);
        wr[s] = *from;
    }
    const IrClamp cl0 = ir_clamp(a.shift0, a.lo0, a.hi0), cl1 = ir_clamp(a.shift1, a.lo1, a.hi1), cl2 = ir_clamp(a.shift2, a.lo2, a.hi2);
    const bool relu0 = ir_relu(a.shift0, a.lo0, a.hi0), relu1 = ir_relu(a.shift1, a.lo1, a.hi1), relu2 = ir_relu(a.shift2, a.lo2, a.hi2);
    const v4i unit = ir_unit(m, hi);
    const int xswz = (m / XR256) & XMASK, oswz = m & 15;
    auto start = [&](const void* b, int block) {                        // accumulators start at the bias, the rounding constant part of it
        v16i acc;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v4i b4 = *(const v4i*)((const int*)b + 32 * block + 8 * q + 4 * hi);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * q + e] = b4[e];
        }
        return acc;
    };
    constexpr int BT = 2;                                               // operands in batches through two sets of registers, a batch ahead of its matrix instructions

    if constexpr (FRONT) {
        // ---- the 3x3 layer ---------------------------------------------------------------------------------------------------------
        for (int i = tid; i < CB / 16; i += 512) *(v4i*)(seam_lds + i * 16) = v4i{0, 0, 0, 0};
        // bit t of vmask[i]: tap t of the lane's pixel of block i lies inside the image
        unsigned vmask[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int px = m0 + p0 + 32 * i + m;
            const unsigned pc = (unsigned)min(px, a.M - 1), n = fast_div(pc, (unsigned)(a.H * a.W), a.magic_hw), rem = pc - n * (unsigned)(a.H * a.W);
            const unsigned oy = fast_div(rem, (unsigned)a.W, a.magic_w), ox = rem - oy * a.W;
            const unsigned rows = (oy > 0 ? 7u : 0u) | 7u << 3 | ((int)oy + 1 < a.H ? 7u << 6 : 0u);
            const unsigned cols = (ox > 0 ? 0111u : 0u) | 0222u | ((int)ox + 1 < a.W ? 0444u : 0u);
            vmask[i] = px < a.M ? rows & cols : 0u;
        }
        v16i acc[TM];
        acc[0] = start(a.b0, jb);
        if constexpr (TM == 2) acc[1] = acc[0];
        const int slab = CB + (p0 + m) * PITCH + hi * 16, nothing = hi * 16;
        lds_barrier();                                                  // slab and zeros are there
        int pa[TM];
        auto set_tap = [&](int t, int row) {
#pragma unroll
            for (int i = 0; i < TM; ++i) pa[i] = (vmask[i] >> t) & 1u ? slab + (row + 32 * i) * PITCH : nothing;
        };
        v4i gx[2][BT][TM];
        auto read = [&](int s0, int set) {
#pragma unroll
            for (int s = 0; s < BT; ++s)
#pragma unroll
                for (int i = 0; i < TM; ++i) gx[set][s][i] = *(const v4i*)(seam_lds + pa[i] + (s0 + s) * 32);
        };
        set_tap(0, 0);
        read(0, 0);
        constexpr int TU = S0T == 4 ? 2 : 1;                            // taps per trip: the weights are back in the same registers
        auto taps = [&](int t, auto n_tag) {                            // taps t, t + 1, ...
            static_for<decltype(n_tag)::value>([&](auto k_tag) {
                constexpr int K = decltype(k_tag)::value;
                const int tap = t + K, nt = tap + 1;
                static_for<S0T / BT>([&](auto b_tag) {
                    constexpr int B = decltype(b_tag)::value, SET = B & 1;
                    if constexpr (B + 1 < S0T / BT) read((B + 1) * BT, SET ^ 1);
                    else {
                        set_tap(nt, nt / 3 * a.W + nt % 3);             // behind the last tap every lane reads zeros (no bit 9)
                        read(0, SET ^ 1);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    static_for<BT>([&](auto s_tag) {
                        constexpr int S = B * BT + decltype(s_tag)::value, W = (K * S0T + S) % R;
#pragma unroll
                        for (int i = 0; i < TM; ++i) acc[i] = mfma(wr[W], gx[SET][S - B * BT][i], acc[i]);
                        // the weights R steps ahead: of this layer, or the first ones of the first piece
                        const int ahead = tap * S0T + S + R;
                        const v4i* from = ahead < S0 ? (const v4i*)(w0 + (unsigned)ahead * 1024u) : piece_weight(0, ahead - S0);
                        wr[W] = *from;                                  // one load: the address is chosen
                        __builtin_amdgcn_sched_barrier(0);
                    });
                });
            });
        };
        static_assert(S0T / BT % 2 == 0, "a tap is whole pairs of batches");
        int t = 0;
#pragma clang loop unroll(disable)
        for (; t + TU <= 9; t += TU) taps(t, std::integral_constant<int, TU>{});
        if constexpr (TU == 2) taps(8, std::integral_constant<int, 1>{});
        // results, 16 bytes per lane (int8), between the layers
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            unsigned char* const row = seam_lds + m_off + (p0 + 32 * i + m) * CB;
            *(v4i*)(row + (((2 * jb + hi) ^ xswz) << 4)) = ir_requant_pack(acc[i], cl0, relu0);
        }
    }
    v16i acc2[TM];
    acc2[0] = start(a.b2, jb);
    if constexpr (TM == 2) acc2[1] = acc2[0];
    lds_barrier();                                                      // the wide layer's input and the first residual are there

    // ---- the wide layer and the next one, 256 wide channels at a time -----------------------------------------------------------------
    constexpr int PP = PB > 2 ? 2 : PB;                                 // blocks of pixels at a time
    static_assert(PP == PB || S1 <= R, "the weights of several passes stay in registers");
    // CH: the piece's number modulo the pieces after which the weights are back in the same registers
    auto piece = [&](int c, auto ch_tag) {
        constexpr int BASE = (POS + decltype(ch_tag)::value * SC) % R;
        unsigned char* const lo = seam_lds + buffer(c);
        const v16i bias = start(a.b1, c * 8 + wave);
        static_for<PB / PP>([&](auto pass_tag) {
            constexpr int I0 = decltype(pass_tag)::value * PP;
            constexpr bool LAST = I0 + PP == PB;
            const unsigned char* const xm = seam_lds + m_off + (32 * I0 + m) * CB;
            v16i acc[PP];
#pragma unroll
            for (int i = 0; i < PP; ++i) acc[i] = bias;
            v4i xr[2][BT][PP];
            auto read = [&](int s0, int set) {
#pragma unroll
                for (int s = 0; s < BT; ++s)
#pragma unroll
                    for (int i = 0; i < PP; ++i) xr[set][s][i] = *(const v4i*)(xm + 32 * i * CB + (((2 * (s0 + s) + hi) ^ xswz) << 4));
            };
            read(0, 0);
            static_for<S1 / BT>([&](auto b_tag) {
                constexpr int B = decltype(b_tag)::value;
                if constexpr (B + 1 < S1 / BT) read((B + 1) * BT, (B + 1) & 1);
                __builtin_amdgcn_sched_barrier(0);
                static_for<BT>([&](auto s_tag) {
                    constexpr int S = B * BT + decltype(s_tag)::value, W = (BASE + S) % R;
#pragma unroll
                    for (int i = 0; i < PP; ++i) acc[i] = mfma(wr[W], xr[B & 1][S - B * BT][i], acc[i]);
                    if constexpr (LAST) wr[W] = *piece_weight(S + R >= SC ? c + 1 : c, (S + R) % SC);
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
#pragma unroll
            for (int i = 0; i < PP; ++i) {
                unsigned char* const cell = lo + (32 * (I0 + i) + m) * OROW + (((2 * wave + hi) ^ oswz) << 4);
                ir_add_residual(acc[i], *(const v4i*)cell, a.res_shift, unit);
                *(v4i*)cell = ir_requant_pack<false>(acc[i], cl1, relu1);
            }
        });
        lds_barrier();                                                  // the piece is complete
        // the next layer's share of it
        const unsigned char* const xo = lo + (p0 + m) * OROW;
        v4i yr[2][BT][TM];
        auto read2 = [&](int s0, int set) {
#pragma unroll
            for (int s = 0; s < BT; ++s)
#pragma unroll
                for (int i = 0; i < TM; ++i) yr[set][s][i] = *(const v4i*)(xo + 32 * i * OROW + (((2 * (s0 + s) + hi) ^ oswz) << 4));
        };
        read2(0, 0);
        static_for<S2 / BT>([&](auto b_tag) {
            constexpr int B = decltype(b_tag)::value;
            if constexpr (B + 1 < S2 / BT) read2((B + 1) * BT, (B + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            static_for<BT>([&](auto s_tag) {
                constexpr int S = B * BT + decltype(s_tag)::value, W = (BASE + S1 + S) % R;
#pragma unroll
                for (int i = 0; i < TM; ++i) acc2[i] = mfma(wr[W], yr[B & 1][S - B * BT][i], acc2[i]);
                wr[W] = *piece_weight(S1 + S + R >= SC ? c + 1 : c, (S1 + S + R) % SC);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    static_assert(SC % R == 0 || (2 * SC % R == 0 && NP == 2), "the weights' registers repeat from piece to piece");
    if constexpr (SC % R == 0) {
#pragma clang loop unroll(disable)
        for (int c = 0; c < NP; ++c) piece(c, std::integral_constant<int, 0>{});
    } else {
        piece(0, std::integral_constant<int, 0>{});
        piece(1, std::integral_constant<int, 1>{});
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int px = m0 + p0 + 32 * i + m;
        const v4i out = ir_requant_pack(acc2[i], cl2, relu2);
        if (px < a.M) *(v4i*)((unsigned char*)a.y2 + (size_t)(unsigned)px * CB + 32 * jb + 16 * hi) = out;
    }
}

bool conv_seam_supported(int es, int c, int n1, int n2) { return es == 1 && (c == 128 || c == 256) && n1 == 4 * c && n2 == c; }

template <int NB, int TM, bool FRONT>
static hipError_t launch_seam_shape(const SeamArgs& a, hipStream_t s)
{
    using Sh = SeamShape<NB, TM>;
    const int lds = Sh::lds_bytes(FRONT, a.W);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    static const hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_seam_kernel<NB, TM, FRONT>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (granted != hipSuccess) return granted;
    EE_LAUNCH((conv_seam_kernel<NB, TM, FRONT>), dim3(xcd_grid((a.M + Sh::BM - 1) / Sh::BM)), dim3(768), (size_t)lds, s, a, Sh::over_bytes(FRONT, a.W), (unsigned)Sh::slab_bytes(a.W));
    return hipGetLastError();
}

bool conv_seam_config_ok(int cfg, int c, int W, bool front)
{
    const int tm = cfg & 15;
    if ((cfg & ~(15 | EE_CFG_SEAM_FRONT)) != EE_CFG_SEAM || (tm != 1 && tm != 2) || ((cfg & EE_CFG_SEAM_FRONT) && !front)) return false;
    const bool f = (cfg & EE_CFG_SEAM_FRONT) != 0;
    return (c == 128 ? (tm == 1 ? SeamShape<4, 1>::lds_bytes(f, W) : SeamShape<4, 2>::lds_bytes(f, W)) : tm == 1 ? SeamShape<8, 1>::lds_bytes(f, W) : SeamShape<8, 2>::lds_bytes(f, W)) <= 160 * 1024;
}

// Untuned: the configuration, or 0 for the layers one by one.  A tile's time is its weights' way through one CU, whatever the number of tiles, so what decides is how many rounds of 256
// workgroups (one to a CU) the tiles make.  Measured on the two groups of the ResNet-50-style network (all layers of the segment, one by one / with the seams, us):
//   C = 128 (28x28), tiles of 64 pixels in one round: 1 sample 44.3 / 39.2, 16 75.4 / 64.4; of 128 in one round: 24 97.2 / 83.1, 40 114.9 / 96.7; in two: 48 135.3 / 131.7, 64 151.4 / 139.7, 80 168.0 / 165.7;
//     in three: 128 262.9 / 272.9
//   C = 256 (14x14), tiles of 32 pixels: 16 samples (98 tiles) 98.0 / 100.4, 24 (147) 119.5 / 109.9, 40 (245) 143.3 / 133.1; of 64: 48 (147) 177.7 / 158.7, 64 192.9 / 174.3, 80 (245) 208.0 / 189.0;
//     96 (294) 249.6 / 272.9
// Without the 3x3 layer in front (the first block's is of stride 2) 2 to 3 us a seam at C = 128 in one round, 1 to 2 at C = 256, and nothing in two rounds.
// It is the tiles that count and not the image: four blocks of 3x3 to 56x56 and of 4x60 and 8x64 pixels at 7 to 1024 tiles, one by one / with the seams, are within 0.03 of each other at the same number
// of tiles (C = 128: 7 tiles 1.10, 150 1.36, 250 1.38, 500 1.32, in two rounds of large ones 1.09 to 1.16; C = 256: 150 1.09, 250 1.11, 350 1.12, 500 1.14; without the 3x3 layer 1.04 to 1.16 and 1.05).
// Where the last of the layers has a sibling that it shares a launch with (joint), the seam leaves that one a launch of its own: C = 128, beside a 64- or 512-channel 1x1, 13 tiles 0.98 / 0.89, 75 0.91 / 1.03,
// 147 1.13 / 1.09, 250 1.18 / 1.15, 500 1.16 / 1.19; C = 256, 150 0.94 / 0.94, 250 1.01 / 1.07, 350 (in 175 large ones) 0.98 / 1.03, 500 (250) 1.08 / 1.12; without the 3x3 layer 0.82 to 1.05.
int conv_seam_default(const SeamArgs& a, bool front, bool joint)
{
    const int px = a.C == 128 ? 64 : 32, small = (a.M + px - 1) / px, large = (a.M + 2 * px - 1) / (2 * px), f = front ? EE_CFG_SEAM_FRONT : 0;
    int cfg = 0;
    if (a.C == 128) cfg = small <= 256 ? EE_CFG_SEAM | 1 : large <= (front ? 512 : 256) ? EE_CFG_SEAM | 2 : 0;
    else cfg = small > 128 && small <= 256 ? EE_CFG_SEAM | 1 : small > 256 && large <= 256 ? EE_CFG_SEAM | 2 : 0;
    if (joint && (!front || ((cfg & 15) == 1 ? small : large) < (a.C == 128 ? 128 : 192))) return 0;
    return cfg && conv_seam_config_ok(cfg | f, a.C, a.W, front) ? cfg | f : 0;
}

hipError_t launch_conv_seam(const SeamArgs& a, int cfg, hipStream_t s)
{
    if (a.M <= 0) return hipSuccess;
    const int tm = cfg & 15;
    if (!conv_seam_supported(1, a.C, a.N1, a.N2) || !conv_seam_config_ok(cfg, a.C, a.W, a.w0 != nullptr)) return hipErrorInvalidValue;
#define EE_SEAM(NB_, TM_) if (a.C == 32 * NB_ && tm == TM_) return (cfg & EE_CFG_SEAM_FRONT) ? launch_seam_shape<NB_, TM_, true>(a, s) : launch_seam_shape<NB_, TM_, false>(a, s);
    EE_SEAM(4, 1) EE_SEAM(4, 2) EE_SEAM(8, 1) EE_SEAM(8, 2)
#undef EE_SEAM
    return hipErrorInvalidValue;
}

}  // namespace ee
