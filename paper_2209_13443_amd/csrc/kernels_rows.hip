// 1x1 convolution with resident weights (int8 and bf16) for gfx950: layers over many pixels whose reduction is short, i.e. whose time is
// the traffic of their tensors.
//
// The staged kernel (igemm_kernel.hpp) starts a workgroup per tile: the first copies' latency, a handful of steps, the epilogue and its stores follow one
// another, and what is in flight per CU is what three or so such workgroups happen to have in flight.  Here a persistent workgroup keeps the
// weights of 128 or 256 output channels in registers (ready operands, 32 channels per wavefront) and walks over tiles of 32 or 64 pixels: while a tile is
// multiplied, the activation rows and the residual tile of the next one are on their way to LDS and the stores of the one before are draining.
// Per tile:
//   wait for the tile's copies (by count: behind them only the stores of the tile before are outstanding), barrier;
//   request the next tile into the other buffer;
//   every wavefront multiplies its 32 channels with all pixels, adds bias and residual, and writes the results over the residual in LDS;
//   barrier; the tile goes out as whole 16-byte chunks, the LDS read in order, the channels' permutation in the global address.
// The number of stores per tile is fixed (rows past the end store out of the buffer's range), which the counting needs.
// Rows of the activations: chunk c of row r at c ^ swz(r) (igemm_kernel.hpp); rows of the output tile: chunk c of row r at c ^ (r mod chunks per row).
// Sums run in the order of the staged kernel, so bf16 results are the same bits.  Takes slot tables, does not pool for the exit head.
#include <algorithm>

#include "ee_internal.hpp"
#include "igemm_device.hpp"
#include "ir_device.hpp"

namespace ee {

struct RowsGrid {
    int tiles;                 // tiles of RB pixels
    int ng;                    // groups of NB * 32 output channels
    int row_slots;             // workgroups per XCD and channel group
    unsigned magic_ng;
    int past_caches;           // the results are stored past the caches (rows_past_caches)
};

// ES: element bytes; KB: bytes per input pixel; NB: blocks of 32 output channels per workgroup; RB: pixels per tile; RW: blocks of 32 pixels per wavefront
template <int ES, int KB, int NB, int RB>
struct RowsShape {
    static constexpr int RW = NB == 8 ? RB / 32 : 1;
    static constexpr int WAVES = NB * RB / (32 * RW);
    static constexpr int NT = 64 * WAVES;
    static constexpr int OROW = NB * 32 * ES, CR = OROW / 16;          // output tile: bytes and chunks per row
    static constexpr int X_BYTES = RB * KB, O_BYTES = RB * OROW;
    static constexpr int S = O_BYTES / 1024 / WAVES;                    // residual copies and stores per wavefront and tile
    static constexpr int LDS = 2 * (X_BYTES + O_BYTES) + 4 * EE_ZC_MAX_B;
    static_assert(S * WAVES * 1024 == O_BYTES && S >= 1, "whole copy instructions per wavefront");
};

template <int ES, int KB, int NB, int RB, bool RES>
__global__ __launch_bounds__((RowsShape<ES, KB, NB, RB>::NT), 2) void conv_rows_kernel(ConvArgs a, RowsGrid g)
{
    request_args<sizeof(ConvArgs) + sizeof(RowsGrid)>();
    using Sh = RowsShape<ES, KB, NB, RB>;
    constexpr int RW = Sh::RW, WAVES = Sh::WAVES, NT = Sh::NT, OROW = Sh::OROW, CR = Sh::CR, S = Sh::S;
    constexpr int NS = KB / 32;                                         // matrix instructions of a reduction
    constexpr int XC = KB / 16, XROWS = 1024 / KB, XT = Sh::X_BYTES / 1024;   // chunks per activation row, rows per copy instruction, instructions per tile
    constexpr int R256 = KB >= 256 ? 1 : 256 / KB, XMASK = XC < 16 ? XC - 1 : 15;
    extern __shared__ __attribute__((aligned(16))) unsigned char rows_lds[];
    unsigned char* const l_x = rows_lds;                                // two buffers each
    unsigned char* const l_o = rows_lds + 2 * Sh::X_BYTES;
    unsigned short* const l_xs = (unsigned short*)(l_o + 2 * Sh::O_BYTES);
    unsigned short* const l_ys = l_xs + EE_ZC_MAX_B;
    const unsigned lds0 = lds_addr(rows_lds);
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xcd = (int)(blockIdx.x & 7), slot = (int)(blockIdx.x >> 3);
    const int rslot = __builtin_amdgcn_readfirstlane((int)fast_div((unsigned)slot, (unsigned)g.ng, g.magic_ng)), grp = slot - rslot * g.ng;
    const int u_end = xcd_first(xcd + 1, g.tiles), u0 = xcd_first(xcd, g.tiles) + rslot;
    if (rslot >= g.row_slots || u0 >= u_end) return;                    // whole workgroup
    const int n0 = grp * NB * 32;
    const int cb = wave % NB, rb0 = wave / NB * RW;                     // this wavefront's block of channels, its first block of pixels
    const unsigned howo = (unsigned)(a.Ho * a.Wo);
    const bool plain = a.stride == 1 && !a.xs;                          // activation row m is pixel m of x
    if (a.xs || a.ys)
        for (int i = tid; i < EE_ZC_MAX_B; i += NT) {                   // one entry per sample, at most EE_ZC_MAX_B with a table: checked by the launcher
            const bool live = (unsigned)i * howo < (unsigned)a.M;
            l_xs[i] = a.xs && live ? a.xs[i] : 0;
            l_ys[i] = a.ys && live ? a.ys[i] : 0;
        }
    v4i w[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) w[s] = *(const v4i*)((const unsigned char*)a.wo + ((size_t)((n0 / 32 + cb) * (a.Kp * ES / 32) + s) * 64 + lane) * 16);
    v4i bias[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) bias[q] = *(const v4i*)((const int*)a.bias + n0 + 32 * cb + 8 * q + 4 * hi);
    auto request = [&](int u, int buf) {                                // asynchronous; rows past the end read the last one
        const int m0 = u * RB;
        const unsigned xbase = lds0 + (unsigned)(buf * Sh::X_BYTES), obase = lds0 + (unsigned)(2 * Sh::X_BYTES + buf * Sh::O_BYTES);
#pragma unroll
        for (int j = 0; j < (XT + WAVES - 1) / WAVES; ++j) {
            const int i = (wave + WAVES * j) % XT;                      // fewer instructions than wavefronts: the same bytes once more
            const int row = i * XROWS + lane / XC, chunk = (lane % XC) ^ ((row / R256) & XMASK);
            const unsigned r = (unsigned)min(m0 + row, a.M - 1);
            unsigned px = r;
            if (!plain) {
                const unsigned n = fast_div(r, howo, a.magic_howo), rem = r - n * howo, oy = fast_div(rem, (unsigned)a.Wo, a.magic_wo), ox = rem - oy * a.Wo;
                px = ((a.xs ? (unsigned)l_xs[n] : n) * a.H + oy * a.stride) * a.W + ox * a.stride;
            }
            dma16(xbase + (unsigned)(i * 1024), a.x, px * KB + chunk * 16);
        }
        if constexpr (RES) {
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const int i = wave * S + j, row = i * (1024 / OROW) + lane / CR, chunk = (lane % CR) ^ (row & (CR - 1));
                const unsigned r = (unsigned)min(m0 + row, a.M - 1);
                dma16(obase + (unsigned)(i * 1024), a.res, (r * (unsigned)a.Co + n0) * ES + chunk * 16);
            }
        }
    };
    // the first tile is on its way with the weights: int8, 64 samples, 9.4 -> 8.9, 11.0 -> 10.7 and 13.9 -> 13.6 us a layer
    __builtin_amdgcn_sched_barrier(0);
    if (a.xs || a.ys) lds_barrier();                                    // the slot tables are in LDS
    request(u0, 0);
    // every weight has arrived before the loop, so that nothing inside it waits for a weight by count
#pragma unroll
    for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(w[s]));
#pragma unroll
    for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(bias[q]));
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(a.y, (short)0, 0x7fffffff, 0x00020000);
    const IrClamp cl = ir_clamp(a.shift, a.lo, a.hi);
    const bool relu = ir_relu(a.shift, a.lo, a.hi);
    const v4i unit = ES == 1 && RES ? ir_unit(m, hi) : v4i{0, 0, 0, 0};
    const int swz = (m / R256) & XMASK;
    using acc_t = typename std::conditional<ES == 1, v16i, v16f>::type;

    int buf = 0;
    for (int u = u0; u < u_end; u += g.row_slots, buf ^= 1) {
        if (u == u0) wait_all_then_barrier<0>();
        else wait_all_then_barrier<S>();                                // behind this tile's copies: the stores of the tile before
        if (u + g.row_slots < u_end) request(u + g.row_slots, buf ^ 1);
        const unsigned char* xt = l_x + buf * Sh::X_BYTES + (rb0 * 32 + m) * KB;
        unsigned char* ot = l_o + buf * Sh::O_BYTES + (rb0 * 32 + m) * OROW;
        acc_t acc[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if constexpr (ES == 1) acc[i][e] = bias[e >> 2][e & 3];
                else acc[i][e] = 0.f;
            }
        // operands in batches through two sets of registers, a batch ahead of its matrix instructions
        constexpr int BT = NS < 4 ? NS : 4 / RW < 2 ? 2 : 4 / RW;
        v4i xr[2][BT][RW];
        auto read = [&](int s0, int set) {
#pragma unroll
            for (int s = 0; s < BT; ++s)
#pragma unroll
                for (int i = 0; i < RW; ++i) xr[set][s][i] = *(const v4i*)(xt + i * 32 * KB + (((2 * (s0 + s) + hi) ^ swz) << 4));
        };
        read(0, 0);
        static_for<NS / BT>([&](auto b_tag) {
            constexpr int B = decltype(b_tag)::value;
            if constexpr (B + 1 < NS / BT) read((B + 1) * BT, (B + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < BT; ++s)
#pragma unroll
                for (int i = 0; i < RW; ++i) {
                    if constexpr (ES == 1) acc[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[B * BT + s], xr[B & 1][s][i], acc[i], 0, 0, 0);
                    else acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, w[B * BT + s]), __builtin_bit_cast(v8bf, xr[B & 1][s][i]), acc[i], 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        });
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            // rows rb0 * 32 + 32 i + m: the same position modulo the chunks of a row for every i
            unsigned char* orow = ot + i * 32 * OROW;
            if constexpr (ES == 1) {
                unsigned char* cell = orow + (((2 * cb + hi) ^ (m & (CR - 1))) << 4);
                if constexpr (RES) {
                    const v4i rv = *(const v4i*)cell;
                    ir_add_residual(acc[i], rv, a.res_shift, unit);
                }
                *(v4i*)cell = ir_requant_pack<!RES>(acc[i], cl, relu);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    unsigned char* cell = orow + (((4 * cb + q) ^ (m & (CR - 1))) << 4) + 8 * hi;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[i][4 * q + e] + __int_as_float(bias[q][e]);
                    if constexpr (RES) {
                        const uint2 r = *(const uint2*)cell;
                        v[0] += __uint_as_float(r.x << 16); v[1] += __uint_as_float(r.x & 0xFFFF0000u);
                        v[2] += __uint_as_float(r.y << 16); v[3] += __uint_as_float(r.y & 0xFFFF0000u);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = clamp_f32(v[e], a.f_lo, a.f_hi);
                    *(uint2*)cell = uint2{pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
                }
            }
        }
        lds_barrier();                                                  // the output tile is complete
        auto store = [&](auto policy) {
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const int i = wave * S + j, row = i * (1024 / OROW) + lane / CR, chunk = (lane % CR) ^ (row & (CR - 1));
                const unsigned r = (unsigned)(u * RB + row);
                unsigned orow = r;
                if (a.ys) {
                    const unsigned rc = min(r, (unsigned)a.M - 1), n = fast_div(rc, howo, a.magic_howo);
                    orow = (unsigned)l_ys[n] * howo + (rc - n * howo);
                }
                const v4i v = *(const v4i*)(l_o + buf * Sh::O_BYTES + i * 1024 + lane * 16);
                const unsigned off = (orow * (unsigned)a.ldc + (unsigned)(a.c_off + n0)) * ES + chunk * 16;
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, v), rsrc, r < (unsigned)a.M ? (int)off : (int)0x80000000u, 0, decltype(policy)::value);
            }
        };
        if (ES == 2 && g.past_caches) store(std::integral_constant<int, 2>{});
        else store(std::integral_constant<int, 0>{});
    }
}

// 1x1 layers over pixels of 128 .. 1024 bytes to a multiple of 128 channels, whole 16-byte chunks throughout, tensors below 2 GiB
bool conv_rows_supported(const ConvArgs& a, int es)
{
    const int kb = a.Ci * es;
    if (a.mode != 0 || a.gap_sums || a.kh != 1 || a.kw != 1 || a.pad != 0 || a.pad_w != 0 || !a.wo) return false;
    if ((kb != 128 && kb != 256 && kb != 512 && kb != 1024) || a.Co % 128 != 0 || (a.Co > 128 && a.Co % 256 != 0)) return false;
    if ((a.ldc * es) % 16 != 0 || (a.c_off * es) % 16 != 0 || a.Co > 4096) return false;
    if ((long long)(a.M / (a.Ho * a.Wo)) * a.H * a.W * kb >= (1ll << 31)) return false;
    return (long long)a.M * a.ldc * es < (1ll << 31) && (long long)a.M * a.Co * es < (1ll << 31);
}

bool conv_rows_config_ok(const ConvArgs& a, int cfg, int es) { return cfg_is_rows(cfg) && conv_rows_supported(a, es) && !(cfg == EE_CFG_ROWS64 && a.Ci * es == 1024); }

// Untuned: the configuration of a layer this kernel is the faster one for, else 0.  Measured against the best configuration of the staged kernel on the 1x1
// layers of the ResNet-50-style network; what decides is how many tiles a resident workgroup walks over, i.e. the size of the output (in 64 x 64 blocks):
//   int8: from 2560 on it wins (28x28, 128 -> 512 + residual, 64 samples: 11.1 us against 14.7; 56x56, 256 -> 512 / 2 12.1 / 15.8; 14x14, 256 -> 1024 + residual
//     8.5 / 10.0; 256 samples 34.8 / 43.2, 30.5 / 45.2, 21.2 / 34.1), from 1536 to 1814 it is level on some layers and loses 10 to 20 % on others;
//   bf16 (twice the bytes): from 1536 on (28x28, 128 -> 512 + residual, 64 samples 16.9 / 25.5; 7x7, 512 -> 2048 + residual 13.4 / 15.0; 256 samples 86.5 / 117.7,
//     14x14, 256 -> 1024 + residual 35.2 / 62.2, 56x56, 256 -> 512 / 2 62.9 / 106.4), at 906 to 928 it loses 7 to 12 %.
// Tiles of 64 pixels for large bf16 outputs (56x56, 64 -> 256, 256 samples 91.6 us, 105.0 with 32; 256 -> 512 / 2 62.9 / 73.8), else of 32: they spread better
// over the workgroups (int8 56x56, 256 -> 512 / 2, 256 samples 30.5 us, 37.8 with 64; bf16 at 64 samples 3 to 9 %).
int conv_rows_default(const ConvArgs& a, int es)
{
    const long long blocks = (long long)((a.M + 63) / 64) * ((a.Co + 63) / 64);
    if (blocks < (es == 1 ? 2560 : 1536) || !conv_rows_supported(a, es)) return 0;
    return es == 2 && blocks >= 8192 && a.Ci * es <= 512 ? EE_CFG_ROWS64 : EE_CFG_ROWS32;
}

// bf16 results of half of the L2s (32 MB) and more go past the caches: they displace the weights and narrow tensors that the next layers need.  ResNet-50, stream of 8,000 requests in 256 slots on two lanes, ms, six tunings:
// none 70.3-70.7, all, from 32, 64 and 96 MB on 69.4-70.0, from 128 MB on 70.0-70.4.  Smaller results the next layer finds in the caches; all segments, us, none / all / from 16 MB on: 4 samples 295 / 298 / 295, 8 348 / 351 / 348,
// 12 409 / 416 / 409, 16 451 / 461 / 451, 24 614 / 601 / 599, 32 701 / 696 / 704, 40 751 / 746 / 756, 50 882 / 890 / 893, 64 1,030 / 1,018 / 1,018, 100 1,417 / 1,452 / 1,458, 160 2,034 / 2,034 / 2,037, 200 2,551 / 2,601 / 2,603,
// 256 3,110 / 3,138 / 3,144: between 24 and 256 samples alone no limit is the better one throughout, in streams all of them are alike.  int8, half of the bytes, is as fast either way.
static bool rows_past_caches(const ConvArgs& a, int es) { return es == 2 && (long long)a.M * a.Co * es >= 16 << 20; }

template <int ES, int KB, int NB, int RB, bool RES>
static hipError_t launch_rows_shape(const ConvArgs& a, hipStream_t s)
{
    using Sh = RowsShape<ES, KB, NB, RB>;
    static const hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_rows_kernel<ES, KB, NB, RB, RES>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (granted != hipSuccess) return granted;
    static const int per_cu = [] {                                      // workgroups that share a CU: the persistent grid is exactly what is resident
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, conv_rows_kernel<ES, KB, NB, RB, RES>, Sh::NT, Sh::LDS) != hipSuccess || n < 1) n = 1;
        return n;
    }();
    RowsGrid g;
    g.tiles = (a.M + RB - 1) / RB;
    g.ng = a.Co / (NB * 32);
    g.magic_ng = (unsigned)(0x100000000ull / (unsigned)g.ng - (g.ng == 1));
    const int per_xcd = (g.tiles + 7) / 8;
    g.row_slots = std::max(1, 32 * per_cu / g.ng);
    if (g.row_slots > per_xcd) g.row_slots = per_xcd;
    g.past_caches = rows_past_caches(a, ES);
    EE_LAUNCH((conv_rows_kernel<ES, KB, NB, RB, RES>), dim3((unsigned)(8 * g.row_slots * g.ng)), dim3(Sh::NT), (size_t)Sh::LDS, s, a, g);
    return hipGetLastError();
}

// hipErrorInvalidValue for a layer or configuration it does not cover
template <int ES>
hipError_t launch_conv_rows(const ConvArgs& a, int cfg, hipStream_t s)
{
    if (a.M <= 0) return hipSuccess;
    const int rb = cfg == EE_CFG_ROWS64 ? 2 : 1, kb = a.Ci * ES;
    if (!conv_rows_config_ok(a, cfg, ES)) return hipErrorInvalidValue;
#define EE_ROWS(KB_, NB_, RB_) \
    if (kb == KB_ && (a.Co == 128) == (NB_ == 4) && rb == RB_ / 32) return a.res ? launch_rows_shape<ES, KB_, NB_, RB_, true>(a, s) : launch_rows_shape<ES, KB_, NB_, RB_, false>(a, s);
    EE_ROWS(128, 8, 32) EE_ROWS(128, 8, 64) EE_ROWS(128, 4, 32) EE_ROWS(128, 4, 64)
    EE_ROWS(256, 8, 32) EE_ROWS(256, 8, 64) EE_ROWS(256, 4, 32) EE_ROWS(256, 4, 64)
    EE_ROWS(512, 8, 32) EE_ROWS(512, 8, 64) EE_ROWS(512, 4, 32) EE_ROWS(512, 4, 64)
    EE_ROWS(1024, 8, 32) EE_ROWS(1024, 4, 32)
#undef EE_ROWS
    return hipErrorInvalidValue;
}

template hipError_t launch_conv_rows<1>(const ConvArgs&, int, hipStream_t);
template hipError_t launch_conv_rows<2>(const ConvArgs&, int, hipStream_t);

}  // namespace ee
