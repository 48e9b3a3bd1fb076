// Stride-1 "same" convolutions over pixels of whole 32-byte runs (bf16: 64) on the matrix cores, the activations of a tile resident in LDS and the weights
// streamed from global memory straight into registers: no barrier and no copy between the first matrix instruction and the last.
//
// Output row m and input pixel m coincide (kernels_slab.hip), so the input rows of a tile are one contiguous run, copied to LDS once and read at shifted
// addresses by every tap.  What bounds the staged kernels on these layers is the path that fills LDS (64 bytes/clk and CU; 128 x 128 tiles in 128-byte steps
// need 1.2 times the matrix time for it, smaller tiles more) and a barrier per step.  Here a wavefront owns 32 output channels and multiplies them with every
// pixel of the tile: its weights are one contiguous KiB per 32 bytes of the reduction (ConvArgs::wo), loaded 8 steps ahead into registers and used for 2 to 7
// matrix instructions; the activations are the only LDS traffic, one 1 KiB read per matrix instruction, 128 bytes/clk of about 190; and nothing makes
// wavefronts wait for one another.  Slab rows are padded by 16 bytes, an odd number of chunks, which spreads 16 rows over all banks and makes the position inside a
// pixel a compile-time offset of the read.  Taps outside the image read a row of zeros.
// Four wavefronts (128 channels) per workgroup, two or three of which share a CU; eight (256 channels) where the slab fills it, two where channels are few.  Where the tiles are few (at most
// one or two workgroups per CU) the reduction itself is the chain: 2 or 4 wavefronts share it, a slice of (r, s, c) each, and add up through LDS.  With one
// wavefront per block of channels the sums run in the order of the staged kernel, so bf16 results are the same bits.
// Writes slots and pools for the exit head; does not read slots.
// Layers without padding (int8, pixels of whole 16-byte chunks): all taps exist, so lanes test nothing.  The run of input rows under a tile has what lies between its pixels in it
// where it goes on to another row or image (its length is bounded by the host, the tile copies what it needs), and a step may straddle two taps, a half-wavefront in either.
// 74x74, 3x3, 80 -> 192, best configuration of the other kernels -> this one, us: 16 samples 21.4 -> 17.9, 32 37.2 -> 28.3, 64 68.6 -> 48.6 (1.84 POP/s).
// Measured, best configuration of the other kernels -> this one, 3x3, us:
//   256 samples: bf16 28x28, 128 -> 128 71.1 -> 45.8, 14x14, 256 -> 256 66.9 -> 43.6 (1.36 PFLOP/s, the rate of a large matrix product here), 7x7, 512 -> 512
//     63.1 -> 47.1; int8 35.1 -> 28.7, 31.2 -> 26.2, 33.4 -> 27.2
//   64 samples: bf16 21.0 -> 17.2, 20.1 -> 16.9, 25.2 -> 17.2; int8 11.9 -> 11.6, 11.1 -> 10.6, 13.8 -> 10.4
//   int8, residual, 32 samples: 28x28, 128 -> 128 8.8 -> 7.5, 14x14, 256 -> 256 9.0 -> 7.4, 7x7, 512 -> 512 11.7 -> 7.6
//   int8, 64 samples: 35x35, 96 -> 96 15.7 -> 11.3, 17x17, 1x7, 160 -> 160 8.8 -> 7.7, 192 -> 192 10.0 -> 8.4, 8x8, 3x3, 448 -> 384 12.6 -> 10.0
#include <algorithm>
#include <type_traits>

#include "ee_internal.hpp"
#include "igemm_device.hpp"
#include "igemm_epilogue.hpp"
#include "ir_device.hpp"

namespace ee {

constexpr unsigned taps_part_bytes(int tm, int nw, int kp) { return kp == 1 ? 0 : (unsigned)((tm < kp ? tm : kp) * (kp - 1) * nw * ((tm + kp - 1) / kp) * 4096); }

// ES: element bytes; TM: blocks of 32 pixels of a tile, all of them multiplied by every wavefront; NW: blocks of 32 output channels; KP: wavefronts that
// share the reduction of a block of channels; UNROLL: steps (32 bytes of the reduction) per group, a pixel is a whole number of groups; 0: a layer without padding
template <int ES, int TM, int NW, int KP, int UNROLL>
__global__ __launch_bounds__(64 * NW * KP, 2) void conv_taps_kernel(ConvArgs a, int gm, int gn, unsigned magic_gn, unsigned magic_p, unsigned slab_bytes, unsigned gap_off)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr bool VALID = UNROLL == 0;
    static_assert(!VALID || (ES == 1 && KP == 1), "what is behind the last tap is not cleared, a reduction begins with the first tap");
    constexpr int U = VALID ? 1 : UNROLL;
    constexpr int BM = 32 * TM, BN = 32 * NW, NT = 64 * NW * KP;
    using T = OutTile<ES, BN>;
    constexpr int OROW = T::OROW, CR = T::CR, NO = (BM * CR + NT - 1) / NT;    // output tile: bytes and chunks per row, chunks per lane
    constexpr int WR = U == 1 ? 4 : 8, NG = WR / U;                     // weight operands in flight, groups they make
    constexpr int FD = TM >= 4 || U == 1 ? 1 : U - U / 4, NS = FD == 1 ? 2 : 4;      // activation operands are read FD steps ahead into NS register sets used in turn
    constexpr unsigned PART_BYTES = taps_part_bytes(TM, NW, KP);        // partial sums, over the slab
    constexpr int OWN = (TM + KP - 1) / KP;                             // blocks of pixels a wavefront finishes: wavefront `part` those with i % KP == part
    typedef float v4f __attribute__((ext_vector_type(4)));
    using acc_t = typename std::conditional<ES == 1, v16i, v16f>::type;
    preload(a);
    const int xcd = blockIdx.x & 7, wslot = blockIdx.x >> 3;
    const int mslot = (int)fast_div((unsigned)wslot, (unsigned)gn, magic_gn);
    const int mt = xcd_unit((unsigned)(mslot << 3 | xcd), gm), nt = wslot - mslot * gn;
    if (mt < 0) return;
    const int tid = threadIdx.x, lane = tid & 63, frow = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = mt * BM, n0 = nt * BN;
    const int CiB = a.Ci * ES, pitch = VALID ? CiB | 16 : CiB + 16, P = pitch >> 4;     // an odd number of chunks per slab row spreads 16 rows over all banks
    const unsigned lds0 = lds_addr(lds);
    const bool has_res = a.res != nullptr;

    // ---- weights of the first steps ------------------------------------------------------------------------------
    const int steps = VALID ? (a.kh * a.kw * CiB + 31) >> 5 : a.kh * a.kw * (CiB >> 5), groups = steps / U;
    const int part = wave / NW, wn = wave % NW;                         // this wavefront's share of the reduction, its block of channels
    const bool idle = n0 / 32 + wn >= (a.Co + 31) / 32;                 // its channels lie past the layer's
    const int g0 = KP == 1 ? 0 : groups * part / KP, g1 = idle ? g0 : KP == 1 ? groups : groups * (part + 1) / KP;
    const int co_blocks = (a.Co + 127) / 128 * 4, cb = min(n0 / 32 + wn, co_blocks - 1);
    const unsigned char* const wbase = (const unsigned char*)a.wo + (size_t)cb * (size_t)(a.Kp * ES / 32) * 1024;
    auto weight = [&](int s) { return *(const v4i*)(wbase + (size_t)(unsigned)min(s, steps - 1) * 1024 + lane * 16); };
    v4i wr[WR];
#pragma unroll
    for (int s = 0; s < WR; ++s) wr[s] = weight(g0 * U + s);

    // ---- LDS: zeros for the taps outside the image | slab rows of P chunks | residual tile.  The slab is input rows m0 - halo_lo .. m0 + BM + halo_hi - 1,
    // clamped into the tensor (a clamped row is only ever the source of taps that the validity mask rejects)
    const int halo_lo = a.pad * a.W + a.pad_w;
    // without padding: the input pixel of output pixel m's first tap
    auto first_tap = [&](unsigned m) {
        const unsigned n = fast_div(m, (unsigned)(a.Ho * a.Wo), a.magic_howo), rem = m - n * (unsigned)(a.Ho * a.Wo), oy = fast_div(rem, (unsigned)a.Wo, a.magic_wo);
        return (int)((n * (unsigned)a.H + oy) * (unsigned)a.W + rem - oy * (unsigned)a.Wo);
    };
    const int row0 = VALID ? first_tap((unsigned)m0) : m0 - halo_lo;
    const int row_end = VALID ? first_tap((unsigned)min(m0 + BM, a.M) - 1u) + (a.kh - 1) * a.W + a.kw : a.M;       // without padding the last row the tile needs, in the tensor as well
    const unsigned ro_off = has_res ? max((unsigned)CiB + slab_bytes, PART_BYTES) : PART_BYTES;
    const unsigned slab_chunks = VALID ? min(slab_bytes / 16, (unsigned)((row_end - row0) * P + NT - 1) / NT * NT) : slab_bytes / 16;
    for (unsigned q = tid; q < slab_chunks; q += NT) {
        const unsigned row = fast_div(q, (unsigned)P, magic_p), pos = q - row * (unsigned)P;
        const int g = clamp_i32(row0 + (int)row, 0, row_end - 1);
        dma16(lds0 + (unsigned)CiB + __builtin_amdgcn_readfirstlane(q) * 16u, a.x, __umul24((unsigned)g, (unsigned)CiB) + (pos * 16u >= (unsigned)CiB ? 0u : pos * 16u));
    }
    if (has_res)
#pragma unroll
        for (int j = 0; j < NO; ++j) {
            const int q = tid + NT * j, row = q / CR, chunk = (q % CR) ^ T::oswz(row);
            const int m = min(m0 + row, a.M - 1), ch = n0 + chunk * (16 / ES);
            if (NT * j + 64 * wave < BM * CR)                           // wave-uniform
                dma16(lds0 + ro_off + (unsigned)(NT * j + 64 * wave) * 16u, (const unsigned char*)a.res + ((size_t)(unsigned)m * a.Co + (ch < a.Co ? ch : 0)) * ES);
        }
    if constexpr (!VALID)
        for (int i = tid; i < CiB / 16; i += NT) *(v4i*)(lds + i * 16) = v4i{0, 0, 0, 0};

    // ---- operand addresses: bit t of vmask[i] says whether tap t of the lane's pixel of block i lies inside the image ------------------
    unsigned vmask[TM];                                                 // without padding: the lane's pixel of block i in the slab
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        int m = m0 + 32 * i + frow;
        const bool live = m < a.M;
        m = live ? m : a.M - 1;
        if constexpr (VALID) {
            vmask[i] = (unsigned)CiB + (unsigned)((first_tap((unsigned)m) - row0) * pitch);
            continue;
        }
        const unsigned n = fast_div((unsigned)m, (unsigned)(a.Ho * a.Wo), a.magic_howo), rem = (unsigned)m - n * (unsigned)(a.Ho * a.Wo);
        const unsigned oy = fast_div(rem, (unsigned)a.Wo, a.magic_wo), ox = rem - oy * a.Wo;
        const int iy0 = (int)oy - a.pad, ix0 = (int)ox - a.pad_w;
        const int s_lo = max(0, -ix0), s_hi = min(a.kw, a.W - ix0), r_lo = max(0, -iy0), r_hi = min(a.kh, a.H - iy0);
        const unsigned colmask = s_hi > s_lo ? ((1u << s_hi) - 1u) & ~((1u << s_lo) - 1u) : 0u;
        const unsigned rowsel = r_hi > r_lo ? a.tap_rows & ((1u << (r_hi * a.kw)) - 1u) & ~((1u << (r_lo * a.kw)) - 1u) : 0u;
        vmask[i] = live ? colmask * rowsel : 0u;
    }
    int r_tap = 0, r_ts = 0, r_row = 0, r_cb = 0;                       // the reader's tap, its column, the slab row of the tile's first pixel under it, bytes inside the pixel
    const unsigned lane_off = (unsigned)(frow * pitch + hi * 16);
    unsigned pa[TM];
    // Without padding a step may straddle two taps, the half-wavefronts' 16 bytes are then in different ones: the place of either, its tap, column, byte inside the pixel and offset in the slab, in scalar
    // registers.  Behind the last tap (the weights are zero there) the lanes read their first one.
    struct { int tap, ts, c, off; } place[2];
    const int v_pixel = pitch - CiB, v_row = (a.W - a.kw) * pitch, ntaps = a.kh * a.kw;
    auto set_place = [&]() {
        const int lo = place[0].tap < ntaps ? place[0].off : 0, up = place[1].tap < ntaps ? place[1].off : 0;
        const unsigned off = (unsigned)(hi ? up : lo);
#pragma unroll
        for (int i = 0; i < TM; ++i) pa[i] = vmask[i] + off;
    };
    auto set_tap = [&]() {
        const unsigned at = (unsigned)CiB + (unsigned)(r_row * pitch) + lane_off;
#pragma unroll
        for (int i = 0; i < TM; ++i) pa[i] = (vmask[i] >> r_tap) & 1u ? at + (unsigned)(32 * i * pitch) : (unsigned)(hi * 16);
    };
    auto advance = [&]() {                                              // one group further along (r, s, c); behind the last tap every lane reads zeros
        if constexpr (VALID) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                place[h].c += 32;
                place[h].off += 32;
                if (place[h].c >= CiB) {                                // once: a pixel has 32 bytes or more
                    place[h].c -= CiB;
                    place[h].off += v_pixel;
                    ++place[h].tap;
                    if (++place[h].ts == a.kw) { place[h].ts = 0; place[h].off += v_row; }
                }
            }
            set_place();
            return;
        }
        r_cb += 32 * U;
        if (r_cb == CiB) {
            r_cb = 0;
            ++r_tap;
            ++r_row;
            if (++r_ts == a.kw) { r_ts = 0; r_row += a.W - a.kw; }
            set_tap();
        } else
#pragma unroll
            for (int i = 0; i < TM; ++i) pa[i] += 32 * U;
    };
    if constexpr (VALID) {
        place[0] = {0, 0, 0, 0};
        place[1] = {0, 0, 16, 16};
    } else if (KP > 1 && part > 0) {
        r_tap = g0 * (32 * U) / CiB;
        r_cb = g0 * (32 * U) - r_tap * CiB;
        r_row = r_tap / a.kw * a.W;
        r_ts = r_tap % a.kw;
        r_row += r_ts;
    }
    if constexpr (VALID) set_place();
    else set_tap();
    if (!VALID && KP > 1 && r_cb)
#pragma unroll
        for (int i = 0; i < TM; ++i) pa[i] += (unsigned)r_cb;

    acc_t acc[TM];
    {
        v4i bias[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) bias[q] = ES == 1 && part == 0 ? *(const v4i*)((const int*)a.bias + cb * 32 + 8 * q + 4 * hi) : v4i{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if constexpr (ES == 1) acc[i][e] = bias[e >> 2][e & 3];
                else acc[i][e] = 0.f;
            }
    }
    wait_all_then_barrier<0>();                                         // slab, zeros and residual tile are there

    // ---- main loop -------------------------------------------------------------------------------------------------
    v4i gx[NS][TM];
#pragma unroll
    for (int u = 0; u < FD; ++u)
#pragma unroll
        for (int i = 0; i < TM; ++i) gx[u][i] = *(const v4i*)(lds + pa[i] + u * 32);
    // every matrix instruction is followed by one operand read of a later step, every step by one load of weights WR steps ahead
    auto group = [&](auto h_tag, int g) {
        constexpr int H = decltype(h_tag)::value * U;
        static_for<U>([&](auto u_tag) {
            constexpr int S = decltype(u_tag)::value, R = S + FD;
            if constexpr (R == U) advance();
            static_for<TM>([&](auto i_tag) {
                constexpr int I = decltype(i_tag)::value;
                if constexpr (ES == 1) acc[I] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wr[H + S], gx[(H + S) % NS][I], acc[I], 0, 0, 0);
                else acc[I] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, wr[H + S]), __builtin_bit_cast(v8bf, gx[(H + S) % NS][I]), acc[I], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                gx[(H + R) % NS][I] = *(const v4i*)(lds + pa[I] + (R % U) * 32);
                __builtin_amdgcn_sched_barrier(0);
            });
            wr[H + S] = weight(g * U + S + WR);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    int g = g0;
    for (; g + NG <= g1; g += NG) static_for<NG>([&](auto h_tag) { group(h_tag, g + decltype(h_tag)::value); });
    static_for<NG - 1>([&](auto h_tag) {
        if (g + decltype(h_tag)::value < g1) group(h_tag, g + decltype(h_tag)::value);
    });

    // ---- results: through LDS (rows of OutTile, over the residual if there is one), then whole chunks ----
    v4i bias[4];
    if constexpr (ES == 2)
#pragma unroll
        for (int q = 0; q < 4; ++q) bias[q] = *(const v4i*)((const int*)a.bias + cb * 32 + 8 * q + 4 * hi);
    const IrClamp cl = ir_clamp(a.shift, a.lo, a.hi);
    lds_barrier();                                                      // every wavefront is done with the slab
    if constexpr (KP > 1) {                                             // the other wavefronts' sums of a block, through LDS, to the one that finishes it
        v4i* const l_part = (v4i*)lds;                                  // [part that finishes][other part][block of channels][block of its own][quad][lane]
        auto cell = [&](int to, int from, int i, int q) { return l_part + (((((to * (KP - 1) + (from > to ? from - 1 : from)) * NW + wn) * OWN + i) * 4 + q) << 6) + lane; };
#pragma unroll
        for (int i = 0; i < TM; ++i)
            if (i % KP != part)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    typename std::conditional<ES == 1, v4i, v4f>::type v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[i][4 * q + e];
                    *cell(i % KP, part, i / KP, q) = __builtin_bit_cast(v4i, v);
                }
        lds_barrier();
#pragma unroll
        for (int i = 0; i < TM; ++i)
            if (i % KP == part)
#pragma unroll
                for (int o = 0; o < KP; ++o)
                    if (o != part)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const auto v = __builtin_bit_cast(typename std::conditional<ES == 1, v4i, v4f>::type, *cell(i % KP, o, i / KP, q));
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[i][4 * q + e] += v[e];
                        }
    }
    const bool relu = ir_relu(a.shift, a.lo, a.hi);
    const v4i unit = ES == 1 && has_res ? ir_unit(frow, hi) : v4i{0, 0, 0, 0};
    auto finish = [&](auto res_tag) {
        constexpr bool RES = decltype(res_tag)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (KP > 1 && i % KP != part) continue;
            unsigned char* orow = lds + ro_off + (32 * i + frow) * OROW;
            if constexpr (ES == 1) {
                unsigned char* cell = orow + (((2 * wn + hi) ^ T::oswz(frow)) << 4);
                if constexpr (RES) {
                    const v4i rv = *(const v4i*)cell;
                    ir_add_residual(acc[i], rv, a.res_shift, unit);
                }
                *(v4i*)cell = ir_requant_pack<!RES && KP == 1>(acc[i], cl, relu);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    unsigned char* cell = orow + (((4 * wn + q) ^ T::oswz(frow)) << 4) + 8 * hi;
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
    };
    if (has_res) finish(std::true_type{});
    else finish(std::false_type{});
    int* const gacc = (int*)(lds + gap_off);
    const bool pool = ES == 1 && a.gap_sums != nullptr;
    if (pool)
        for (int i = tid; i < GAP_S * BN; i += NT) gacc[i] = 0;
    lds_barrier();
    if (pool) gap_tile_sums<ES, BM, BN, NT>(a, lds + ro_off, gacc, m0, tid);
    auto out_row = [&](int m) -> long long {                            // zero-copy compaction: sample n of the output goes to slot ys[n] of y
        if (!a.ys || m >= a.M) return m;
        const unsigned howo = (unsigned)(a.Ho * a.Wo), n = fast_div((unsigned)m, howo, a.magic_howo);
        return (long long)a.ys[n] * howo + ((unsigned)m - n * howo);
    };
#pragma unroll
    for (int j = 0; j < NO; ++j) {
        const int q = tid + NT * j, row = q / CR, chunk = (q % CR) ^ T::oswz(row);
        const int m = m0 + row, ch = n0 + chunk * (16 / ES);
        if (q < BM * CR && m < a.M && ch < a.Co) *(v4i*)((unsigned char*)a.y + ((size_t)out_row(m) * a.ldc + a.c_off + ch) * ES) = *(const v4i*)(lds + ro_off + q * 16);
    }
    if (pool) {
        lds_barrier();
        gap_tile_flush<BM, BN, NT>(a, gacc, m0, n0, tid);
    }
}

// no padding at all and an output smaller than the input, so that every tap of every pixel exists (int8)
static constexpr bool taps_valid_tile(int tm, int nw, int kp) { return tm == 4 && nw <= 4 && kp == 1; }       // the tiles that are built for it
static bool taps_valid(const ConvArgs& a, int es) { return es == 1 && a.pad == 0 && a.pad_w == 0 && (a.Ho != a.H || a.Wo != a.W); }

// Stride 1, 2 .. 31 taps, whole 16-byte chunks in the output, a tensor below 2 GiB and 2^24 pixels (the address arithmetic multiplies 24-bit row numbers), and either an output as large as
// the input and a pixel of 64 bytes or more in whole groups of steps (a group never straddles two taps), or no padding and a pixel of 64 bytes or more in whole 16-byte chunks (a step may)
bool conv_taps_supported(const ConvArgs& a, int es)
{
    const int cib = a.Ci * es;
    const bool valid = taps_valid(a, es);
    if (a.xs || a.mode != 0 || !a.wo || a.stride != 1 || (!valid && (a.Ho != a.H || a.Wo != a.W))) return false;
    if (cib % (valid ? 16 : es == 1 ? 32 : 64) != 0 || cib < 64 || cib > 2048 || a.kh * a.kw > 31 || a.kh * a.kw < 2) return false;
    if (a.H + 2 * a.pad - a.kh + 1 != a.Ho || a.W + 2 * a.pad_w - a.kw + 1 != a.Wo) return false;
    if ((a.Co * es) % 16 != 0 || (a.ldc * es) % 16 != 0 || (a.c_off * es) % 16 != 0) return false;
    const long long pixels = (long long)(a.M / (a.Ho * a.Wo)) * a.H * a.W;
    return pixels * cib < (1ll << 31) && pixels < 1 << 24;
}

// the tiles that are built (TAPS_CFGS): blocks of 32 pixels, blocks of 32 channels, wavefronts that share a reduction
#define EE_TAPS_TILES \
    EE_TAPS(2, 4, 1) EE_TAPS(3, 4, 1) EE_TAPS(4, 4, 1) EE_TAPS(5, 4, 1) EE_TAPS(7, 4, 1) EE_TAPS(2, 4, 2) EE_TAPS(4, 4, 2) EE_TAPS(2, 2, 4) EE_TAPS(4, 8, 1) EE_TAPS(7, 8, 1) \
    EE_TAPS(2, 2, 1) EE_TAPS(4, 2, 1) EE_TAPS(2, 2, 2) EE_TAPS(4, 3, 1)

struct TapsLds { unsigned slab, gap_off; size_t bytes; };
static TapsLds taps_lds(const ConvArgs& a, int es, int tm, int nw, int kp)
{
    const int cib = a.Ci * es, nt = 64 * nw * kp;
    long long rows = 32 * tm + (a.kh - 1) * (long long)a.W + (a.kw - 1);
    if (taps_valid(a, es)) {                                            // and what lies between the pixels where the tile goes on to another row or image
        const int last = 32 * tm - 1;
        rows += (last + a.Wo - 1) / a.Wo * (long long)(a.W - a.Wo) + (last + (long long)a.Ho * a.Wo - 1) / ((long long)a.Ho * a.Wo) * (a.H - a.Ho) * a.W;
    }
    const long long chunks = rows * (taps_valid(a, es) ? cib / 16 | 1 : cib / 16 + 1);
    TapsLds l;
    l.slab = (unsigned)((chunks + nt - 1) / nt * nt * 16);
    const size_t parts = taps_part_bytes(tm, nw, kp), tile = (size_t)(32 * tm) * (32 * nw) * es, front = std::max((size_t)cib + l.slab, parts);
    l.bytes = a.res ? front + tile : std::max(front, parts + tile);
    l.gap_off = (unsigned)l.bytes;
    if (a.gap_sums) l.bytes += (size_t)GAP_S * 32 * nw * 4;
    return l;
}

static bool taps_fits(const ConvArgs& a, int es, int tm, int nw, int kp)
{
    return taps_lds(a, es, tm, nw, kp).bytes <= 160 * 1024 && (!a.gap_sums || (es == 1 && (32 * tm - 1) / (a.Ho * a.Wo) + 2 <= GAP_S));
}

bool conv_taps_config_ok(const ConvArgs& a, int cfg, int es)
{
    if (!conv_taps_supported(a, es)) return false;
    const bool any_tile = a.Ci * es % 128 == 0 && !taps_valid(a, es);   // else only tiles of 2 and 4 blocks of pixels exist
#define EE_TAPS(TM_, NW_, KP_) \
    if (cfg == taps_cfg(TM_, NW_, KP_)) return (any_tile || TM_ == 2 || TM_ == 4) && (taps_valid(a, es) ? taps_valid_tile(TM_, NW_, KP_) : NW_ != 3) && taps_fits(a, es, TM_, NW_, KP_);
    EE_TAPS_TILES
#undef EE_TAPS
    return false;
}

// Untuned: the configuration of a layer this kernel is the faster one for, else 0.  Measured over the layers of the ResNet-50, ResNet-18 and Inception-style
// networks at 1-256 samples; blocks are 64 x 64 tiles of the output, us, best configuration of the other kernels / this one.
//   Few pixels, int8: up to 53 blocks (100 for reductions below 2 KiB) the few-pixel kernel is level or the faster one (7x7, 512 -> 512, 4 samples 7.2 / 7.2,
//     17x17, 1x7, 128 -> 128, 8 samples 4.0 / 4.4; from 8 samples 9.0 / 7.3, 14x14, 256 -> 256, 5 samples 6.6 / 5.7).  Up to 256 blocks wavefronts share the
//     reduction of a 64 x 64 tile, four of them a long one (7x7, 512 -> 512, 16 samples 7.5, with two 7.8, with none 10.7), two a shorter one (14x14, 256 -> 256, 16
//     samples 5.8, with four 6.1, with none 7.5); up to 512 two that of a 64 x 128 tile if it is long (14x14, 256 -> 256, 32 samples 7.2, with none 7.7).
//   bf16 does not share: one order of summation.  From 32 blocks on level (18.9 / 18.5 at 32, 11.5 / 10.9 at 64), faster with more.
//   Channels that leave half of a 128-channel tile empty: tiles of 64 channels, two wavefronts sharing up to 512 blocks (17x17, 1x7, 192 -> 192, 32 samples 7.6 / 6.0,
//     with none 7.5), none beyond (64 samples 10.0 / 8.4; 56x56, 64 -> 64, 32 samples 9.7 / 9.0; bf16, 256 samples 72.0 / 65.4), of 128 pixels from 8192 blocks on
//     (56x56, 64 -> 64, 256 samples 44.2 / 38.5, of 64 pixels 41.5).
//   Otherwise the tile with the least work on the busiest CU: its workgroups times (blocks of 32 pixels + 1 for start and end), three tenths more where four wavefronts
//     have a CU to themselves.  Over 27 layers and sizes the choice is the fastest configuration or within 3 % of it but once (7 %).
//   Reductions below 512 bytes were not measured.
//   Without padding (int8): from 1280 blocks on and reductions of 640 bytes tiles of 128 pixels and 128 channels (56x56, 64 -> 64 without padding, 576 bytes, 64 samples 13.4 / 14.5; 30x30, 128 -> 256, 16
//     samples in 784 blocks 8.1 / 9.1, 32 12.2 / 11.6, 64 21.7 / 20.0; 40x40, 5x5, 96 -> 96, 32 samples in 1296 18.3 / 17.1, 64 28.8 / 22.8; 35x70, 3x2, 176 -> 320 72.6 / 58.9), of 96 channels where
//     those leave fewer empty and four workgroups share a CU's LDS (74x74, 80 -> 192, 8 samples 12.7 / 11.1, 64 68.6 / 48.6, with 128 channels 51.1; with three workgroups, 35x70 64 samples, 76.4).
int conv_taps_default(const ConvArgs& a, int es)
{
    const long long blocks = (long long)((a.M + 63) / 64) * ((a.Co + 63) / 64), kbytes = (long long)a.kh * a.kw * a.Ci * es;
    const bool half = (a.Co - 1) % 128 < 64;                            // the last 128-channel tile at most half full
    if (kbytes < 512 || blocks < (es == 2 ? (half ? 200 : 32) : kbytes < 2048 ? 101 : 54) || !conv_taps_supported(a, es)) return 0;
    if (taps_valid(a, es)) {
        if (blocks < 1280 || kbytes < 640) return 0;
        const bool three = (a.Co + 95) / 96 * 96 < (a.Co + 127) / 128 * 128 && taps_lds(a, es, 4, 3, 1).bytes <= 40 * 1024;
        return three && taps_fits(a, es, 4, 3, 1) ? taps_cfg(4, 3, 1) : taps_fits(a, es, 4, 4, 1) ? taps_cfg(4, 4, 1) : 0;
    }
    const bool wide_groups = a.Ci * es % 128 == 0;                      // every tile exists; else 2 and 4 blocks of pixels
    auto fits = [&](int tm, int nw, int kp) { return taps_fits(a, es, tm, nw, kp); };
    if (es == 1 && blocks <= 256 && kbytes >= 3072 && fits(2, 2, 4)) return taps_cfg(2, 2, 4);
    if (es == 1 && blocks <= (half ? 512 : 256) && fits(2, 2, 2)) return taps_cfg(2, 2, 2);
    if (half) {
        if (es == 1 && blocks >= 8192 && fits(4, 2, 1)) return taps_cfg(4, 2, 1);
        return fits(2, 2, 1) ? taps_cfg(2, 2, 1) : 0;
    }
    if (es == 1 && blocks <= 512 && kbytes >= 2048 && fits(2, 4, 2)) return taps_cfg(2, 4, 2);
    int best = 0;
    long long least = 0;
    auto weigh = [&](int tm, int nw) {
        if (!fits(tm, nw, 1) || (!wide_groups && tm != 2 && tm != 4)) return;
        const long long wgs = ((a.M + 32 * tm - 1) / (32 * tm)) * (long long)((a.Co + 32 * nw - 1) / (32 * nw)), rounds = (wgs + 255) / 256;
        const bool alone = nw == 4 && (wgs <= 256 || taps_lds(a, es, tm, nw, 1).bytes > 80 * 1024);
        const long long cost = rounds * (tm + 1) * (nw / 4) * (alone ? 13 : 10);
        if (!best || cost < least) { best = taps_cfg(tm, nw, 1); least = cost; }
    };
    for (const int tm : {2, 3, 4, 5, 7}) weigh(tm, 4);
    if (a.Co % 256 == 0)
        for (const int tm : {4, 7}) weigh(tm, 8);
    return best;
}

template <int ES, int TM, int NW, int KP, int U>
static hipError_t launch_taps_unroll(const ConvArgs& a, hipStream_t s)
{
    constexpr int BM = 32 * TM, BN = 32 * NW;
    const int gm = (a.M + BM - 1) / BM, gn = (a.Co + BN - 1) / BN, p = U == 0 ? a.Ci * ES / 16 | 1 : a.Ci * ES / 16 + 1;
    const TapsLds l = taps_lds(a, ES, TM, NW, KP);
    static const hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_taps_kernel<ES, TM, NW, KP, U>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (granted != hipSuccess) return granted;
    const unsigned magic_gn = (unsigned)(0x100000000ull / (unsigned)gn - (gn == 1)), magic_p = (unsigned)(0x100000000ull / (unsigned)p);
    EE_LAUNCH((conv_taps_kernel<ES, TM, NW, KP, U>), dim3(xcd_grid(gm) * (unsigned)gn), dim3(64 * NW * KP), l.bytes, s, a, gm, gn, magic_gn, magic_p, l.slab, l.gap_off);
    return hipGetLastError();
}

template <int ES, int TM, int NW, int KP>
static hipError_t launch_taps_shape(const ConvArgs& a, hipStream_t s)
{
    const int cib = a.Ci * ES;
    if (taps_valid(a, ES)) {
        if constexpr (ES == 1 && taps_valid_tile(TM, NW, KP)) return launch_taps_unroll<ES, TM, NW, KP, 0>(a, s);
        else return hipErrorInvalidValue;
    }
    if constexpr (NW != 3) {
        if (cib % 128 == 0) return launch_taps_unroll<ES, TM, NW, KP, 4>(a, s);
        if constexpr (TM == 2 || TM == 4) {
            if (cib % 64 == 0) return launch_taps_unroll<ES, TM, NW, KP, 2>(a, s);
            if constexpr (ES == 1) return launch_taps_unroll<ES, TM, NW, KP, 1>(a, s);
        }
    }
    return hipErrorInvalidValue;
}

// hipErrorInvalidValue for a layer it does not cover or a tile whose slab does not fit LDS
template <int ES>
hipError_t launch_conv_taps(const ConvArgs& a, int cfg, hipStream_t s)
{
    if (a.M <= 0) return hipSuccess;
    if (!conv_taps_config_ok(a, cfg, ES)) return hipErrorInvalidValue;
#define EE_TAPS(TM_, NW_, KP_) \
    if (cfg == taps_cfg(TM_, NW_, KP_)) return launch_taps_shape<ES, TM_, NW_, KP_>(a, s);
    EE_TAPS_TILES
#undef EE_TAPS
    return hipErrorInvalidValue;
}

template hipError_t launch_conv_taps<1>(const ConvArgs&, int, hipStream_t);
template hipError_t launch_conv_taps<2>(const ConvArgs&, int, hipStream_t);

}  // namespace ee
