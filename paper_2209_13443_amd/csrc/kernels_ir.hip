// Inverted-residual block (int8) in one launch, for gfx950: 1x1 expansion -> 3x3 depthwise -> 1x1 projection
// (+ residual), the block of MobileNetV2-style networks.  Run layer by layer, the expanded tensor (6 x the block's
// input) is written by the expansion, read and written by the depthwise layer and read by the projection; here it
// only ever exists in LDS, one group of 32 expanded channels at a time, and all three layers run on the matrix cores.
//
// A workgroup (4 wavefronts) owns a tile of output pixels of one image: blocks of 32 pixels (NBH rows x NBW columns,
// NBH * NBW <= 32), at most MAXB blocks per wavefront.
//   * The block's input pixels under the tile (with the one-pixel frame of the 3x3 window) are staged once in LDS,
//     8 or 16 bytes per lane and load, a pixel's channels followed by padding up to the reduction length (a multiple of 32)
//     plus 16 bytes (an odd number of 16-byte chunks per pixel spreads consecutive pixels over the banks).  Bytes behind
//     a pixel's channels are never written: the expansion weights are zero there.
//   * For every group g of 32 expanded channels:
//       expansion   E_g[pixel][32] = requant(W_e[g] . x[pixel] + b_e[g]) for the staged pixels inside the image
//                   (v_mfma_i32_32x32x32_i8, rows = channels, columns = 32 staged pixels, shared out over the
//                   wavefronts), written to one of two LDS buffers laid out like the tile (32 bytes per pixel, 16 bytes
//                   of padding per row); pixels outside the image are zero there from the start and stay zero: the
//                   depthwise layer pads its input, the *expanded* tensor, with zeros;
//       depthwise   per block of 32 output pixels one dense matrix instruction for the first tap, whose A operand is the diagonal matrix diag(w_d[c][tap]) of the group's channels and
//                   whose B operand is the 32 channels of the tap's input pixels (one 16-byte LDS read per lane), and four sparse ones (v_smfmac_i32_32x32x64_i8, as fast as a dense
//                   one of half the reduction) for two taps each: two diagonals side by side keep one of every four reduction bytes, and a 4:2 sparse operand has room for two.  A
//                   multiply-add per output and tap costs a sixty-fourth of the instruction, and it is still several times cheaper than byte transposes and dot products on the
//                   vector ALU.  With nine dense ones, and the biases read from LDS in front of every block, the launches took 4-9 % longer (7x7, 160 -> 960 -> 160, 64 samples 13.4 us,
//                   now 12.5; 14x14, 64 -> 384 -> 64 8.9, now 8.4);
//       projection  the requantised depthwise outputs of a block are, after one exchange between the two halves of
//                   the wavefront (v_permlane32_swap), exactly the B operand (32 reduction channels x 32 pixels) of
//                   the projection, whose accumulators (NCO blocks of 32 output channels per pixel block) stay in
//                   registers over all groups.
//     The expansion of group g + 1 runs behind the depthwise + projection of group g without a barrier in between
//     (other buffer); there is one workgroup barrier per group.
//   * Epilogue: projection bias, residual, requantisation, 16-byte stores; for the block that ends a segment also the exit head's pooling (a.gap_sums): a
//     tile lies in one image, so its channel sums go out with an atomic addition per channel (int32, exact in any order).  Without it the block ran as three launches,
//     the last with the pooling (serving MobileNetV2, 64 slots, 4,096 requests: 14.65 -> 14.02 ms).
// Few tiles (ir_block_plan) run the second form, GP: tiles of one or two blocks whose four or eight wavefronts share the *channel groups* instead of the pixels.  Each wavefront
// expands, filters and projects every pixel of the tile for the groups g = wavefront, wavefront + 4 (or 8), ... through a buffer
// of its own, with no barrier inside the loop; the partial projection sums are added in LDS (integer adds,
// exact in any order) and the epilogue is shared out by (pixel block, output block).
// What bounds it: blocks on large images issue vector instructions for half of their time (112 x 112 -> 56 x 56, 16 -> 96 -> 24 channels, 64 images: 7.4 M, 12.0 of 23.5 us; 56 x 56, 24 -> 144 -> 24: 5.2 M, 8.5
// of 18.8, launches back to back) and matrix instructions for 2.7 and 3.7 us; a third of a workgroup's life is
// the way to its first group (6,000 of 17,000 cycles on the first of them: arguments 1,900, pixels there 3,500, barrier 6,000).  Those on small images wait for their chain of loads, matrix instructions and barriers; 7 x 7, 160 -> 960 -> 160 for the 450 KB of weights that a workgroup reads through its CU's path, 3.9 of 11.7 us.
// (Loading the first group's weights in front of the input, and the next group's ahead in GP, was 0-8 % slower everywhere: weights queue in front of the input.)
// Every accumulation is int32 and exact, rounding points are those of the three separate layers: results are equal
// bit for bit.
#include "ee_internal.hpp"
#include "ir_device.hpp"

namespace ee {

struct IrTile {
    int nbw, nbh;          // a block of 32 output pixels: nbh rows x nbw columns
    int pbw, pbh;          // blocks per workgroup tile along x and y
    int tiles_x, tiles_y;
    int iw, ih;            // staged pixels under a tile
    int cpp, wide;         // chunks per input pixel, of 16 bytes (wide) or 8
    unsigned magic_cpp, magic_iw;   // floor(2^32 / d) + 1: n / d for n < 2^16
    unsigned magic_tx, magic_ty;    // the same for tiles_x, tiles_y (n * d < 2^32: checked by ir_block_plan)
    int magic_nbw, magic_pbw;       // floor(2^16 / d) + 1: n / d for n < 2^8
    int xp;                // bytes per staged input pixel
    int x_bytes, e_bytes;  // LDS: staged input, one buffer of expanded pixels
    int total;             // workgroups with work
    int gp;                // 4 or 8: that many wavefronts share the channel groups (small images), 0: four share the pixels
};

constexpr int IR_BATCH = 8, IR_BATCHES = 2;   // loads per lane that stage a tile, in batches: ih * iw * cpp <= 4096
// blocks of 32 staged pixels per wavefront in the expansion: ih * iw <= 384, or, where the wavefronts share the channel groups, 96 (stride 2: 160, a block of 4 x 8 output pixels)
constexpr int ir_maxcb(int gp, int stride) { return gp && stride == 2 ? 5 : 3; }
constexpr int IR_SHARED_LDS = 96 * 1024;      // LDS bytes where the wavefronts share the channel groups (their registers leave one workgroup to a CU)
constexpr int IR_FILL = 4;                    // 16-byte loads per lane that fill a buffer without expansion: ih * iw * 2 <= 1024
constexpr int IR_MAXK = 5;                    // reduction steps of 32 input channels: c_in <= 160 (template parameter MAXK: 1, 2 or 5)

// The block's input image n as a buffer, of which loads out of range (before the image too: offsets are unsigned) give zeros.  Where a load's address was chosen by a condition instead, the compiler made
// two loads of it, one for the lanes on either side, and waited in front of each for the one before: a tile's chunks arrived one round trip to memory after the other.  64 samples, us: 112x112 stride 2,
// 16 -> 96 -> 24 27.8 -> 25.9, 56x56 stride 2, 24 -> 144 -> 32 13.8 -> 12.6, 28x28, 32 -> 192 -> 32 12.3 -> 11.2; all segments 262 -> 253, of 20 samples 185 -> 178, of one 129 -> 126.
__device__ __forceinline__ auto image(const IrArgs& a, int n)
{
    const int bytes = a.H * a.W * a.Cin;
    return __builtin_amdgcn_make_buffer_rsrc((char*)a.x + (size_t)n * bytes, (short)0, bytes, 0x00020000);
}
template <typename V>
__device__ __forceinline__ V image_load(__amdgpu_buffer_rsrc_t x, int at)
{
    if constexpr (sizeof(V) == 16) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(x, at, 0, 0));
    else return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(x, at, 0, 0));
}

// GP = 0: four wavefronts share the pixels; GP = 4 or 8: that many wavefronts share the channel groups.
// MAXK = 0: a block without expansion (depthwise -> projection): the buffers of "expanded" pixels are filled with the
// block's input itself, 32 channels at a time.
// POOL: the exit head's pooling in the epilogue (a kernel of its own: with a branch the others' launches on one image took 0.15 us longer each)
// Without expansion and to one output block four workgroups share a CU like with one: 112x112, 32 -> 16, us, 146 registers / 128: 4 samples 4.4 / 4.5, 16 7.2 / 6.7, 32 10.9 / 10.3, 64 18.3 / 17.0, 128
// 32.6 / 29.3 (with two or three registers in scratch memory 4.7, 7.1, 10.7, 17.3 and 29.8).
// Registers: <1, 1, 2, 1, 0, true>, held to 128, keeps two more in scratch memory (12 bytes a lane); no other form spills.
template <int STRIDE, int NCO, int MAXB, int MAXK, int GP, bool POOL>
__global__ __launch_bounds__(GP ? 64 * GP : 256, (NCO == 1 && !GP && MAXK <= 1) ? (MAXK == 0 && POOL ? 3 : 4) : 2) void ir_block_i8_kernel(IrArgs a, IrTile t)
{
    request_args<sizeof(IrArgs) + sizeof(IrTile)>();
    constexpr int NW = GP ? GP : 4, NT = 64 * NW;                      // wavefronts and lanes per workgroup
    constexpr bool EXP = MAXK > 0;
    constexpr int MAXCB = ir_maxcb(GP, STRIDE);
    extern __shared__ __attribute__((aligned(16))) unsigned char ir_lds[];
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int u = xcd_unit(blockIdx.x, t.total);
    if (u < 0) return;                                          // whole workgroup: no barrier is skipped by a part of it
    // divisions by host-made factors: a division by a value the compiler does not know is some 25 instructions, and the
    // blocks on large images are bound by instruction issue
    const int uq = t.tiles_x == 1 ? u : (int)__umulhi((unsigned)u, t.magic_tx), n = t.tiles_y == 1 ? uq : (int)__umulhi((unsigned)uq, t.magic_ty);
    const int tx_i = u - uq * t.tiles_x, ty_i = uq - n * t.tiles_y;
    const int ox0 = tx_i * t.pbw * t.nbw, oy0 = ty_i * t.pbh * t.nbh;
    const int ix0 = ox0 * STRIDE - a.pad, iy0 = oy0 * STRIDE - a.pad;
    unsigned char* const l_be = ir_lds;                                 // expansion bias, depthwise bias (int32 per expanded channel)
    unsigned char* const l_bd = ir_lds + 4 * a.Ce32;
    unsigned char* const l_x = ir_lds + 8 * a.Ce32;
    unsigned char* const l_e = l_x + t.x_bytes;
    const int e_row = t.iw * 32 + 16;                                   // bytes per row of expanded pixels
    const int kx32 = a.Kx >> 5;
    const IrClamp cl_e = ir_clamp(a.sh_e, a.lo_e, a.hi_e), cl_d = ir_clamp(a.sh_d, a.lo_d, a.hi_d), cl_p = ir_clamp(a.sh_p, a.lo_p, a.hi_p);

    // ---- the pixels inside the image under the tile --------------------------------------------------------------------------
    const int y0 = max(0, -iy0), y1 = min(t.ih, a.H - iy0), x0 = max(0, -ix0), x1 = min(t.iw, a.W - ix0);
    const int sw = max(x1 - x0, 1), npix = max(x1 - x0, 0) * max(y1 - y0, 0);
    const bool frame = npix < t.ih * t.iw;                              // a part of the tile's window is outside the image
    const int ngroups = a.Ce32 >> 5;

    // ---- stage the input pixels under the tile; clear the expanded-pixel buffers; biases to LDS ----------------------------
    {
        v4i_r bias_e{}, bias_d{};                                       // up to 4 * NT channels with the first trip
        const bool bias_in = tid * 16 < 4 * a.Ce32;
        if (bias_in) {
            if constexpr (EXP) bias_e = *(const v4i_r*)((const unsigned char*)a.be + tid * 16);
            bias_d = *(const v4i_r*)((const unsigned char*)a.bd + tid * 16);
        }
        const auto x = image(a, n);
        const int nchunks = EXP ? t.ih * t.iw * t.cpp : 0;
        // A chunk e of the window lies CB * e bytes behind its first one, and (W - iw) pixels further for every row.  What the window reaches over the image's rows reads zeros (out of the buffer's
        // range), what it reaches over their ends the next row's pixels: the expansion reads neither.  Lanes past the last chunk copy that one again.
        const int skip = (a.W - t.iw) * a.Cin, gap = t.xp - a.Cin;
        auto stage_chunks = [&](auto zero) {                            // in chunks of 8 or 16 bytes
            using V = decltype(zero);
            constexpr int CB = sizeof(V);
            const int origin = (iy0 * a.W + ix0) * a.Cin;
            V stage[IR_BATCH];
            unsigned dst[IR_BATCH];                                     // LDS byte offset
#pragma unroll
            for (int batch = 0; batch < IR_BATCHES; ++batch) {
                if (batch > 0 && NT * IR_BATCH * batch >= nchunks) break;   // wave-uniform
#pragma unroll
                for (int i = 0; i < IR_BATCH; ++i) {
                    const int e0 = NT * (batch * IR_BATCH + i);
                    if (e0 < nchunks) {                                     // wave-uniform
                        const int e = min(e0 + tid, nchunks - 1);
                        const int q = t.cpp == 1 ? e : (int)__umulhi((unsigned)e, t.magic_cpp), py = (int)__umulhi((unsigned)q, t.magic_iw);      // 2^32 / 1 + 1 does not fit the magic number
                        stage[i] = image_load<V>(x, origin + py * skip + CB * e);
                        dst[i] = (unsigned)(CB * e + q * gap);
                    }
                }
                if (batch == 0) {
                    // the buffers of expanded pixels (two, or one per wavefront) where the tile reaches over the image's edge, the only
                    // bytes the groups do not write, and, behind them, the projection sums (GP)
                    const int bufs = (GP ? NW : ngroups > 1 ? 2 : 1) * t.e_bytes;
                    const int c0 = EXP && frame ? 0 : bufs, c1 = bufs + (GP ? MAXB * NCO * 4096 : 0);
                    for (int o = c0 + tid * 16; o < c1; o += 16 * NT) *(v4i_r*)(l_e + o) = v4i_r{0, 0, 0, 0};
                    if (bias_in) {
                        if constexpr (EXP) *(v4i_r*)(l_be + tid * 16) = bias_e;
                        *(v4i_r*)(l_bd + tid * 16) = bias_d;
                    }
                    for (int o = (NT + tid) * 16; o < 4 * a.Ce32; o += 16 * NT) {
                        if constexpr (EXP) *(v4i_r*)(l_be + o) = *(const v4i_r*)((const unsigned char*)a.be + o);
                        *(v4i_r*)(l_bd + o) = *(const v4i_r*)((const unsigned char*)a.bd + o);
                    }
                }
#pragma unroll
                for (int i = 0; i < IR_BATCH; ++i)
                    if (NT * (batch * IR_BATCH + i) < nchunks) *(V*)(l_x + dst[i]) = stage[i];
            }
        };
        if constexpr (GP || MAXK > 1) {
            if (t.wide) stage_chunks(v4i_r{});
            else stage_chunks(v2i_r{});
        } else stage_chunks(v2i_r{});
    }

    // ---- the staged pixels inside the image, in blocks of 32 for the expansion -----------------------------------------
    const int ncb = (npix + 31) >> 5;
    const float inv_sw = __builtin_amdgcn_rcpf((float)sw);              // hp < 2^9: (hp + 1/2) / sw is further from a whole number than the product's error
    int xoff[MAXCB], eoff[MAXCB];                                 // this lane's pixel in the wavefront's j-th block: byte offsets (eoff < 0: none)
#pragma unroll
    for (int j = 0; j < MAXCB; ++j) {
        const int hp = (GP ? j : wave + 4 * j) * 32 + m, hpc = min(hp, max(npix - 1, 0));
        const int ry = (int)(((float)hpc + 0.5f) * inv_sw), rx = hpc - ry * sw;
        xoff[j] = ((y0 + ry) * t.iw + x0 + rx) * t.xp + 16 * hi;
        eoff[j] = hp < npix ? (y0 + ry) * e_row + (x0 + rx) * 32 + 16 * hi : -1;
    }
    // ---- this lane's output pixel in the wavefront's s-th block ---------------------------------------------------------
    const int ty = (m * t.magic_nbw) >> 16, tx = m - ty * t.nbw;
    const bool lane_px = ty < t.nbh;
    const int tyc = lane_px ? ty : 0, txc = lane_px ? tx : 0;
    const int nblocks = t.pbw * t.pbh;
    // the last wavefronts take the first output blocks: the first ones have more of the expansion where it does not come out even
    const int dwave = 3 - wave;
    int woff[MAXB];                                                     // window origin of the lane's pixel in the expanded-pixel buffer
#pragma unroll
    for (int s = 0; s < MAXB; ++s) {
        const int b = min(GP ? s : dwave + 4 * s, nblocks - 1), by = (b * t.magic_pbw) >> 16, bx = b - by * t.pbw;
        woff[s] = (by * t.nbh + tyc) * STRIDE * e_row + (bx * t.nbw + txc) * STRIDE * 32 + 16 * hi;
    }

    const unsigned char* const we_lane = (const unsigned char*)a.we + (size_t)m * a.Kx + 16 * hi;       // + g * 32 * Kx + k * 32
    const unsigned wd_lane = (unsigned)lane * 16, wp_lane = (unsigned)(m * a.Ce32 + 16 * hi);           // behind a uniform address: one register each
    v4i_r we[EXP ? MAXK : 1], wd[5], wp[NCO];
    const int sparse = 0x11111111 * ((m & 3) == 3 ? 12 : 12 | (m & 3));   // which two of four reduction bytes the lane's row keeps: its own and (of no weight) another
    v16i_r accp[MAXB][NCO];
#pragma unroll
    for (int s = 0; s < MAXB; ++s)
#pragma unroll
        for (int c = 0; c < NCO; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {                               // pixels shared out: the sums start at the bias; it is padded to whole
                v4i_r b4 = v4i_r{0, 0, 0, 0};                           // blocks of 32, rounding constant included
                if constexpr (!GP) b4 = *(const v4i_r*)(a.bp + 32 * c + 8 * q + 4 * hi);
#pragma unroll
                for (int e = 0; e < 4; ++e) accp[s][c][4 * q + e] = b4[e];
            }

    auto load_we = [&](int g) {
#pragma unroll
        for (int k = 0; k < MAXK; ++k)
            if (k < kx32) we[k] = *(const v4i_r*)(we_lane + (size_t)g * 32 * a.Kx + k * 32);
    };
    auto load_wd_wp = [&](int g) {
#pragma unroll
        for (int k = 0; k < 5; ++k) wd[k] = *(const v4i_r*)((const unsigned char*)a.wd + (size_t)(g * 5 + k) * 1024 + wd_lane);
#pragma unroll
        for (int c = 0; c < NCO; ++c) wp[c] = *(const v4i_r*)((const unsigned char*)a.wp + ((size_t)c * 32 * a.Ce32 + g * 32) + wp_lane);
    };
    auto bias16 = [&](const unsigned char* lb, int g) {                 // the group's bias in the accumulator layout
        v16i_r acc;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v4i_r b4 = *(const v4i_r*)(lb + 4 * (g * 32 + 8 * q + 4 * hi));
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * q + e] = b4[e];
        }
        return acc;
    };
    auto expand = [&](int g, unsigned char* ebuf) {
        const v16i_r bias = bias16(l_be, g);                            // once: read in front of every block it was a quarter of the kernel's LDS traffic
#pragma unroll
        for (int j = 0; j < MAXCB; ++j)
            if ((GP ? j : wave + 4 * j) < ncb) {                        // wave-uniform
                v16i_r acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(we[0], *(const v4i_r*)(l_x + xoff[j]), bias, 0, 0, 0);
#pragma unroll
                for (int k = 1; k < MAXK; ++k)
                    if (k < kx32) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(we[k], *(const v4i_r*)(l_x + xoff[j] + k * 32), acc, 0, 0, 0);
                const v4i_r out = ir_requant_any(acc, cl_e);
                if (eoff[j] >= 0) *(v4i_r*)(ebuf + eoff[j]) = out;
            }
    };
    // without expansion: the group's 32 channels of the tile's input pixels, 16 bytes per lane and load, zeros past the last
    // channel and outside the image.  Loads and stores are separate so that the loads of
    // the next group can be in flight over the work on this one.
    constexpr int FT = GP ? 64 : NT;                                    // lanes that fill one buffer: a wavefront's own (GP) or the workgroup's
    v4i_r fl[EXP ? 1 : IR_FILL];
    auto fill_load = [&](int g) {
        if constexpr (!EXP) {
            const auto x = image(a, n);
            const int nch = t.ih * t.iw * 2, ft = GP ? lane : tid;
#pragma unroll
            for (int i = 0; i < IR_FILL; ++i)
                if (FT * i < nch) {                                     // wave-uniform; lanes past the last chunk copy that one again
                    const int e = min(FT * i + ft, nch - 1), p = e >> 1, half = e & 1;
                    const int py = (int)__umulhi((unsigned)p, t.magic_iw), px = p - py * t.iw, ix = ix0 + px, ch = g * 32 + 16 * half;
                    const int at = ((iy0 + py) * a.W + ix) * a.Cin + ch;
                    // rows outside the image lie out of the buffer's range by themselves
                    fl[i] = image_load<v4i_r>(x, (unsigned)ix < (unsigned)a.W && ch < a.Cin ? at : (int)0x80000000u);
                }
        }
    };
    auto fill_store = [&](unsigned char* ebuf) {
        if constexpr (!EXP) {
            const int nch = t.ih * t.iw * 2, ft = GP ? lane : tid;
#pragma unroll
            for (int i = 0; i < IR_FILL; ++i)
                if (FT * i < nch) {                                     // the place once more: kept over the work on a group it was registers that are short
                    const int e = min(FT * i + ft, nch - 1), py = (int)__umulhi((unsigned)(e >> 1), t.magic_iw);
                    *(v4i_r*)(ebuf + 16 * e + py * (e_row - 32 * t.iw)) = fl[i];
                }
        }
    };
    auto dw_project = [&](int g, const unsigned char* ebuf) {
        // The bias once for all blocks, but where the kernel is held to 128 registers: there it is read in front of every block.  Sixteen more registers over the loop were four to six spilled
        // to memory (3-4 MB each way a launch); 64 samples, us: 112x112 stride 2, 16 -> 96 -> 24 28.7 -> 25.8, 56x56, 24 -> 144 -> 24 22.0 -> 20.6, 28x28, 32 -> 192 -> 32 13.0 -> 11.5.
        constexpr bool ONCE = GP || MAXK > 1;
        v16i_r bias;
        if constexpr (ONCE) bias = bias16(l_bd, g);
#pragma unroll
        for (int s = 0; s < MAXB; ++s)
            if ((GP ? s : dwave + 4 * s) < nblocks) {                   // wave-uniform
                const unsigned char* win = ebuf + woff[s];
                auto tap = [&](int t) { return *(const v4i_r*)(win + t / 3 * e_row + t % 3 * 32); };
                if constexpr (!ONCE) bias = bias16(l_bd, g);
                v16i_r acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wd[0], tap(0), bias, 0, 0, 0);
#pragma unroll
                for (int k = 1; k < 5; ++k)
                    acc = __builtin_amdgcn_smfmac_i32_32x32x64_i8(wd[k], __builtin_shufflevector(tap(2 * k - 1), tap(2 * k), 0, 1, 2, 3, 4, 5, 6, 7), acc, sparse, 0, 0);
                const v4i_r dq = ir_requant_any(acc, cl_d);
#pragma unroll
                for (int c = 0; c < NCO; ++c) accp[s][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wp[c], dq, accp[s][c], 0, 0, 0);
            }
    };

    int* const l_r = (int*)(l_e + NW * t.e_bytes);                       // GP: projection sums [block][output block][register][lane]
    if constexpr (GP) {
        unsigned char* const my_e = l_e + wave * t.e_bytes;
        __syncthreads();                                                // staged pixels, cleared buffers and biases are in LDS
        for (int g = wave; g < ngroups; g += NW) {
            if constexpr (EXP) load_we(g); else fill_load(g);
            load_wd_wp(g);
            if constexpr (EXP) expand(g, my_e); else fill_store(my_e);
            dw_project(g, my_e);                                        // same wavefront, same buffer: LDS keeps a wavefront's accesses in order
        }
#pragma unroll
        for (int s = 0; s < MAXB; ++s)
            if (s < nblocks)
#pragma unroll
                for (int c = 0; c < NCO; ++c)
#pragma unroll
                    for (int i = 0; i < 16; ++i) atomicAdd(l_r + ((s * NCO + c) * 16 + i) * 64 + lane, accp[s][c][i]);
        __syncthreads();                                                // all four partial sums are in
    } else {
        constexpr bool LATE = !EXP && NCO == 1;                         // the next group's pixels behind this group's work: held over it they cost the registers of a fourth workgroup on the CU
        if constexpr (EXP) load_we(0); else fill_load(0);
        load_wd_wp(0);
        __syncthreads();                                                // staged pixels, cleared buffers and biases are in LDS
        if constexpr (EXP) expand(0, l_e); else fill_store(l_e);
        for (int g = 0; g < ngroups; ++g) {
            if (g + 1 < ngroups) {
                if constexpr (EXP) load_we(g + 1);
                else if constexpr (!LATE) fill_load(g + 1);
            }
            __syncthreads();                                            // group g is in its buffer; nobody reads the other buffer any more
            dw_project(g, l_e + (g & 1) * t.e_bytes);
            if (g + 1 < ngroups) {
                if constexpr (LATE) fill_load(g + 1);
                load_wd_wp(g + 1);
                if constexpr (EXP) expand(g + 1, l_e + ((g + 1) & 1) * t.e_bytes); else fill_store(l_e + ((g + 1) & 1) * t.e_bytes);
            }
        }
    }

    // ---- epilogue: bias, residual, requantisation, stores, the exit head's pooling ------------------------------------------------------------------
    v4i_r unit;                                                         // the unit matrix as a B operand: column m, channels 16 hi .. 16 hi + 15
    if constexpr (POOL)
#pragma unroll
        for (int w = 0; w < 4; ++w) unit[w] = (m >> 2) == 4 * hi + w ? 1 << (8 * (m & 3)) : 0;
#pragma unroll
    for (int s = 0; s < MAXB; ++s)
        if ((GP ? s : dwave + 4 * s) < nblocks) {                       // wave-uniform
            const int b = GP ? s : dwave + 4 * s, by = (b * t.magic_pbw) >> 16, bx = b - by * t.pbw;
            int me = m;
            if constexpr (!EXP && NCO == 1) asm volatile("" : "+v"(me));        // the lane's place in the block once more: kept over the groups it was two registers in scratch memory
            const int ey = (me * t.magic_nbw) >> 16, ex = me - ey * t.nbw;
            const int oy = oy0 + by * t.nbh + ey, ox = ox0 + bx * t.nbw + ex;
            const bool px_ok = ey < t.nbh && oy < a.Ho && ox < a.Wo;
            const unsigned pix = px_ok ? (unsigned)(((n * a.Ho + oy) * a.Wo + ox) * a.Cout) : 0u;      // < 2^31: checked by the launcher
#pragma unroll
            for (int c = 0; c < NCO; ++c) {
                if (GP && ((s * NCO + c) & (NW - 1)) != wave) continue; // wave-uniform: the (pixel block, output block) pairs take turns
                const int ch = 32 * c + 16 * hi;                        // first of the 16 channels this lane stores
                const int left = a.Cout - ch;                           // channels from there on (a multiple of 8)
                v16i_r acc = accp[s][c];
                if constexpr (GP) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const v4i_r b4 = *(const v4i_r*)(a.bp + 32 * c + 8 * q + 4 * hi);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[4 * q + e] = l_r[((s * NCO + c) * 16 + 4 * q + e) * 64 + lane] + b4[e];
                    }
                }
                if (a.res) {
                    // the residual in the store layout, unconditional and in range, then back into the accumulator layout
                    const unsigned char* rp = (const unsigned char*)a.res + pix + (left >= 8 ? ch : 0);
                    const v2i_r r01 = *(const v2i_r*)rp, r23 = *(const v2i_r*)(rp + (left >= 16 ? 8 : 0));
                    const auto s02 = __builtin_amdgcn_permlane32_swap((unsigned)r01[0], (unsigned)r01[1], false, false);
                    const auto s13 = __builtin_amdgcn_permlane32_swap((unsigned)r23[0], (unsigned)r23[1], false, false);
                    const unsigned rq[4] = {s02[0], s13[0], s02[1], s13[1]};
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[4 * q + e] += __builtin_amdgcn_sbfe((int)rq[q], 8 * e, 8) << a.res_shift;
                }
                const v4i_r out = ir_requant_any(acc, cl_p);
                if constexpr (POOL) {
                    // channel sums of the block's 32 pixels: the results are in operand layout (row = pixel), and times the unit matrix they come back with a
                    // lane per channel and the pixels in its registers
                    v16i_r t16 = {};
                    t16 = __builtin_amdgcn_mfma_i32_32x32x32_i8(px_ok ? out : v4i_r{0, 0, 0, 0}, unit, t16, 0, 0, 0);
                    int sum = 0;
#pragma unroll
                    for (int e = 0; e < 16; ++e) sum += t16[e];
                    if (32 * c + m < a.Cout) atomicAdd(a.gap_sums + (size_t)n * a.Cout + 32 * c + m, sum);      // both halves of the wavefront, half of the pixels each
                }
                if (px_ok) {
                    unsigned char* yp = (unsigned char*)a.y + pix + ch;
                    if (left >= 16) *(v4i_r*)yp = out;
                    else if (left >= 8) *(v2i_r*)yp = v2i_r{out[0], out[1]};
                }
            }
        }
}

int ir_block_out_blocks(int c_out)
{
    const int nco = (c_out + 31) / 32;
    return nco == 4 ? 5 : nco;                                          // instantiated: 1, 2, 3, 5 blocks of 32 output channels
}

// Shapes the kernel covers, and the tile it takes them with.
bool ir_block_plan(const IrArgs& a, IrTile& t, int& nco, int& maxb)
{
    if ((a.stride != 1 && a.stride != 2) || a.pad != 1 || a.B < 1) return false;
    const bool expands = a.Kx > 0;                                      // Kx = 0: depthwise -> projection, no expansion in front
    if (a.Cout % 8 != 0 || a.Ce32 % 32 != 0 || a.Ce32 < 32) return false;
    if (expands ? (a.Cin % 8 != 0 || a.Cin > 32 * IR_MAXK || a.Kx % 32 != 0 || a.Kx < a.Cin) : (a.Cin % 16 != 0 || a.Ce32 < a.Cin || a.Ce32 - a.Cin >= 32)) return false;
    if ((double)a.B * a.H * a.W * a.Cin >= 2147483648.0 || (double)a.B * a.Ho * a.Wo * a.Cout >= 2147483648.0) return false;
    nco = ir_block_out_blocks(a.Cout);
    if (nco > 5) return false;
    maxb = nco == 1 ? 2 : nco <= 3 ? 2 : 1;
    t.nbw = a.Wo % 8 == 0 ? 8 : a.Wo % 14 == 0 ? 14 : a.Wo % 7 == 0 ? 7 : 8;
    t.nbh = 32 / t.nbw;
    const int bx_max = (a.Wo + t.nbw - 1) / t.nbw, by_max = (a.Ho + t.nbh - 1) / t.nbh;
    t.pbw = 1; t.pbh = 1; t.gp = 0;
    auto fits = [&] {
        t.iw = (t.pbw * t.nbw - 1) * a.stride + 3;
        t.ih = (t.pbh * t.nbh - 1) * a.stride + 3;
        t.wide = a.Cin % 16 == 0 && (t.gp || a.Kx > 32);                // Where the kernel has both (14x14, 64 -> 384 -> 64, 1 sample 6.3 / 6.1 us,
                                                                        // 7x7, 160 -> 960 -> 160 12.0 / 11.4): elsewhere a second form's code costs 24 channels 1-2 %, more than 16 and 32 gain
        t.cpp = expands ? a.Cin / (t.wide ? 16 : 8) : 1;
        t.xp = a.Kx + 16;
        t.x_bytes = expands ? t.ih * t.iw * t.xp + 128 : 0;             // the last pixel's reduction bytes may be read past its channels
        t.e_bytes = t.ih * (t.iw * 32 + 16);
        if (t.pbw * t.pbh > 4 * maxb || 8 * a.Ce32 + t.x_bytes + 2 * t.e_bytes > 64 * 1024) return false;
        return expands ? t.ih * t.iw <= 128 * ir_maxcb(0, a.stride) && t.ih * t.iw * t.cpp <= 256 * IR_BATCH * IR_BATCHES
                       : t.ih * t.iw * 2 <= 256 * IR_FILL;
    };
    if (!fits()) return false;
    // Few tiles: the wavefronts share the channel groups of a tile of one block, or two where one-block tiles would not all run at once (a workgroup to a CU, two where one output block leaves
    // registers for them).  A tile's time is a chain of groups whatever the number of tiles, so both forms' times are steps of whole rounds and the line lies where a round of the groups' form stops
    // paying.  Back to back, the pixels shared out / the groups, us (tiles):
    //   one output block, stride 1: 28x28, 32 -> 192 -> 32, 8 samples 6.5 / 5.2, 32 (448) 8.7 / 7.6, 40 (560) 10.1 / 10.7, 48 (672) 12.6 / 10.8, 54 (756) 12.6 / 10.9, 64 (896) 11.4 / 13.0; 40x40,
    //     8 samples (400) 7.1 / 6.1, 12 (600) 8.3 / 8.8; 32x32, 32 -> 160 -> 32, 24 samples (768) 8.1 / 8.9: between 512 and 768 either may be the faster one by a tenth
    //   stride 2, to three output blocks: 56x56, 24 -> 144 -> 32, 8 samples (224) 6.9 / 5.8, 10 (280) 7.5 / 9.6; 28x28, 32 -> 192 -> 64, 32 (224) 7.7 / 6.4, 37 (259) 8.5 / 10.8
    //   two or three output blocks, stride 1, one reduction step: 28x28, 32 -> 192 -> 64, 18 samples (252) 7.6 / 6.2, 24 (336) 8.7 / 10.6; to 96, 16 (224) 8.7 / 6.9, 24 9.5 / 12.1; more steps or
    //     none: 14x14, 64 -> 384 -> 64, 128 (512) 17.6 / 14.4, 160 (640) 21.4 / 20.6, 256 19.9 / 27.4, 40 samples in 280 tiles of one block 11.2, in 160 of two 8.3; 128 -> 64 without expansion, 128
    //     samples (512) 7.6 / 5.8
    //   five output blocks, one reduction step: 28x28, 32 -> 192 -> 128, 9 samples (252) 7.8 / 6.2, 16 (448) 10.5 / 10.8, 32 (896) 11.1 / 20.5; stride 2, to 160, 36 (252) 9.1 / 7.2, 64 (448) 10.8 / 12.9;
    //     more steps or none: 14x14 stride 2, 96 -> 576 -> 160, 1 to 128 samples 19.5 / 10.5, 384 (768) 29.5 / 28.8, 448 (896) 29.7 / 37.2; 64 -> 384 -> 160, 109 (763) 24.5 / 19.7, 128 (896) 16.3 /
    //     25.3; 160 -> 160 without expansion 109 11.4 / 10.8, 128 10.2 / 12.0; 7x7, 160 -> 960 -> 160, 384 (768) 46.7 / 37.9, 512 (1024) 48.1 / 49.1
    if (a.Ce32 >= (a.Kx == 32 ? 160 : 128) && (a.Kx == 32 || nco >= 2)) {       // the forms that are instantiated
        const int nw = a.Ce32 >= (a.Kx == 32 ? 160 : 320) ? 8 : 4;
        const long long limit = nco == 1 ? (a.stride == 1 ? 768 : 256) : a.Kx == 32 ? 256 : nco == 5 ? 768 : a.stride == 1 ? 512 : 256;
        auto shared_tiles = [&](int blocks) -> long long {                      // how many tiles of that many blocks there are, 0: they do not fit
            t.pbw = t.pbh = 1; t.gp = nw;
            if (blocks == 2) (by_max > 1 && (bx_max == 1 || t.nbh <= t.nbw) ? t.pbh : t.pbw) = 2;
            if (t.pbw > bx_max || !fits() || 8 * a.Ce32 + t.x_bytes + nw * t.e_bytes + maxb * nco * 4096 > IR_SHARED_LDS) return 0;
            const int px = t.ih * t.iw;
            if (expands ? px > 32 * ir_maxcb(nw, a.stride) || px * t.cpp > 64 * nw * IR_BATCH * IR_BATCHES : px * 2 > 64 * IR_FILL) return 0;
            return (long long)a.B * ((bx_max + t.pbw - 1) / t.pbw) * ((by_max + t.pbh - 1) / t.pbh);
        };
        const long long one = shared_tiles(1);
        long long n = one;
        if (maxb == 2 && (one == 0 || one > 256)) {
            n = shared_tiles(2);
            if (n == 0) n = shared_tiles(1);
        }
        if (n == 0 || n > limit) t.pbw = t.pbh = 1, t.gp = 0;
    }
    while (!t.gp) {                                                     // grow the shorter side in pixels while the tile fits
        const bool can_x = t.pbw < bx_max, can_y = t.pbh < by_max;
        const bool prefer_y = can_y && (!can_x || t.pbh * t.nbh <= t.pbw * t.nbw);
        bool grown = false;
        for (int pass = 0; pass < 2 && !grown; ++pass) {
            const bool grow_y = pass == 0 ? prefer_y : !prefer_y;
            if (grow_y ? !can_y : !can_x) continue;
            (grow_y ? t.pbh : t.pbw) += 1;
            const long long wgs = (long long)a.B * ((bx_max + t.pbw - 1) / t.pbw) * ((by_max + t.pbh - 1) / t.pbh);
            if (fits() && wgs >= 256) grown = true; else (grow_y ? t.pbh : t.pbw) -= 1;   // a larger tile only while every CU still gets a workgroup
        }
        if (!grown) break;
    }
    fits();
    t.tiles_x = (bx_max + t.pbw - 1) / t.pbw;
    t.tiles_y = (by_max + t.pbh - 1) / t.pbh;
    t.magic_cpp = t.cpp > 1 ? (unsigned)(4294967296.0 / t.cpp) + 1u : 0u;
    t.magic_iw = (unsigned)(4294967296.0 / t.iw) + 1u;
    const long long total = (long long)a.B * t.tiles_x * t.tiles_y;
    if (total > 0x3fffffff || total * std::max(t.tiles_x, t.tiles_y) > 0xffffffffLL) return false;
    t.magic_tx = t.tiles_x > 1 ? (unsigned)(4294967296.0 / t.tiles_x) + 1u : 0u;
    t.magic_ty = t.tiles_y > 1 ? (unsigned)(4294967296.0 / t.tiles_y) + 1u : 0u;
    t.magic_nbw = 65536 / t.nbw + 1;
    t.magic_pbw = 65536 / t.pbw + 1;
    t.total = (int)total;
    return true;
}

bool ir_block_pools(const IrArgs& a) { return a.stride == 1; }      // built for the blocks that can end a segment with their input as residual

bool ir_block_supported(const IrArgs& a)
{
    IrTile t;
    int nco, maxb;
    return ir_block_plan(a, t, nco, maxb);
}

template <int STRIDE, int NCO, int MAXB, int MAXK, int GP, bool POOL>
static hipError_t ir_launch6(const IrArgs& a, const IrTile& t, size_t lds, hipStream_t s)
{
    if (lds > 64 * 1024) {                                              // a grant that failed once fails every launch that needs it
        static const hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void*>(&ir_block_i8_kernel<STRIDE, NCO, MAXB, MAXK, GP, POOL>), hipFuncAttributeMaxDynamicSharedMemorySize, IR_SHARED_LDS);
        if (granted != hipSuccess) return granted;
    }
    EE_LAUNCH((ir_block_i8_kernel<STRIDE, NCO, MAXB, MAXK, GP, POOL>), dim3(xcd_grid(t.total)), dim3(GP ? 64 * GP : 256), lds, s, a, t);
    return hipGetLastError();
}

template <int STRIDE, int NCO, int MAXB, int MAXK, int GP>
static hipError_t ir_launch5(const IrArgs& a, const IrTile& t, size_t lds, hipStream_t s)
{
    if constexpr (STRIDE == 1) {
        if (a.gap_sums) return ir_launch6<1, NCO, MAXB, MAXK, GP, true>(a, t, lds, s);
    }
    return ir_launch6<STRIDE, NCO, MAXB, MAXK, GP, false>(a, t, lds, s);
}

template <int STRIDE, int NCO, int MAXB>
static hipError_t ir_launch(const IrArgs& a, const IrTile& t, size_t lds, hipStream_t s)
{
    const int kx32 = a.Kx >> 5;                                         // registers for the expansion weights: 1, 2 or 5 steps
    if (kx32 == 0) {                                                    // no expansion
        if constexpr (NCO >= 2) {
            if (t.gp == 4) return ir_launch5<STRIDE, NCO, MAXB, 0, 4>(a, t, lds, s);
            if (t.gp == 8) return ir_launch5<STRIDE, NCO, MAXB, 0, 8>(a, t, lds, s);
        }
        return ir_launch5<STRIDE, NCO, MAXB, 0, 0>(a, t, lds, s);
    }
    if constexpr (NCO >= 2) {
        if (t.gp == 4) return kx32 <= 2 ? ir_launch5<STRIDE, NCO, MAXB, 2, 4>(a, t, lds, s) : ir_launch5<STRIDE, NCO, MAXB, IR_MAXK, 4>(a, t, lds, s);
        if (t.gp == 8 && kx32 > 1) return kx32 <= 2 ? ir_launch5<STRIDE, NCO, MAXB, 2, 8>(a, t, lds, s) : ir_launch5<STRIDE, NCO, MAXB, IR_MAXK, 8>(a, t, lds, s);
    }
    if (kx32 <= 1 && t.gp == 8) return ir_launch5<STRIDE, NCO, MAXB, 1, 8>(a, t, lds, s);
    if (kx32 <= 1) return ir_launch5<STRIDE, NCO, MAXB, 1, 0>(a, t, lds, s);
    if (kx32 <= 2) return ir_launch5<STRIDE, NCO, MAXB, 2, 0>(a, t, lds, s);
    return ir_launch5<STRIDE, NCO, MAXB, IR_MAXK, 0>(a, t, lds, s);
}

hipError_t launch_ir_block(const IrArgs& a, hipStream_t s)
{
    IrTile t;
    int nco, maxb;
    if (!ir_block_plan(a, t, nco, maxb) || (a.gap_sums && !ir_block_pools(a))) return hipErrorInvalidValue;
    const size_t lds = (size_t)8 * a.Ce32 + t.x_bytes + (t.gp ? t.gp * (size_t)t.e_bytes + (size_t)maxb * nco * 4096 : (a.Ce32 > 32 ? 2 : 1) * (size_t)t.e_bytes);
    const int v = (a.stride - 1) * 4 + (nco == 1 ? 0 : nco == 2 ? 1 : nco == 3 ? 2 : 3);
    switch (v) {
    case 0: return ir_launch<1, 1, 2>(a, t, lds, s);
    case 1: return ir_launch<1, 2, 2>(a, t, lds, s);
    case 2: return ir_launch<1, 3, 2>(a, t, lds, s);
    case 3: return ir_launch<1, 5, 1>(a, t, lds, s);
    case 4: return ir_launch<2, 1, 2>(a, t, lds, s);
    case 5: return ir_launch<2, 2, 2>(a, t, lds, s);
    case 6: return ir_launch<2, 3, 2>(a, t, lds, s);
    default: return ir_launch<2, 5, 1>(a, t, lds, s);
    }
}

}  // namespace ee
