// Bottleneck block (bf16) of the 56 x 56 group of ResNet-50-style networks in one launch, for gfx950: the bf16 form of
// bneck_block_i8_kernel (kernels_bneck.hip): 1x1 reduction (64 or 256 -> 64 channels) -> 3x3 (64 -> 64, stride 1) -> 1x1 expansion
// (64 -> 256) + residual, or, with the 1x1 convolution on the block's shortcut inside, four layers.  Layer by layer a block of 256 samples moves
// 1.85 GB; here it reads its input and writes its output, 0.82 GB.
//
// One persistent workgroup of eight wavefronts per CU walks over tiles of 8 x 8 output pixels.  All weights (137 KB) stay in registers as
// ready matrix-instruction operands, so wavefronts have roles, one of each per SIMD:
//   first half   front (wavefronts 0-3), one tile ahead: 32 of the 10 x 10 input pixels under tile i + 1 each, both blocks of 32 middle
//                channels.  A wavefront's pixels are read by nobody else, so it copies them itself (asynchronously, global -> LDS, a
//                whole tile ahead, in pieces of 64 channels through a ring of its own) and waits for its own copies only: no
//                barrier between copy and use.  Results go to LDS as the second layer's input, zeros outside the image.
//                back (wavefronts 4-7), tile i: request the residual tile into LDS, then (8 x 4 pixels, 32 of the middle channels) each:
//                nine taps x four steps, the result to LDS as the last layer's operands;
//   second half  all eight: (8 x 4 pixels, 64 of the 256 output channels) each: last layer, bias, residual, clamp, rounding in place of the
//                residual in LDS, read back in whole lines and stored.
// Two workgroup barriers per tile that wait for LDS only; copies and stores are counted with vmcnt, which the fixed number of them per tile allows
// (lanes outside the image store out of the buffer's range: the instruction still counts).  Sums run in the order of the staged kernel and values are
// rounded to bf16 where the layers store them: the results are those of the separate layers bit for bit.
//
// Measured at 256 samples of 56 x 56: identity blocks 332 us as three launches, 191 fused (4.3 TB/s in and out); the first block 262 / 177 without its
// shortcut, 373 / 159 with it.  What bounds the identity blocks: memory.  Counters, 208 samples a launch: 626 MB read, the input 1.9 times (the residual tile is
// requested two tiles after the same pixels, when little of it can still be in the XCD's L2), 335 MB written, 5.6 TB/s over a launch; the tensors alone would be 120 us at
// that rate.  The first block reads 85 MB and writes 335 in 149 us: matrix instructions 56 us, LDS 67 us and vector issue about as much at 256 samples, in two halves per
// tile that overlap only through the second wavefront of each SIMD.  Few samples: a whole first segment (first layer included, untuned) of 1
// sample 59 -> 42 us, 5 samples 77 -> 51, 37 samples 233 -> 140, 256 samples 1542 -> 765, so untuned launches are fused at every size.
#include "ee_internal.hpp"
#include "igemm_device.hpp"

namespace ee {

struct Bn16Tile {
    int tiles_x, tiles_y;      // tiles of 8 x 8 output pixels per image
    int total;                 // tiles in all
    int nslots;                // workgroups per XCD
};

constexpr int B16_M1_PX = 128 + 16;                // second layer's input: bytes per pixel
constexpr int B16_M1_ROW = 6 * 256 + 128;          // ten pixels; rows half a bank cycle apart: the 16 lanes of a phase (two rows of eight pixels) touch all banks once
constexpr int B16_M1_BYTES = 10 * B16_M1_ROW;
constexpr int B16_M2_BYTES = 8 * 1024;             // last layer's operands [pixel block][step][lane][16]
constexpr int B16_OUT_BYTES = 64 * 512;            // residual tile, then output tile: rows of 32 chunks, chunk c of pixel p at c ^ (p & 31)
constexpr int B16_BIAS_BYTES = 4 * (64 + 64 + 256 + 256);
constexpr int B16_SLOT_BYTES = 2 * EE_ZC_MAX_B;
constexpr int b16_ring(int nc, bool sc) { return nc == 4 ? 5 : sc ? 3 : 2; }       // pieces: one more than are in flight; with the shortcut also the tile whose last layer is due
constexpr int b16_lds(int nc, bool sc)
{
    return b16_ring(nc, sc) * 4 * 4096 + 2 * B16_M1_BYTES + B16_M2_BYTES + B16_OUT_BYTES + B16_BIAS_BYTES + B16_SLOT_BYTES + (sc ? 32 * 1024 : 0);
}
static_assert(b16_lds(4, false) <= 160 * 1024 && b16_lds(1, true) <= 160 * 1024 && b16_lds(1, false) <= 160 * 1024, "LDS of a CU");

// NC: input channels / 64; SC: the residual is a 1x1 convolution of the block's input (64 -> 256 channels), rounded to bf16 as that layer would store it
template <int NC, bool SC>
__global__ __launch_bounds__(512, 1) __attribute__((amdgpu_waves_per_eu(2, 2))) void bneck_block_bf16_kernel(IrArgs a, Bn16Tile t)
{
    request_args<sizeof(IrArgs) + sizeof(Bn16Tile)>();
    static_assert(!SC || NC == 1, "the shortcut convolution reads 64 channels");
    constexpr int PB = NC * 128, RING = b16_ring(NC, SC);               // bytes per input pixel, pieces per front wavefront
    extern __shared__ __attribute__((aligned(16))) unsigned char b16_raw[];
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool front = wave < 4;
    const int xcd = (int)(blockIdx.x & 7), slot = (int)(blockIdx.x >> 3);
    const int u_xcd = xcd_first(xcd, t.total), cnt = xcd_first(xcd + 1, t.total) - u_xcd;      // tiles of this XCD
    if (cnt <= slot) return;                                           // whole workgroup: no barrier is skipped by a part of it
    const int T = (cnt - slot + t.nslots - 1) / t.nslots;              // tiles of this workgroup: u0, u0 + nslots, ...
    const int u0 = u_xcd + slot, tpi = t.tiles_x * t.tiles_y;
    unsigned char* const l_x = b16_raw;                                 // [ring][front wavefront][32 pixels][128]
    unsigned char* const l_m1 = l_x + RING * 4 * 4096;
    unsigned char* const l_m2 = l_m1 + 2 * B16_M1_BYTES;
    unsigned char* const l_out = l_m2 + B16_M2_BYTES;
    float* const l_b1 = (float*)(l_out + B16_OUT_BYTES);
    float* const l_b2 = l_b1 + 64;
    float* const l_b3 = l_b1 + 128;
    float* const l_bs = l_b1 + 384;
    unsigned short* const l_slot = (unsigned short*)(l_b1 + 640);
    unsigned char* const l_ws = (unsigned char*)(l_b1 + 640) + B16_SLOT_BYTES;     // the shortcut's operands [block][step][lane][16] (SC)
    const unsigned lds0 = lds_addr(b16_raw), out0 = lds_addr(l_out);

    if (tid < 64) { l_b1[tid] = ((const float*)a.be)[tid]; l_b2[tid] = ((const float*)a.bd)[tid]; }
    if (tid < 256) l_b3[tid] = ((const float*)a.bp)[tid];
    if constexpr (SC) {
        if (tid < 256) l_bs[tid] = ((const float*)a.bs)[tid];
#pragma unroll
        for (int i = 0; i < 4; ++i) *(v4i*)(l_ws + (512 * i + tid) * 16) = *(const v4i*)((const unsigned char*)a.ws + (512 * i + tid) * 16);
    }
    if (a.ys && tid < a.B) l_slot[tid] = a.ys[tid];                     // B <= EE_ZC_MAX_B <= 512 with a slot table: checked by the launcher

    // A workgroup's tiles are nslots apart: a tile's (sample, tile row, tile column) follows from the one before by additions
    struct Cursor { int n, ty, tx; };
    const int step_n = t.nslots / tpi, step_r = t.nslots - step_n * tpi, step_ty = step_r / t.tiles_x, step_tx = step_r - step_ty * t.tiles_x;
    auto advance = [&](Cursor& c) {
        c.tx += step_tx;
        if (c.tx >= t.tiles_x) { c.tx -= t.tiles_x; ++c.ty; }
        c.ty += step_ty;
        if (c.ty >= t.tiles_y) { c.ty -= t.tiles_y; ++c.n; }
        c.n += step_n;
    };
    Cursor c_out;                                                       // the tile of the last layer
    c_out.n = u0 / tpi;
    c_out.ty = (u0 - c_out.n * tpi) / t.tiles_x;
    c_out.tx = u0 - c_out.n * tpi - c_out.ty * t.tiles_x;

    // ---- the last layer: (pixel block, two of the eight blocks of 32 output channels) per wavefront of either role ------------------
    const int pb = wave & 1, half = (wave >> 1) & 1;
    const int cb0 = 4 * half + (front ? 2 : 0);
    auto load_w3 = [&](v4i (&w3)[2][4]) {                               // operands [block][step]
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) w3[c][k] = *(const v4i*)((const unsigned char*)a.wp + ((size_t)((cb0 + c) * 4 + k) * 64 + lane) * 16);
    };
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(a.y, (short)0, 0x7fffffff, 0x00020000);
    int xs_slot = 0;                                                    // ring piece of the tile in hand (SC)
    auto last_layer = [&](const v4i (&w3)[2][4]) {
        const int n = c_out.n, oy0 = 8 * c_out.ty, ox0 = 8 * c_out.tx;
        // addresses are worked out here each time: kept over the loop they would not fit beside the weights
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
        const int m = lane & 31, hi = lane >> 5;
        const int hp_out = (4 * pb + (m >> 3) + 1) * 10 + (m & 7) + 1;      // the lane's output pixel among the staged ones (SC)
        const int xs_row = hp_out & 31, xs_wave = hp_out >> 5;
        unsigned char* const cell0 = l_out + (32 * pb + m) * 512 + 8 * hi;
        v4i d[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = *(const v4i*)(l_m2 + ((pb * 4 + k) * 64 + lane) * 16);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint2 res[4];
            if constexpr (SC) {
                v16f s;
#pragma unroll
                for (int i = 0; i < 16; ++i) s[i] = 0.f;
                const unsigned char* xp = l_x + (xs_slot * 4 + xs_wave) * 4096 + xs_row * 128;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const v4i x = *(const v4i*)(xp + (((2 * k + hi) ^ (xs_row >> 1 & 7)) << 4));
                    const v4i w = *(const v4i*)(l_ws + (((cb0 + c) * 4 + k) * 64 + lane) * 16);
                    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, w), __builtin_bit_cast(v8bf, x), s, 0, 0, 0);
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4i b4 = *(const v4i*)(l_bs + (cb0 + c) * 32 + 8 * g + 4 * hi);
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = clamp_f32(s[4 * g + e] + __int_as_float(b4[e]), a.f_lo_s, a.f_hi_s);
                    res[g] = uint2{pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
                }
            }
            v16f acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, w3[c][k]), __builtin_bit_cast(v8bf, d[k]), acc, 0, 0, 0);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                unsigned char* cell = cell0 + ((((cb0 + c) * 4 + g) ^ m) << 4);
                const uint2 r = SC ? res[g] : *(const uint2*)cell;
                const v4i b4 = *(const v4i*)(l_b3 + (cb0 + c) * 32 + 8 * g + 4 * hi);
                const float r4[4] = {__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xFFFF0000u), __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xFFFF0000u)};
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = clamp_f32((acc[4 * g + e] + __int_as_float(b4[e])) + r4[e], a.f_lo_p, a.f_hi_p);
                *(uint2*)cell = uint2{pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
            }
        }
        // this wavefront's 32 pixels x 128 bytes back in whole lines; nobody else has touched them.  Always four stores
        const int slot_n = a.ys ? (int)l_slot[n] : n;
        const unsigned base = (unsigned)(slot_n * a.H * a.W + (oy0 + 4 * pb) * a.W + ox0) * 512u + (unsigned)cb0 * 64u;       // < 2^31: checked by the launcher
        const int sx = lane >> 3, sc = lane & 7;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = 8 * j + sx;
            const v4i v = *(const v4i*)(l_out + (32 * pb + p) * 512 + (((cb0 * 4 + sc) ^ p) << 4));
            const bool ok = oy0 + 4 * pb + j < a.H && ox0 + sx < a.W;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, v), rsrc, ok ? (int)(base + (unsigned)((j * a.W + sx) * 512 + 16 * sc)) : (int)0x80000000u, 0, 0);
        }
        advance(c_out);
    };

    // Each role has its own loop; both run the same iterations with the same two barriers, so the workgroup's barriers pair up.  Weights are
    // loaded inside the branch: arrays shared by the roles cost copies, and copies at this many registers are spills.
    if (front) {
        v4i w1[8 * NC], w3[2][4];                                       // the first layer's operands [block][step]
#pragma unroll
        for (int k = 0; k < 8 * NC; ++k) w1[k] = *(const v4i*)((const unsigned char*)a.we + ((size_t)k * 64 + lane) * 16);
        load_w3(w3);
        const int hp = 32 * wave + m, hpc = min(hp, 99), hy = hpc / 10, hx = hpc - 10 * hy;
        unsigned char* const m1 = l_m1 + hy * B16_M1_ROW + hx * B16_M1_PX + 8 * hi;
        // this lane's share of a piece: rows 8 j + lane / 8 of the wavefront's 32 pixels
        int cpy[4], cpx[4], crel[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = 8 * j + (lane >> 3), p = min(32 * wave + row, 99);
            cpy[j] = p / 10 - 1;
            cpx[j] = p - 10 * (cpy[j] + 1) - 1;
            crel[j] = ((lane & 7) ^ (row >> 1 & 7)) * 16;
        }
        Cursor c_ld = c_out, c_l1 = c_out;                              // the tile whose pixels are requested, the tile of the first layer
        int ld_left = T - 1;                                            // tiles behind c_ld: past the last one it is requested again, nobody reads it
        unsigned voff[4];
        const unsigned char* xn = nullptr;
        auto x_tile = [&] {                                             // in range: a pixel outside the image reads the nearest one inside
            xn = (const unsigned char*)a.x + (size_t)c_ld.n * a.H * a.W * PB;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int iy = min(max(8 * c_ld.ty + cpy[j], 0), a.H - 1), ix = min(max(8 * c_ld.tx + cpx[j], 0), a.W - 1);
                voff[j] = (unsigned)((iy * a.W + ix) * PB + crel[j]);
            }
            if (ld_left > 0) { --ld_left; advance(c_ld); }
        };
        int q_ld = 0, q_use = 0;                                        // ring pieces
        auto x_piece = [&](int c) {
            const unsigned dst = lds0 + (unsigned)(q_ld * 4 + wave) * 4096u;
#pragma unroll
            for (int j = 0; j < 4; ++j) dma16(dst + j * 1024, xn + c * 128, voff[j]);
            q_ld = q_ld + 1 == RING ? 0 : q_ld + 1;
        };
        x_tile();
#pragma unroll
        for (int c = 0; c < NC; ++c) x_piece(c);
        // every weight has arrived before the loop, so that nothing inside it waits for a weight by count
#pragma unroll
        for (int k = 0; k < 8 * NC; ++k) asm volatile("" : "+v"(w1[k]));
#pragma unroll
        for (int k = 0; k < 8; ++k) asm volatile("" : "+v"(w3[k >> 2][k & 3]));
        lds_barrier();                                                  // biases are in LDS
        for (int it = -1; it < T; ++it) {
            if (it + 1 < T) {
                const int oy0 = 8 * c_l1.ty, ox0 = 8 * c_l1.tx;
                advance(c_l1);
                const bool in_img = hp < 100 && (unsigned)(oy0 - 1 + hy) < (unsigned)a.H && (unsigned)(ox0 - 1 + hx) < (unsigned)a.W;
                x_tile();
                v16f acc0, acc1;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc0[i] = acc1[i] = 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    // younger than this piece: the NC - 1 behind it and, from the second tile on, the four stores of the last layer
                    if (it >= 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * (NC - 1) + 4) : "memory");
                    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * (NC - 1)) : "memory");
                    v4i b[4];
                    const unsigned char* xp = l_x + (q_use * 4 + wave) * 4096 + m * 128;
#pragma unroll
                    for (int k = 0; k < 4; ++k) b[k] = *(const v4i*)(xp + (((2 * k + hi) ^ (m >> 1 & 7)) << 4));
                    x_piece(c);                                         // into the piece read one step ago (its operands have been multiplied)
                    q_use = q_use + 1 == RING ? 0 : q_use + 1;
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, w1[4 * c + k]), __builtin_bit_cast(v8bf, b[k]), acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, w1[4 * NC + 4 * c + k]), __builtin_bit_cast(v8bf, b[k]), acc1, 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                unsigned char* mp = m1 + ((it + 1) & 1) * B16_M1_BYTES;
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const v4i b4 = *(const v4i*)(l_b1 + 32 * j + 8 * g + 4 * hi);
                        float v[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = clamp_f32((j ? acc1 : acc0)[4 * g + e] + __int_as_float(b4[e]), a.f_lo_e, a.f_hi_e);
                        uint2 o = {pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
                        if (!in_img) o = uint2{0u, 0u};
                        if (hp < 100) *(uint2*)(mp + 64 * j + 16 * g) = o;
                    }
            }
            lds_barrier();                                              // the second layer's output and the residual tile are in LDS
            if (it >= 0) {
                last_layer(w3);
                if constexpr (SC) xs_slot = xs_slot + 1 == RING ? 0 : xs_slot + 1;
            }
            lds_barrier();                                              // tile it + 1 is through the first layer, tile it is read out
        }
    } else {
        v4i w2[36], w3[2][4];                                           // operands [tap][step] of the 3x3 layer for 32 of its channels
#pragma unroll
        for (int k = 0; k < 36; ++k) w2[k] = *(const v4i*)((const unsigned char*)a.wd + ((size_t)(half * 36 + k) * 64 + lane) * 16);
        load_w3(w3);
        const int b4w = wave - 4;                                       // its share of the residual tile: pixels 16 b4w ..
#pragma unroll
        for (int k = 0; k < 36; ++k) asm volatile("" : "+v"(w2[k]));
#pragma unroll
        for (int k = 0; k < 8; ++k) asm volatile("" : "+v"(w3[k >> 2][k & 3]));
        lds_barrier();                                                  // biases are in LDS
        for (int it = -1; it < T; ++it) {
            if (it >= 0) {
                int lane = tid & 63;                                    // as in the last layer
                asm volatile("" : "+v"(lane));
                const int m = lane & 31, hi = lane >> 5;
                if constexpr (!SC) {
                    const unsigned char* rn = (const unsigned char*)a.res + (size_t)c_out.n * a.H * a.W * 512;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int px = 16 * b4w + 2 * i + hi;
                        const int oy = min(8 * c_out.ty + (px >> 3), a.H - 1), ox = min(8 * c_out.tx + (px & 7), a.W - 1);
                        dma16(out0 + (unsigned)(16 * b4w + 2 * i) * 512u, rn, (unsigned)((oy * a.W + ox) * 512 + ((m ^ (px & 31)) << 4)));
                    }
                }
                const unsigned char* win = l_m1 + (it & 1) * B16_M1_BYTES + (pb * 4 + (m >> 3)) * B16_M1_ROW + (m & 7) * B16_M1_PX + 16 * hi;
                unsigned char* const m2 = l_m2 + ((pb * 4 + 2 * half) * 64 + m) * 16 + 8 * hi;
                auto tap = [&](int k) { return *(const v4i*)(win + (k / 12) * B16_M1_ROW + ((k / 4) % 3) * B16_M1_PX + (k & 3) * 32); };
                v16f acc;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i] = 0.f;
                // the 36 operands in batches of four through two sets of registers, a batch ahead of its matrix instructions
                v4i b[2][4];
#pragma unroll
                for (int k = 0; k < 4; ++k) b[0][k] = tap(k);
#pragma unroll
                for (int k0 = 0; k0 < 36; k0 += 4) {
                    if (k0 + 4 < 36) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) b[(k0 >> 2 & 1) ^ 1][k] = tap(k0 + 4 + k);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, w2[k0 + k]), __builtin_bit_cast(v8bf, b[k0 >> 2 & 1][k]), acc, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // channels 32 half + 8 g + 4 hi ..: step 2 half + g / 2 of the last layer, the operand's upper 8 channels for odd g
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4i b4 = *(const v4i*)(l_b2 + 32 * half + 8 * g + 4 * hi);
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = clamp_f32(acc[4 * g + e] + __int_as_float(b4[e]), a.f_lo_d, a.f_hi_d);
                    *(uint2*)(m2 + ((g >> 1) * 64 + 32 * (g & 1)) * 16) = uint2{pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
                }
            }
            wait_all_then_barrier<0>();                                 // the residual tile has landed too
            if (it >= 0) {
                last_layer(w3);
                if constexpr (SC) xs_slot = xs_slot + 1 == RING ? 0 : xs_slot + 1;
            }
            lds_barrier();
        }
    }
}

// Shapes the kernel covers, and its tiling.
static bool bneck16_plan(const IrArgs& a, Bn16Tile& t)
{
    if (a.stride != 1 || a.pad != 1 || a.B < 1 || a.Ho != a.H || a.Wo != a.W || a.H < 1 || a.W < 1) return false;
    if ((a.Cin != 64 && a.Cin != 256) || a.Kx != a.Cin || a.Ce32 != 64 || a.Cout != 256) return false;
    if ((double)a.B * a.H * a.W * 512 >= 2147483648.0 || (a.ys && a.B > EE_ZC_MAX_B)) return false;
    t.tiles_x = (a.W + 7) / 8;
    t.tiles_y = (a.H + 7) / 8;
    const long long total = (long long)a.B * t.tiles_x * t.tiles_y;
    if (total > 0x3fffffff) return false;
    t.total = (int)total;
    const int per_xcd = (t.total + 7) / 8;
    t.nslots = per_xcd < 32 ? per_xcd : 32;                             // one workgroup per CU at most: 32 CUs per XCD
    return true;
}

bool bneck_block_bf16_supported(const IrArgs& a)
{
    Bn16Tile t;
    return bneck16_plan(a, t);
}

template <int NC, bool SC>
static hipError_t bneck16_launch(const IrArgs& a, const Bn16Tile& t, hipStream_t s)
{
    static const hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void*>(&bneck_block_bf16_kernel<NC, SC>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (granted != hipSuccess) return granted;
    EE_LAUNCH((bneck_block_bf16_kernel<NC, SC>), dim3((unsigned)(8 * t.nslots)), dim3(512), (size_t)b16_lds(NC, SC), s, a, t);
    return hipGetLastError();
}

// either a residual tensor or, from 64 channels, the convolution on the shortcut
hipError_t launch_bneck_block_bf16(const IrArgs& a, hipStream_t s)
{
    Bn16Tile t;
    if (!bneck16_plan(a, t) || (a.ws != nullptr) == (a.res != nullptr) || (a.ws && a.Cin != 64)) return hipErrorInvalidValue;
    if (a.ws) return bneck16_launch<1, true>(a, t, s);
    return a.Cin == 64 ? bneck16_launch<1, false>(a, t, s) : bneck16_launch<4, false>(a, t, s);
}

}  // namespace ee
