// First convolution and max-pool of a ResNet-style network in one launch (int8, and a bf16 form further down), for gfx950: the folded stride-2 first layer
// (4 x 4 taps over 16-channel super-pixels, 64 output channels; what conv_stream_i8_kernel runs alone) and the 3 x 3 / 2 max-pool
// with padding 1 behind it.  Layer by layer the convolution's output, the largest tensor of the network, is written once and read
// once for a quarter of its size to come out of the pool; here it only exists in LDS, a tile at a time.
//
// A workgroup (4 wavefronts) walks over tiles of 14 x 8 pooled pixels of one image.  The 29 x 17 convolution outputs under a tile's
// windows are computed in 16 strips of 32, four per wavefront, as in the streaming kernel: weights in registers for good, the activation
// operands straight from global memory, requested two strips ahead through four sets of registers (also across the pooling and into the
// next tile: a strip's operands come out of L2 in about the time two strips take), 16 matrix instructions per strip, requantisation, and the strip's pixels
// go to the tile's LDS image -- the smallest int8 value where the convolution has no output (the pool's padding: every window
// has at least one pixel that exists).  After a barrier the lanes take (pooled pixel, 16 channels) items, 448 per tile: nine 16-byte
// LDS reads, byte-wise maximum on 16-bit halves, one 16-byte store.  A seventh of the convolution is computed twice (the windows'
// overlap between tiles and the last strip's padding); results are those of the two layers bit for bit.
#include <cstring>

#include "ee_internal.hpp"
#include "igemm_device.hpp"
#include "ir_device.hpp"

namespace ee {

// ---- images read by the first layers themselves: where they are, their rows into LDS, four pixels of three channels as two super-pixels' rows ----------
// sample n is image n of x or, for requests of a stream, image ids[n] of the pool x: ids by value in front of a kernel's arguments (ImageIds), else, for more than 256, read from device-visible memory in
// front of every tile's copies, which lie a tile ahead (224 x 224, ns a request, the folded copy and the launch behind it / this, at 256 by value, 512 and 1024: 7x7 and pool 379, 362, 367 / 274, 273, 276;
// bf16 688, 686, 686 / 496, 495, 524; 3x3 206, 228, 197 / 119, 103, 95)
struct ImageArgs {
    const void* x;
    const int32_t* gather;      // ids that do not fit the arguments, else null
    int by_value;               // the table in front of the arguments holds the ids
    int H, row_bytes, pad;      // image rows, bytes of a row, padding of the convolution
};
template <int N>
struct ImageIds { int32_t id[N]; };
typedef const __attribute__((address_space(4))) int* ImageTab;          // the arguments, which begin with that table
__device__ __forceinline__ const unsigned char* image_at(const ImageArgs& im, ImageTab tab, int n)
{
    const long long id = im.by_value ? tab[n] : im.gather ? im.gather[n] : n;
    return (const unsigned char*)im.x + id * im.H * im.row_bytes;
}

// Image rows into LDS, asynchronously: 16-byte chunks of rows of RC chunks, chunk q of the tile at 16 q.  The lane's chunks first (row, byte in the row), then for a tile whose first row is y0 and whose
// rows begin at byte b0 (a multiple of 16, maybe in front of the image): zeros outside the image.  Whole copies of a wavefront.
template <int RC, int CHUNKS>
struct ImageRows {
    static constexpr int PASSES = (CHUNKS + 255) / 256, BYTES = (CHUNKS + 63) / 64 * 1024;
    int row[PASSES], col[PASSES];
    __device__ __forceinline__ explicit ImageRows(int tid)
    {
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int q = min(256 * i + tid, CHUNKS - 1);
            row[i] = q / RC;
            col[i] = 16 * (q - row[i] * RC);
        }
    }
    __device__ __forceinline__ void request(const ImageArgs& im, ImageTab tab, int n, int y0, int b0, unsigned lds, int wave, const void* zeros) const
    {
        const unsigned char* xn = image_at(im, tab, n);
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            if (256 * i + 64 * wave >= CHUNKS) break;
            const int iy = y0 + row[i], at = b0 + col[i];
            const bool ok = (unsigned)iy < (unsigned)im.H && (unsigned)at < (unsigned)im.row_bytes;
            dma16(lds + i * 4096 + wave * 1024, ok ? xn + ((long long)iy * im.row_bytes + at) : (const unsigned char*)zeros);
        }
    }
};

// Four int8 pixels of three channels, 12 contiguous bytes from byte `at` of LDS memory p, as four dwords around them shifted into place: 3 channels and a zero byte each
__device__ __forceinline__ void image_pixels(const unsigned char* p, int at, unsigned* px)
{
    const unsigned* wp = (const unsigned*)(p + (at & ~3));
    const unsigned w0 = wp[0], w1 = wp[1], w2 = wp[2], w3 = wp[3], sh = (unsigned)(at & 3) * 8;
    const unsigned d0 = __builtin_amdgcn_alignbit(w1, w0, sh), d1 = __builtin_amdgcn_alignbit(w2, w1, sh), d2 = __builtin_amdgcn_alignbit(w3, w2, sh);
    px[0] = d0 & 0x00ffffffu;
    px[1] = __builtin_amdgcn_perm(d1, d0, 0x0c050403u);                 // bytes 3, 4, 5 of the twelve
    px[2] = __builtin_amdgcn_perm(d2, d1, 0x0c040302u);                 // bytes 6, 7, 8
    px[3] = d2 >> 8;                                                    // bytes 9, 10, 11
}

typedef short v2s_r __attribute__((ext_vector_type(2)));

struct StemTile {
    int Hq, Wq;                // pooled image
    int tiles_x, tiles_y;      // tiles of 14 x 8 pooled pixels per image
    int total;                 // tiles in all
    unsigned magic_tpi, magic_tx;   // floor(2^32 / d) for the tiles of an image and of a row: fast_div
    int images;
    int pool_pad;              // conv_pool_i8_kernel: the pool's padding, 0 or 1 (the others have 1)
};

static unsigned stem_magic(int d) { return (unsigned)(0x100000000ull / (unsigned)d - (d == 1)); }

// A tile of TW x TH pooled pixels: the convolution outputs under it in strips of 32, whole ones per wavefront
template <int TW, int TH>
struct StemShape {
    static constexpr int RW = 2 * TW + 1, RH = 2 * TH + 1, RPIX = RW * RH, STRIPS = (RPIX + 31) / 32, PER = STRIPS / 4;
    static constexpr int ITEMS = 4 * TW * TH;                           // (pooled pixel, 16 channels)
    static_assert(STRIPS % 4 == 0, "whole strips per wavefront");
    static constexpr size_t lds_bytes() { return (size_t)RPIX * (64 + 16) + 256; }
};
constexpr int ST_TW = 14, ST_TH = 8;                       // 493 outputs, four strips per wavefront
// where there is a CU for every small tile: 117 outputs, one strip per wavefront.  224 x 224, with the folded copy in front: 1 sample 10.0 us in large tiles, 7.9 in small ones, 2 and 3 samples (280 and 420
// small tiles, two to a CU) 10.1 in either
constexpr int ST_SMALL_TW = 6, ST_SMALL_TH = 4;
constexpr int ST_PITCH = 64 + 16;                          // bytes per convolution output in LDS

// byte-wise signed maximum of packed dwords on 16-bit halves, three instructions per dword: the odd bytes decide a half by themselves (whatever is
// in the byte below them: the two halves are equal but for it, or the odd byte decides), the even ones moved up with zeros below them
struct StemMax { v2s_r even, odd; };
__device__ __forceinline__ StemMax stem_split(unsigned d)
{
    StemMax r;
    __builtin_memcpy(&r.odd, &d, 4);
    r.even = r.odd << 8;
    return r;
}
__device__ __forceinline__ StemMax stem_max(const StemMax& a, unsigned d)
{
    const StemMax b = stem_split(d);
    return StemMax{__builtin_elementwise_max(a.even, b.even), __builtin_elementwise_max(a.odd, b.odd)};
}
__device__ __forceinline__ unsigned stem_join(const StemMax& a)
{
    unsigned e, o;
    __builtin_memcpy(&e, &a.even, 4);
    __builtin_memcpy(&o, &a.odd, 4);
    return __builtin_amdgcn_perm(o, e, 0x07030501u);                    // bytes 1 of e, 1 of o, 3 of e, 3 of o
}

template <int TW, int TH>
__global__ __launch_bounds__(256, 2) void stem_pool_i8_kernel(ConvArgs a, void* yq, StemTile t)
{
    using Sh = StemShape<TW, TH>;
    constexpr int RW = Sh::RW, RPIX = Sh::RPIX, ITEMS = Sh::ITEMS, PER = Sh::PER;
    static_assert(PER == 4 || PER == 1, "the loop below");
    request_args<sizeof(ConvArgs) + sizeof(StemTile)>();
    constexpr int NKB = 8, NT = 2;                                      // 32-byte blocks of the reduction (4 rows x 2), blocks of 32 output channels
    extern __shared__ __attribute__((aligned(16))) unsigned char stem_lds[];
    const int tid = threadIdx.x, lane = tid & 63, p = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int* const l_bias = (int*)(stem_lds + RPIX * ST_PITCH);         // 64 biases behind the tile's image (rounding constant included)
    const int in_bias = ((const int*)a.bias)[tid & 63];
    const int tpi = t.tiles_x * t.tiles_y;
    struct Tile { int n, py0, px0; };
    auto tile_at = [&](int u) {
        const int n = (int)fast_div((unsigned)u, (unsigned)tpi, t.magic_tpi), r0 = u - n * tpi, tyi = (int)fast_div((unsigned)r0, (unsigned)t.tiles_x, t.magic_tx);
        return Tile{n, TH * tyi, TW * (r0 - tyi * t.tiles_x)};
    };
    auto load_strip = [&](const Tile& tl, int s, v4i_r* xr) {           // unconditional and in range; the folded input carries its own padding
        const unsigned char* xn = (const unsigned char*)a.x + (size_t)tl.n * a.H * a.W * 16;
        const int r = min(32 * s + p, RPIX - 1), ry = r / RW, rx = r - ry * RW;
        const int cy = min(max(2 * tl.py0 - 1 + ry, 0), a.Ho - 1), cx = min(max(2 * tl.px0 - 1 + rx, 0), a.Wo - 1);
        // the four rows and four columns under the clamped output are inside the folded image (it has three rows and columns more than
        // the convolution's output: checked by the launcher), so the eight operands lie at fixed offsets from the first
        const unsigned char* first = xn + (unsigned)((cy * a.W + cx + hi) * 16);
        const unsigned row = (unsigned)a.W * 16;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) xr[kb] = *(const v4i_r*)(first + (kb >> 1) * row + (kb & 1) * 32);
    };
    // this XCD's tiles, shared by its workgroups; the same trip count for the whole workgroup
    const int u_end = xcd_first((int)(blockIdx.x & 7) + 1, t.total), u_step = (int)(gridDim.x >> 3);
    int u = xcd_first((int)(blockIdx.x & 7), t.total) + (int)(blockIdx.x >> 3);
    // The first strips and the weights, as ready operands (read as rows, 32 lines an instruction), are requested together, in the other two kernels likewise: 64 samples 24.3 -> 22.4 us, one sample 6.2 -> 4.5; bf16, 5
    // samples 13.2 -> 9.4, 256 119.8 -> 116.0; 3x3 layer and pool, 64 samples, 40.8 -> 37.0.  Four strips: wave, wave + 4, wave + 8, wave + 12 of a tile through four operand sets; a strip's operands are requested two strips
    // before it is computed, the first two of the next tile behind this tile's last two.  (A workgroup without a tile asks for the XCD's last one.)
    v4i_r xs[PER][NKB];
    {
        const Tile t0 = tile_at(max(min(u, t.total - 1), 0));
        load_strip(t0, wave, xs[0]);
        if constexpr (PER == 4) load_strip(t0, wave + 4, xs[1]);
    }
    v4i_r wreg[NT][NKB];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) wreg[j][kb] = *(const v4i_r*)((const unsigned char*)a.wo + ((size_t)(j * (a.Kp / 32) + kb) * 64 + lane) * 16);
    __builtin_amdgcn_sched_barrier(0);
    if (tid < 64) l_bias[tid] = in_bias;
    // every weight has arrived before the loop, so that nothing inside it waits for a weight by count
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) asm volatile("" : "+v"(wreg[j][kb]));
    __syncthreads();
    const IrClamp cl = ir_clamp(a.shift, a.lo, a.hi);
    const bool relu = ir_relu(a.shift, a.lo, a.hi);
    // pooling: this lane's items (pooled pixel, channels): tid and tid + 256
    const int pch = tid & 3;
    int pty[2], ptx[2], poff[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int pp = min(tid + 256 * i, ITEMS - 1) >> 2;
        pty[i] = pp / TW; ptx[i] = pp - pty[i] * TW;
        poff[i] = ((2 * pty[i]) * RW + 2 * ptx[i]) * ST_PITCH + 16 * pch;
    }

    auto compute_strip = [&](const Tile& tl, int s, const v4i_r* xr) {
        const int r = 32 * s + p, rc = min(r, RPIX - 1), ry = rc / RW, rx = rc - ry * RW;
        const bool exists = (unsigned)(2 * tl.py0 - 1 + ry) < (unsigned)a.Ho && (unsigned)(2 * tl.px0 - 1 + rx) < (unsigned)a.Wo;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            v16i_r acc;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4i_r b4 = *(const v4i_r*)(l_bias + 32 * j + 8 * g + 4 * hi);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[4 * g + e] = b4[e];
            }
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wreg[j][kb], xr[kb], acc, 0, 0, 0);
            v4i_r o = ir_requant_pack(acc, cl, relu);
            if (!exists) o = v4i_r{(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080};
            if (r < RPIX) *(v4i_r*)(stem_lds + r * ST_PITCH + 32 * j + 16 * hi) = o;
        }
    };
    for (; u < u_end; u += u_step) {
        const Tile tl = tile_at(u);
        const bool more = u + u_step < u_end;
        const Tile tn = tile_at(more ? u + u_step : u);
        const int n = tl.n, py0 = tl.py0, px0 = tl.px0;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (PER == 4) {
            load_strip(tl, wave + 8, xs[2]);
            __builtin_amdgcn_sched_barrier(0);
            compute_strip(tl, wave, xs[0]);
            __builtin_amdgcn_sched_barrier(0);
            load_strip(tl, wave + 12, xs[3]);
            __builtin_amdgcn_sched_barrier(0);
            compute_strip(tl, wave + 4, xs[1]);
            __builtin_amdgcn_sched_barrier(0);
            load_strip(tn, wave, xs[0]);                                // past the last tile: this tile's once more (a fixed number of loads)
            __builtin_amdgcn_sched_barrier(0);
            compute_strip(tl, wave + 8, xs[2]);
            __builtin_amdgcn_sched_barrier(0);
            load_strip(tn, wave + 4, xs[1]);
            __builtin_amdgcn_sched_barrier(0);
            compute_strip(tl, wave + 12, xs[3]);
        } else {
            compute_strip(tl, wave, xs[0]);
            load_strip(tn, wave, xs[0]);
        }
        __syncthreads();                                                // the tile's convolution outputs are in LDS
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (tid + 256 * i >= ITEMS) continue;
            const unsigned char* win = stem_lds + poff[i];
            const v4i_r first = *(const v4i_r*)win;
            StemMax mx[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) mx[d] = stem_split((unsigned)first[d]);
#pragma unroll
            for (int k = 1; k < 9; ++k) {
                const v4i_r v = *(const v4i_r*)(win + ((k / 3) * RW + (k % 3)) * ST_PITCH);
#pragma unroll
                for (int d = 0; d < 4; ++d) mx[d] = stem_max(mx[d], (unsigned)v[d]);
            }
            const int py = py0 + pty[i], px = px0 + ptx[i];
            if (py < t.Hq && px < t.Wq)
                *(v4i_r*)((unsigned char*)yq + ((size_t)(n * t.Hq + py) * t.Wq + px) * 64 + 16 * pch) =
                    v4i_r{(int)stem_join(mx[0]), (int)stem_join(mx[1]), (int)stem_join(mx[2]), (int)stem_join(mx[3])};
        }
        __syncthreads();                                                // the LDS image is free for the next tile
    }
}

// ---- the same straight from the images (int8, 3 channels, rows of whole 16-byte chunks) ---------------------------------------
// Without a folded copy of the batch and the launch that makes it.  The image rows under a tile (40 pieces of 208 bytes for 14 x 8) are copied into LDS asynchronously and a tile ahead, zeros outside
// the image, folded there into super-pixels, and the strips read their operands from LDS: 16 bytes a lane and step at twice the rate of the path from the caches.  A lane folds two neighbouring
// super-pixels of a row: four pixels are 12 contiguous bytes of an image row, read as four dwords around them, shifted into place (the same shift for the whole tile) and spread to 4 bytes per
// pixel with byte permutes.  Requests of a stream: the images at ids in the pool, by value for up to 256 of them (a quarter of the arguments for 64), else read from host memory.
// Three workgroups share a CU (51 KB of LDS, 163 registers).  What bounds it: vector issue, as above, some 630 instructions per wavefront and tile, and 64 matrix instructions, which overlap in part.
// 224 x 224, us, the folded copy and the kernel above / this one, both with the time between launches: 1 sample 13.0 / 10.0 (of which the 1x1 layer behind them 4), 24 19.5 / 15.0, 64 34.2 / 26.5,
// 256 104 / 83; by itself, 64 samples 20.2 / 20.8, 256 70.1 / 63.5 (with two workgroups per CU 66.8).
template <int TW, int TH>
struct StemImageShape : StemShape<TW, TH> {
    using Base = StemShape<TW, TH>;
    static constexpr int FW = Base::RW + 3, FH = Base::RH + 3;          // folded pixels under a tile
    static constexpr int RC = (15 + 6 * FW + 15) / 16, CHUNKS = 2 * FH * RC;   // 16-byte chunks of an image row, whatever its alignment
    using Rows = ImageRows<RC, CHUNKS>;
    static constexpr int PAIRS = FH * FW / 2;
    // the tile's convolution outputs in four planes of 16 channels: neighbouring pixels are written, and the four planes of a window read, without bank conflicts
    static constexpr int PLANE = (Base::RPIX * 16 - 64 + 255) / 256 * 256 + 64, FOLD = 4 * PLANE + 256;
    static constexpr size_t lds_bytes() { return FOLD + FW * FH * 16 + Rows::BYTES; }
};

template <int TW, int TH>
__device__ __forceinline__ void stem_image(const ConvArgs& a, void* yq, const StemTile& t, const ImageArgs& im, ImageTab tab)
{
    using Sh = StemImageShape<TW, TH>;
    constexpr int RW = Sh::RW, RPIX = Sh::RPIX, ITEMS = Sh::ITEMS, PER = Sh::PER, FW = Sh::FW, RC = Sh::RC;
    constexpr int NKB = 8, NT = 2, NST = (ITEMS + 255) / 256;
    constexpr unsigned NOWHERE = 0x80000000u;                           // an offset past the output: the store is dropped
    extern __shared__ __attribute__((aligned(16))) unsigned char stem_lds[];
    const int tid = threadIdx.x, lane = tid & 63, p = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int* const l_bias = (int*)(stem_lds + 4 * Sh::PLANE);               // 64 biases
    unsigned char* const l_fold = stem_lds + Sh::FOLD;
    const int in_bias = ((const int*)a.bias)[tid & 63];
    unsigned char* const l_raw = l_fold + FW * Sh::FH * 16;
    const unsigned raw0 = lds_addr(l_raw);
    const int tpi = t.tiles_x * t.tiles_y;
    struct Tile { int n, py0, px0; };
    auto tile_at = [&](int u) {
        const int n = (int)fast_div((unsigned)u, (unsigned)tpi, t.magic_tpi), r0 = u - n * tpi, tyi = (int)fast_div((unsigned)r0, (unsigned)t.tiles_x, t.magic_tx);
        return Tile{n, TH * tyi, TW * (r0 - tyi * t.tiles_x)};
    };
    // folded pixel (fy, fx) of a tile is image rows 2 (2 py0 - 1 + fy) - pad and the next, columns likewise; its row's first byte may lie in front of the image
    auto first_byte = [&](const Tile& tl) { return 3 * (4 * tl.px0 - 2 - im.pad); };
    const typename Sh::Rows rows(tid);
    auto stage = [&](const Tile& tl) { rows.request(im, tab, tl.n, 4 * tl.py0 - 2 - im.pad, first_byte(tl) & ~15, raw0, wave, a.zeros); };
    const int u_end = xcd_first((int)(blockIdx.x & 7) + 1, t.total), u_step = (int)(gridDim.x >> 3);
    int u = xcd_first((int)(blockIdx.x & 7), t.total) + (int)(blockIdx.x >> 3);
    Tile tl = tile_at(max(min(u, t.total - 1), 0));                     // (a workgroup without a tile asks for the XCD's last one)
    stage(tl);
    v4i_r wreg[NT][NKB];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) wreg[j][kb] = *(const v4i_r*)((const unsigned char*)a.wo + ((size_t)(j * (a.Kp / 32) + kb) * 64 + lane) * 16);
    __builtin_amdgcn_sched_barrier(0);
    if (tid < 64) l_bias[tid] = in_bias;
    const IrClamp cl = ir_clamp(a.shift, a.lo, a.hi);
    const bool relu = ir_relu(a.shift, a.lo, a.hi);
    const int pch = tid & 3;
    int pty[NST], ptx[NST], poff[NST];
#pragma unroll
    for (int i = 0; i < NST; ++i) {
        const int pp = min(tid + 256 * i, ITEMS - 1) >> 2;
        pty[i] = pp / TW; ptx[i] = pp - pty[i] * TW;
        poff[i] = ((2 * pty[i]) * RW + 2 * ptx[i]) * 16 + pch * Sh::PLANE;
    }
    int spy[PER], spx[PER];                                             // this lane's output of its wavefront's strips
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int r = min(32 * (wave + 4 * k) + p, RPIX - 1);
        spy[k] = r / RW; spx[k] = r - spy[k] * RW;
    }
    const auto y_buf = __builtin_amdgcn_make_buffer_rsrc(yq, (short)0, t.images * t.Hq * t.Wq * 64, 0x00020000);
    auto read_strip = [&](int k, v4i_r* xr) {
        const unsigned char* first = l_fold + (spy[k] * FW + spx[k] + hi) * 16;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) xr[kb] = *(const v4i_r*)(first + (kb >> 1) * FW * 16 + (kb & 1) * 32);
    };
    auto compute_strip = [&](int k, const v4i_r* xr) {
        const bool exists = (unsigned)(2 * tl.py0 - 1 + spy[k]) < (unsigned)a.Ho && (unsigned)(2 * tl.px0 - 1 + spx[k]) < (unsigned)a.Wo;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            v16i_r acc;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4i_r b4 = *(const v4i_r*)(l_bias + 32 * j + 8 * g + 4 * hi);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[4 * g + e] = b4[e];
            }
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wreg[j][kb], xr[kb], acc, 0, 0, 0);
            v4i_r o = ir_requant_pack(acc, cl, relu);
            if (!exists) o = v4i_r{(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080};
            *(v4i_r*)(stem_lds + (2 * j + hi) * Sh::PLANE + (spy[k] * RW + spx[k]) * 16) = o;       // (lanes past the last output hold and write the last one)
        }
    };
    // every weight has arrived before the loop, so that nothing inside it waits for a weight by count
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) asm volatile("" : "+v"(wreg[j][kb]));
    wait_all_then_barrier<0>();
    for (; u < u_end; u += u_step) {
        {
            const int skew = first_byte(tl) & 15;
#pragma unroll
            for (int i = 0; i < (Sh::PAIRS + 255) / 256; ++i) {
                if (256 * i + 64 * wave >= Sh::PAIRS) break;
                const int item = min(256 * i + tid, Sh::PAIRS - 1), fr = item / (FW / 2), pr = item - fr * (FW / 2);
                unsigned px[2][4];                                      // [image row of the pair][pixel]
#pragma unroll
                for (int dy = 0; dy < 2; ++dy) image_pixels(l_raw, (2 * fr + dy) * RC * 16 + skew + 12 * pr, px[dy]);
                v4i_r* q = (v4i_r*)(l_fold + (fr * FW + 2 * pr) * 16);
                q[0] = v4i_r{(int)px[0][0], (int)px[0][1], (int)px[1][0], (int)px[1][1]};
                q[1] = v4i_r{(int)px[0][2], (int)px[0][3], (int)px[1][2], (int)px[1][3]};
            }
        }
        lds_barrier();                                                  // the tile is folded, its image rows are free
        const bool more = u + u_step < u_end;
        const Tile tn = tile_at(more ? u + u_step : u);
        stage(tn);                                                      // past the last tile: this tile's once more
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            v4i_r xs[NKB];
            read_strip(k, xs);
            compute_strip(k, xs);
            __builtin_amdgcn_sched_barrier(0);
        }
        lds_barrier();                                                  // the tile's convolution outputs are in LDS
#pragma unroll
        for (int i = 0; i < NST; ++i) {
            const unsigned char* win = stem_lds + poff[i];
            const v4i_r first = *(const v4i_r*)win;
            StemMax mx[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) mx[d] = stem_split((unsigned)first[d]);
#pragma unroll
            for (int k = 1; k < 9; ++k) {
                const v4i_r v = *(const v4i_r*)(win + ((k / 3) * RW + (k % 3)) * 16);
#pragma unroll
                for (int d = 0; d < 4; ++d) mx[d] = stem_max(mx[d], (unsigned)v[d]);
            }
            const int py = tl.py0 + pty[i], px = tl.px0 + ptx[i];
            const bool ok = tid + 256 * i < ITEMS && py < t.Hq && px < t.Wq;
            const unsigned at = ok ? (unsigned)(((tl.n * t.Hq + py) * t.Wq + px) * 64 + 16 * pch) : NOWHERE;
            __builtin_amdgcn_raw_buffer_store_b128(v4i_r{(int)stem_join(mx[0]), (int)stem_join(mx[1]), (int)stem_join(mx[2]), (int)stem_join(mx[3])}, y_buf, at, 0, 0);
        }
        tl = tn;
        wait_all_then_barrier<NST>();                                   // the next tile's image rows are there (NST stores behind them may not be), the tile's convolution outputs are free
    }
}
template <int TW, int TH>
__global__ __launch_bounds__(256, 3) void stem_pool_i8_kernel(ImageIds<64>, ConvArgs a, void* yq, StemTile t, ImageArgs im)
{
    request_args<sizeof(ImageIds<64>) + sizeof(ConvArgs) + sizeof(StemTile) + sizeof(ImageArgs)>();
    stem_image<TW, TH>(a, yq, t, im, (ImageTab)__builtin_amdgcn_kernarg_segment_ptr());
}
template <int TW, int TH>
__global__ __launch_bounds__(256, 3) void stem_pool_i8_kernel(ImageIds<256>, ConvArgs a, void* yq, StemTile t, ImageArgs im)
{
    stem_image<TW, TH>(a, yq, t, im, (ImageTab)__builtin_amdgcn_kernarg_segment_ptr());
}

// The bf16 form.  A super-pixel has 32 bytes and the reduction sixteen steps of one tap each, so a strip's operands are twice the bytes and
// its matrix instructions twice as many; read from global memory per strip they would be eight times the folded image (1.9 GB for 256
// samples through the 64 bytes per clock of the CU's vector memory path: 50 us by themselves).  Here the folded pixels under a tile are copied
// to LDS once, asynchronously and a tile ahead, and a strip's operands are LDS reads (32 neighbouring pixels are 1 KiB in a row: no bank
// conflicts).  Tiles of 7 x 8 pooled pixels: the 15 x 17 convolution outputs under them are 255, eight strips of 32 with one lane to
// spare, two per wavefront, both blocks of 32 output channels per operand; 62 KB of LDS let two workgroups share a CU, so that one
// pools while the other multiplies.  Weights stay in registers (128).
// Sums, bias, clamp and rounding are those of the staged kernel, step by step; a clamp at or above zero (ReLU) is what the rule asks for:
// bf16 values >= 0 order like 16-bit integers, the pool is packed integer maxima, and 0 stands where the convolution has no output.
// 256 samples of 224 x 224, with the folded copy in front: 374 us as two launches behind it (252 and 121 us by themselves; the tensor
// between them, 411 MB, written once and read two and a quarter times), 173 fused.  What bounds it: matrix instructions 49 us, vector issue (epilogue and pool)
// about as much, LDS operand reads 25 us, 211 MB of HBM traffic 38 us, shared out over two workgroups per CU.
constexpr int SB_TW = 7, SB_TH = 8;
constexpr int SB_RW = 2 * SB_TW + 1, SB_RH = 2 * SB_TH + 1, SB_RPIX = SB_RW * SB_RH;      // 15 x 17 convolution outputs
constexpr int SB_SW = SB_RW + 3, SB_SH = SB_RH + 3, SB_CHUNKS = 2 * SB_SW * SB_SH;        // 18 x 20 folded pixels of two 16-byte chunks
constexpr int SB_PASSES = (SB_CHUNKS + 255) / 256, SB_STAGE = SB_PASSES * 4096;           // whole copy passes of the workgroup
constexpr int SB_PITCH = 128 + 16;                                                        // bytes per convolution output in LDS
constexpr int SB_LDS = 2 * SB_STAGE + SB_RPIX * SB_PITCH + 256;
constexpr int SB_ITEMS = 8 * SB_TW * SB_TH;                                               // (pooled pixel, 8 channels)
static_assert((SB_RPIX + 31) / 32 == 8, "two strips per wavefront");
static_assert(2 * SB_LDS <= 160 * 1024, "two workgroups per CU");

__global__ __launch_bounds__(256, 2) void stem_pool_bf16_kernel(ConvArgs a, void* yq, StemTile t)
{
    request_args<sizeof(ConvArgs) + sizeof(StemTile)>();
    constexpr int NK = 16;                                              // taps = reduction steps of 16 channels
    extern __shared__ __attribute__((aligned(16))) unsigned char stem_lds[];
    const int tid = threadIdx.x, lane = tid & 63, p = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned lds0 = lds_addr(stem_lds);
    unsigned char* const l_conv = stem_lds + 2 * SB_STAGE;
    float* const l_bias = (float*)(l_conv + SB_RPIX * SB_PITCH);
    const float in_bias = ((const float*)a.bias)[tid & 63];
    v4i wreg[2][NK];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int k = 0; k < NK; ++k) wreg[j][k] = *(const v4i*)((const unsigned char*)a.wo + ((size_t)(j * (a.Kp / 16) + k) * 64 + lane) * 16);
    __builtin_amdgcn_sched_barrier(0);
    // this lane's chunks of a staged tile: row | column << 8 of the folded pixel, half of it
    int spos[SB_PASSES];
#pragma unroll
    for (int i = 0; i < SB_PASSES; ++i) {
        const int q = min(256 * i + tid, SB_CHUNKS - 1), row = q / (2 * SB_SW), c = q - row * 2 * SB_SW;
        spos[i] = row | (c >> 1) << 8 | (c & 1) << 16;
    }
    // pooling: this lane's items (pooled pixel, channels): tid and tid + 256
    int pty[2], ptx[2], poff[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int pp = min(tid + 256 * i, SB_ITEMS - 1) >> 3;
        pty[i] = pp / SB_TW; ptx[i] = pp - pty[i] * SB_TW;
        poff[i] = (2 * pty[i] * SB_RW + 2 * ptx[i]) * SB_PITCH + 16 * (tid & 7);
    }
    const int tpi = t.tiles_x * t.tiles_y;
    struct Tile { int n, py0, px0; };
    auto tile_at = [&](int u) {
        const int n = (int)fast_div((unsigned)u, (unsigned)tpi, t.magic_tpi), r0 = u - n * tpi, tyi = (int)fast_div((unsigned)r0, (unsigned)t.tiles_x, t.magic_tx);
        return Tile{n, SB_TH * tyi, SB_TW * (r0 - tyi * t.tiles_x)};
    };
    auto stage = [&](const Tile& tl, int buf) {                         // asynchronous; clamped pixels are only ever read by outputs that do not exist
        const unsigned char* xn = (const unsigned char*)a.x + (size_t)tl.n * a.H * a.W * 32;
#pragma unroll
        for (int i = 0; i < SB_PASSES; ++i) {
            const int cy = min(max(2 * tl.py0 - 1 + (spos[i] & 255), 0), a.H - 1), cx = min(max(2 * tl.px0 - 1 + ((spos[i] >> 8) & 255), 0), a.W - 1);
            dma16(lds0 + buf * SB_STAGE + i * 4096 + wave * 1024, xn + (unsigned)((cy * a.W + cx) * 32 + 16 * (spos[i] >> 16)));
        }
    };
    // this XCD's tiles, shared by its workgroups; the same trip count for the whole workgroup
    const int u_end = xcd_first((int)(blockIdx.x & 7) + 1, t.total), u_step = (int)(gridDim.x >> 3);
    int u = xcd_first((int)(blockIdx.x & 7), t.total) + (int)(blockIdx.x >> 3), buf = 0;
    Tile tl = tile_at(u);
    if (u < u_end) stage(tl, 0);                                        // on its way with the weights
    if (tid < 64) l_bias[tid] = in_bias;
    // every weight has arrived before the loop, so that nothing inside it waits for a weight by count
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int k = 0; k < NK; ++k) asm volatile("" : "+v"(wreg[j][k]));
    for (; u < u_end; u += u_step, buf ^= 1) {
        wait_all_then_barrier<0>();                                     // the tile is staged, the pooling of the one before has read its convolution outputs
        const Tile tn = tile_at(u + u_step);
        if (u + u_step < u_end) stage(tn, buf ^ 1);
        const unsigned char* xl = stem_lds + buf * SB_STAGE + 16 * hi;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int r = 32 * (wave + 4 * s) + p, rc = min(r, SB_RPIX - 1), ry = rc / SB_RW, rx = rc - ry * SB_RW;
            const bool exists = (unsigned)(2 * tl.py0 - 1 + ry) < (unsigned)a.Ho && (unsigned)(2 * tl.px0 - 1 + rx) < (unsigned)a.Wo;
            const unsigned char* px = xl + (ry * SB_SW + rx) * 32;
            v16f acc[2];
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[0][i] = acc[1][i] = 0.f;
            // the operands in batches of four through two sets of registers, a batch ahead of its matrix instructions
            v4i xs[2][4];
            auto read = [&](int k0, v4i* x) {
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = *(const v4i*)(px + ((k0 >> 2) * SB_SW + k) * 32);
            };
            read(0, xs[0]);
#pragma unroll
            for (int k0 = 0; k0 < NK; k0 += 4) {
                if (k0 + 4 < NK) read(k0 + 4, xs[(k0 >> 2 & 1) ^ 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, wreg[j][k0 + k]), __builtin_bit_cast(v8bf, xs[k0 >> 2 & 1][k]), acc[j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            unsigned char* cell = l_conv + rc * SB_PITCH + 8 * hi;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4i b4 = *(const v4i*)(l_bias + 32 * j + 8 * g + 4 * hi);
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = clamp_f32(acc[j][4 * g + e] + __int_as_float(b4[e]), a.f_lo, a.f_hi);
                    uint2 o = {pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
                    if (!exists) o = uint2{0u, 0u};
                    if (r < SB_RPIX) *(uint2*)(cell + 64 * j + 16 * g) = o;
                }
        }
        lds_barrier();                                                  // the tile's convolution outputs are in LDS
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (tid + 256 * i >= SB_ITEMS) continue;
            typedef short v8s __attribute__((ext_vector_type(8)));
            const unsigned char* win = l_conv + poff[i];
            v8s mx = *(const v8s*)win;
#pragma unroll
            for (int k = 1; k < 9; ++k) mx = __builtin_elementwise_max(mx, *(const v8s*)(win + ((k / 3) * SB_RW + (k % 3)) * SB_PITCH));
            const int py = tl.py0 + pty[i], px = tl.px0 + ptx[i];
            if (py < t.Hq && px < t.Wq)
                *(v8s*)((unsigned char*)yq + ((size_t)(tl.n * t.Hq + py) * t.Wq + px) * 128 + 16 * (tid & 7)) = mx;
        }
        tl = tn;
    }
}

// The bf16 form straight from the images, as the int8 one: half a super-pixel, two pixels of an image row, is 12 contiguous bytes.  The biases are read behind a strip's last operands, all four
// ahead of their use (each waited for by itself they took some 1000 clocks of a strip).  224 x 224, us, the folded copy and the kernel above / this one, both with the time between launches and the 1x1
// layer behind: 1 sample 14.2 / 10.3, 5 16.9 / 11.3, 64 54.5 / 43.7, 256 192 / 143; by itself, 256 samples 112.6 / 117.2, and the copy was 52.
constexpr int SI_RC = (15 + 12 * SB_SW + 15) / 16, SI_FOLD = SB_CHUNKS * 16;                // 16-byte chunks of an image row under a tile, whatever its alignment
using SiRows = ImageRows<SI_RC, 2 * SB_SH * SI_RC>;
constexpr int SI_LDS = SI_FOLD + SiRows::BYTES + SB_RPIX * SB_PITCH + 256;
static_assert(2 * SI_LDS <= 160 * 1024, "two workgroups per CU");

__device__ __forceinline__ void stem_image_bf16(const ConvArgs& a, void* yq, const StemTile& t, const ImageArgs& im, ImageTab tab)
{
    constexpr int NK = 16;                                              // taps = reduction steps of 16 channels
    extern __shared__ __attribute__((aligned(16))) unsigned char stem_lds[];
    const int tid = threadIdx.x, lane = tid & 63, p = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned char* const l_fold = stem_lds;
    unsigned char* const l_raw = stem_lds + SI_FOLD;
    unsigned char* const l_conv = l_raw + SiRows::BYTES;
    constexpr unsigned NOWHERE = 0x80000000u;                           // an offset past the output: the store is dropped
    float* const l_bias = (float*)(l_conv + SB_RPIX * SB_PITCH);
    const float in_bias = ((const float*)a.bias)[tid & 63];
    v4i wreg[2][NK];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int k = 0; k < NK; ++k) wreg[j][k] = *(const v4i*)((const unsigned char*)a.wo + ((size_t)(j * (a.Kp / 16) + k) * 64 + lane) * 16);
    __builtin_amdgcn_sched_barrier(0);
    const SiRows rows(tid);
    // pooling: this lane's items (pooled pixel, channels): tid and tid + 256
    int pty[2], ptx[2], poff[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int pp = min(tid + 256 * i, SB_ITEMS - 1) >> 3;
        pty[i] = pp / SB_TW; ptx[i] = pp - pty[i] * SB_TW;
        poff[i] = (2 * pty[i] * SB_RW + 2 * ptx[i]) * SB_PITCH + 16 * (tid & 7);
    }
    const int tpi = t.tiles_x * t.tiles_y;
    struct Tile { int n, py0, px0; };
    auto tile_at = [&](int u) {
        const int n = (int)fast_div((unsigned)u, (unsigned)tpi, t.magic_tpi), r0 = u - n * tpi, tyi = (int)fast_div((unsigned)r0, (unsigned)t.tiles_x, t.magic_tx);
        return Tile{n, SB_TH * tyi, SB_TW * (r0 - tyi * t.tiles_x)};
    };
    // folded pixel (fy, fx) of a tile is image rows 2 (2 py0 - 1 + fy) - pad and the next, columns likewise; its row's first byte may lie in front of the image
    auto first_byte = [&](const Tile& tl) { return 6 * (4 * tl.px0 - 2 - im.pad); };
    const unsigned raw0 = lds_addr(l_raw);
    auto stage = [&](const Tile& tl) { rows.request(im, tab, tl.n, 4 * tl.py0 - 2 - im.pad, first_byte(tl) & ~15, raw0, wave, a.zeros); };
    const auto y_buf = __builtin_amdgcn_make_buffer_rsrc(yq, (short)0, t.images * t.Hq * t.Wq * 128, 0x00020000);
    // this XCD's tiles, shared by its workgroups; the same trip count for the whole workgroup
    const int u_end = xcd_first((int)(blockIdx.x & 7) + 1, t.total), u_step = (int)(gridDim.x >> 3);
    int u = xcd_first((int)(blockIdx.x & 7), t.total) + (int)(blockIdx.x >> 3);
    Tile tl = tile_at(max(min(u, t.total - 1), 0));                     // (a workgroup without a tile asks for the XCD's last one)
    stage(tl);                                                          // on its way with the weights
    if (tid < 64) l_bias[tid] = in_bias;
    // every weight has arrived before the loop, so that nothing inside it waits for a weight by count
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int k = 0; k < NK; ++k) asm volatile("" : "+v"(wreg[j][k]));
    wait_all_then_barrier<0>();
    for (; u < u_end; u += u_step) {
        {                                                               // a 16-byte half of a super-pixel (an image row's two pixels) per item
            const int skew = first_byte(tl) & 15;
            const unsigned sh = (unsigned)(skew & 3) * 8;
#pragma unroll
            for (int i = 0; i < (SB_CHUNKS + 255) / 256; ++i) {
                if (256 * i + 64 * wave >= SB_CHUNKS) break;
                const int item = min(256 * i + tid, SB_CHUNKS - 1), fy = item / (2 * SB_SW), c = item - fy * 2 * SB_SW;
                const unsigned* wp = (const unsigned*)(l_raw + (2 * fy + (c & 1)) * SI_RC * 16 + (skew & ~3) + 12 * (c >> 1));
                const unsigned w0 = wp[0], w1 = wp[1], w2 = wp[2], w3 = wp[3];
                const unsigned d0 = __builtin_amdgcn_alignbit(w1, w0, sh), d1 = __builtin_amdgcn_alignbit(w2, w1, sh), d2 = __builtin_amdgcn_alignbit(w3, w2, sh);
                *(v4i*)(l_fold + item * 16) = v4i{(int)d0, (int)(d1 & 0xffffu), (int)__builtin_amdgcn_alignbit(d2, d1, 16), (int)(d2 >> 16)};
            }
        }
        lds_barrier();                                                  // the tile is folded, its image rows are free
        const bool more = u + u_step < u_end;
        const Tile tn = tile_at(more ? u + u_step : u);
        stage(tn);                                                      // past the last tile: this tile's once more
        const unsigned char* xl = l_fold + 16 * hi;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int r = 32 * (wave + 4 * s) + p, rc = min(r, SB_RPIX - 1), ry = rc / SB_RW, rx = rc - ry * SB_RW;
            const bool exists = (unsigned)(2 * tl.py0 - 1 + ry) < (unsigned)a.Ho && (unsigned)(2 * tl.px0 - 1 + rx) < (unsigned)a.Wo;
            const unsigned char* px = xl + (ry * SB_SW + rx) * 32;
            v16f acc[2];
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[0][i] = acc[1][i] = 0.f;
            // the operands in batches of four through two sets of registers, a batch ahead of its matrix instructions
            v4i xs[2][4];
            auto read = [&](int k0, v4i* x) {
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = *(const v4i*)(px + ((k0 >> 2) * SB_SW + k) * 32);
            };
            auto read_bias = [&](int j, v4i* b4) {
#pragma unroll
                for (int g = 0; g < 4; ++g) b4[g] = *(const v4i*)(l_bias + 32 * j + 8 * g + 4 * hi);
            };
            v4i bias[2][4];
            read(0, xs[0]);
#pragma unroll
            for (int k0 = 0; k0 < NK; k0 += 4) {
                if (k0 + 4 < NK) read(k0 + 4, xs[(k0 >> 2 & 1) ^ 1]);
                else read_bias(0, bias[0]);                             // behind the last operands, in the registers they leave
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, wreg[j][k0 + k]), __builtin_bit_cast(v8bf, xs[k0 >> 2 & 1][k]), acc[j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            read_bias(1, bias[1]);
            __builtin_amdgcn_sched_barrier(0);
            unsigned char* cell = l_conv + rc * SB_PITCH + 8 * hi;      // (the lane past the last output holds and writes the last one)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = clamp_f32(acc[j][4 * g + e] + __int_as_float(bias[j][g][e]), a.f_lo, a.f_hi);
                    uint2 o = {pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
                    if (!exists) o = uint2{0u, 0u};
                    *(uint2*)(cell + 64 * j + 16 * g) = o;
                }
        }
        lds_barrier();                                                  // the tile's convolution outputs are in LDS
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            typedef short v8s __attribute__((ext_vector_type(8)));
            const unsigned char* win = l_conv + poff[i];
            v8s mx = *(const v8s*)win;
#pragma unroll
            for (int k = 1; k < 9; ++k) mx = __builtin_elementwise_max(mx, *(const v8s*)(win + ((k / 3) * SB_RW + (k % 3)) * SB_PITCH));
            const int py = tl.py0 + pty[i], px = tl.px0 + ptx[i];
            const bool ok = tid + 256 * i < SB_ITEMS && py < t.Hq && px < t.Wq;
            const unsigned at = ok ? (unsigned)(((tl.n * t.Hq + py) * t.Wq + px) * 128 + 16 * (tid & 7)) : NOWHERE;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, mx), y_buf, at, 0, 0);
        }
        tl = tn;
        wait_all_then_barrier<2>();                                     // the next tile's image rows are there (two stores behind them may not be), the tile's convolution outputs are free
    }
}
__global__ __launch_bounds__(256, 2) void stem_pool_bf16_kernel(ImageIds<64>, ConvArgs a, void* yq, StemTile t, ImageArgs im)
{
    request_args<sizeof(ImageIds<64>) + sizeof(ConvArgs) + sizeof(StemTile) + sizeof(ImageArgs)>();
    stem_image_bf16(a, yq, t, im, (ImageTab)__builtin_amdgcn_kernarg_segment_ptr());
}
__global__ __launch_bounds__(256, 2) void stem_pool_bf16_kernel(ImageIds<256>, ConvArgs a, void* yq, StemTile t, ImageArgs im)
{
    stem_image_bf16(a, yq, t, im, (ImageTab)__builtin_amdgcn_kernarg_segment_ptr());
}

// ---- a 3x3 convolution over 32 channels and the 3x3 / 2 max-pool behind it (int8, 64 output channels) ------------------------
// What Inception-style stems have behind their first layers.  A pixel has 32 bytes, one reduction step per tap: the bf16 kernel's tile and staging with
// nine taps, and zeros staged outside the image where the convolution pads; operands, requantisation and pool as in the first-layer kernel.
// 64 samples of 149 x 149: 52.2 + 19.9 us as two launches (91 MB written and read in between), 42.1 here.  What bounds it: vector issue, some 700
// instructions per wavefront and tile (requantisation, pool, operand addresses) against 36 matrix instructions.
constexpr int CP_SW = SB_RW + 2, CP_SH = SB_RH + 2, CP_CHUNKS = 2 * CP_SW * CP_SH;        // 17 x 19 input pixels of two 16-byte chunks
constexpr int CP_PASSES = (CP_CHUNKS + 255) / 256, CP_STAGE = CP_PASSES * 4096;
constexpr int CP_PITCH = 64 + 16;
constexpr int CP_LDS = 2 * CP_STAGE + SB_RPIX * CP_PITCH + 256;
constexpr int CP_ITEMS = 4 * SB_TW * SB_TH;                                               // (pooled pixel, 16 channels)
static_assert(CP_ITEMS <= 256, "one item per lane");

__global__ __launch_bounds__(256, 3) void conv_pool_i8_kernel(ConvArgs a, void* yq, StemTile t)
{
    request_args<sizeof(ConvArgs) + sizeof(StemTile)>();
    constexpr int NK = 9;
    extern __shared__ __attribute__((aligned(16))) unsigned char stem_lds[];
    const int tid = threadIdx.x, lane = tid & 63, p = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned lds0 = lds_addr(stem_lds);
    unsigned char* const l_conv = stem_lds + 2 * CP_STAGE;
    int* const l_bias = (int*)(l_conv + SB_RPIX * CP_PITCH);
    const int in_bias = ((const int*)a.bias)[tid & 63];
    v4i wreg[2][NK];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int k = 0; k < NK; ++k) wreg[j][k] = *(const v4i*)((const unsigned char*)a.wo + ((size_t)(j * (a.Kp / 32) + k) * 64 + lane) * 16);
    __builtin_amdgcn_sched_barrier(0);
    // this lane's chunks of a staged tile: row | column << 8 of the input pixel, half of it
    int spos[CP_PASSES];
#pragma unroll
    for (int i = 0; i < CP_PASSES; ++i) {
        const int q = min(256 * i + tid, CP_CHUNKS - 1), row = q / (2 * CP_SW), c = q - row * 2 * CP_SW;
        spos[i] = row | (c >> 1) << 8 | (c & 1) << 16;
    }
    const int pp = min(tid, CP_ITEMS - 1) >> 2, pty = pp / SB_TW, ptx = pp - pty * SB_TW;      // pooling: this lane's pixel
    const unsigned char* const win = l_conv + (2 * pty * SB_RW + 2 * ptx) * CP_PITCH + 16 * (tid & 3);
    const int tpi = t.tiles_x * t.tiles_y;
    struct Tile { int n, py0, px0; };
    auto tile_at = [&](int u) {
        const int n = (int)fast_div((unsigned)u, (unsigned)tpi, t.magic_tpi), r0 = u - n * tpi, tyi = (int)fast_div((unsigned)r0, (unsigned)t.tiles_x, t.magic_tx);
        return Tile{n, SB_TH * tyi, SB_TW * (r0 - tyi * t.tiles_x)};
    };
    auto stage = [&](const Tile& tl, int buf) {                         // asynchronous; zeros outside the image
        const unsigned char* xn = (const unsigned char*)a.x + (size_t)tl.n * a.H * a.W * 32;
#pragma unroll
        for (int i = 0; i < CP_PASSES; ++i) {
            const int iy = 2 * tl.py0 - t.pool_pad - a.pad + (spos[i] & 255), ix = 2 * tl.px0 - t.pool_pad - a.pad + ((spos[i] >> 8) & 255);
            const bool ok = (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
            dma16(lds0 + buf * CP_STAGE + i * 4096 + wave * 1024, ok ? xn + (unsigned)((iy * a.W + ix) * 32 + 16 * (spos[i] >> 16)) : (const unsigned char*)a.zeros);
        }
    };
    const IrClamp cl = ir_clamp(a.shift, a.lo, a.hi);
    // this XCD's tiles, shared by its workgroups; the same trip count for the whole workgroup
    const int u_end = xcd_first((int)(blockIdx.x & 7) + 1, t.total), u_step = (int)(gridDim.x >> 3);
    int u = xcd_first((int)(blockIdx.x & 7), t.total) + (int)(blockIdx.x >> 3), buf = 0;
    Tile tl = tile_at(u);
    if (u < u_end) stage(tl, 0);                                        // on its way with the weights
    if (tid < 64) l_bias[tid] = in_bias;
    // every weight has arrived before the loop, so that nothing inside it waits for a weight by count
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int k = 0; k < NK; ++k) asm volatile("" : "+v"(wreg[j][k]));
    for (; u < u_end; u += u_step, buf ^= 1) {
        wait_all_then_barrier<0>();                                     // the tile is staged, the pooling of the one before has read its convolution outputs
        const Tile tn = tile_at(u + u_step);
        if (u + u_step < u_end) stage(tn, buf ^ 1);
        const unsigned char* xl = stem_lds + buf * CP_STAGE + 16 * hi;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int r = 32 * (wave + 4 * s) + p, rc = min(r, SB_RPIX - 1), ry = rc / SB_RW, rx = rc - ry * SB_RW;
            const bool exists = (unsigned)(2 * tl.py0 - t.pool_pad + ry) < (unsigned)a.Ho && (unsigned)(2 * tl.px0 - t.pool_pad + rx) < (unsigned)a.Wo;
            const unsigned char* px = xl + (ry * CP_SW + rx) * 32;
            v4i xs[2][3];                                               // a row of taps at a time, the next one on its way
            auto read = [&](int row, v4i* x) {
#pragma unroll
                for (int k = 0; k < 3; ++k) x[k] = *(const v4i*)(px + (row * CP_SW + k) * 32);
            };
            read(0, xs[0]);
            v16i acc[2];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4i b4 = *(const v4i*)(l_bias + 32 * j + 8 * g + 4 * hi);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[j][4 * g + e] = b4[e];
                }
#pragma unroll
            for (int row = 0; row < 3; ++row) {
                if (row < 2) read(row + 1, xs[(row + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wreg[j][3 * row + k], xs[row & 1][k], acc[j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                v4i o = ir_requant_any(acc[j], cl);
                if (!exists) o = v4i{(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080};
                if (r < SB_RPIX) *(v4i*)(l_conv + r * CP_PITCH + 32 * j + 16 * hi) = o;
            }
        }
        lds_barrier();                                                  // the tile's convolution outputs are in LDS
        if (tid < CP_ITEMS) {
            const v4i first = *(const v4i*)win;
            StemMax mx[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) mx[d] = stem_split((unsigned)first[d]);
#pragma unroll
            for (int k = 1; k < 9; ++k) {
                const v4i v = *(const v4i*)(win + ((k / 3) * SB_RW + (k % 3)) * CP_PITCH);
#pragma unroll
                for (int d = 0; d < 4; ++d) mx[d] = stem_max(mx[d], (unsigned)v[d]);
            }
            const int py = tl.py0 + pty, px = tl.px0 + ptx;
            if (py < t.Hq && px < t.Wq)
                *(v4i*)((unsigned char*)yq + ((size_t)(tl.n * t.Hq + py) * t.Wq + px) * 64 + 16 * (tid & 3)) =
                    v4i{(int)stem_join(mx[0]), (int)stem_join(mx[1]), (int)stem_join(mx[2]), (int)stem_join(mx[3])};
        }
        tl = tn;
    }
}

bool conv_pool_supported(const ConvArgs& a, int es, int Hq, int Wq, int pool_pad)
{
    if (es != 1 || a.mode != 0 || a.res != nullptr || a.xs || a.M <= 0 || a.Ci != 32 || a.kh != 3 || a.kw != 3 || a.stride != 1) return false;
    if (a.pad != a.pad_w || a.pad < 0 || a.pad > 1 || pool_pad < 0 || pool_pad > 1 || a.Ho != a.H + 2 * a.pad - 2 || a.Wo != a.W + 2 * a.pad - 2) return false;
    if (a.Co != 64 || a.ldc != 64 || a.c_off != 0 || a.Kp < 288 || a.Ho + 2 * pool_pad < 3 || a.Wo + 2 * pool_pad < 3) return false;
    if (Hq != (a.Ho + 2 * pool_pad - 3) / 2 + 1 || Wq != (a.Wo + 2 * pool_pad - 3) / 2 + 1) return false;
    return (double)(a.M / (a.Ho * a.Wo)) * a.H * a.W * 32 < 2147483648.0;
}

hipError_t launch_conv_pool(const ConvArgs& a, void* yq, int Hq, int Wq, int pool_pad, hipStream_t s)
{
    if (!conv_pool_supported(a, 1, Hq, Wq, pool_pad)) return hipErrorInvalidValue;
    StemTile t;
    t.Hq = Hq; t.Wq = Wq; t.images = a.M / (a.Ho * a.Wo); t.pool_pad = pool_pad;
    t.tiles_x = (Wq + SB_TW - 1) / SB_TW;
    t.tiles_y = (Hq + SB_TH - 1) / SB_TH;
    const long long total = (long long)(a.M / (a.Ho * a.Wo)) * t.tiles_x * t.tiles_y;
    if (total > 0x3fffffff) return hipErrorInvalidValue;
    t.total = (int)total;
    t.magic_tpi = stem_magic(t.tiles_x * t.tiles_y);
    t.magic_tx = stem_magic(t.tiles_x);
    const unsigned blocks = total < 768 ? xcd_grid(total) : 768u;      // three workgroups on every CU; the loop takes the rest
    EE_LAUNCH(conv_pool_i8_kernel, dim3(blocks), dim3(256), CP_LDS, s, a, yq, t);
    return hipGetLastError();
}

// the convolution as the launcher of the streaming kernel sees it (folded input), the pool behind it by its output size
bool stem_pool_supported(const ConvArgs& a, int es, int Hq, int Wq)
{
    if (es == 2 && !(a.f_lo >= 0.f)) return false;
    if (a.mode != 0 || a.res != nullptr || a.M <= 0 || a.Ci != 16 || a.kh != 4 || a.kw != 4 || a.stride != 1 || a.pad != 0 || a.pad_w != 0) return false;
    if (a.Co != 64 || a.ldc != 64 || a.c_off != 0 || a.Kp < 256 || a.H < a.Ho + 3 || a.W < a.Wo + 3) return false;
    if (Hq != (a.Ho + 2 - 3) / 2 + 1 || Wq != (a.Wo + 2 - 3) / 2 + 1 || Hq < 1 || Wq < 1) return false;
    return (double)(a.M / (a.Ho * a.Wo)) * a.H * a.W * 16 * es < 2147483648.0;
}

// A tile shape and what goes with it: small tiles where there is a CU for every one (int8)
static bool stem_tiles(const ConvArgs& a, int es, int Hq, int Wq, StemTile& t, bool& small)
{
    t.Hq = Hq; t.Wq = Wq; t.pool_pad = 1;
    t.images = a.M / (a.Ho * a.Wo);
    auto tiles = [&](int tw, int th) {
        t.tiles_x = (Wq + tw - 1) / tw;
        t.tiles_y = (Hq + th - 1) / th;
        return (long long)t.images * t.tiles_x * t.tiles_y;
    };
    small = es == 1 && tiles(ST_SMALL_TW, ST_SMALL_TH) <= 256;
    const long long total = small ? tiles(ST_SMALL_TW, ST_SMALL_TH) : es == 1 ? tiles(ST_TW, ST_TH) : tiles(SB_TW, SB_TH);
    if (total > 0x3fffffff) return false;
    t.total = (int)total;
    t.magic_tpi = stem_magic(t.tiles_x * t.tiles_y);
    t.magic_tx = stem_magic(t.tiles_x);
    return true;
}
// two workgroups on every CU (what matters is the CU's share, not the workgroup's); the loop takes the rest
static unsigned stem_blocks(const StemTile& t, unsigned most = 512) { return t.total < (int)most ? xcd_grid(t.total) : most; }

hipError_t launch_stem_pool(const ConvArgs& a, int es, void* yq, int Hq, int Wq, hipStream_t s)
{
    if (!stem_pool_supported(a, es, Hq, Wq)) return hipErrorInvalidValue;
    StemTile t;
    bool small;
    if (!stem_tiles(a, es, Hq, Wq, t, small)) return hipErrorInvalidValue;
    using K = void (*)(ConvArgs, void*, StemTile);
    const dim3 grid(stem_blocks(t));
    if (es == 2) EE_LAUNCH(static_cast<K>(stem_pool_bf16_kernel), grid, dim3(256), SB_LDS, s, a, yq, t);
    else if (small) EE_LAUNCH((static_cast<K>(stem_pool_i8_kernel<ST_SMALL_TW, ST_SMALL_TH>)), grid, dim3(256), (StemShape<ST_SMALL_TW, ST_SMALL_TH>::lds_bytes()), s, a, yq, t);
    else EE_LAUNCH((static_cast<K>(stem_pool_i8_kernel<ST_TW, ST_TH>)), grid, dim3(256), (StemShape<ST_TW, ST_TH>::lds_bytes()), s, a, yq, t);
    return hipGetLastError();
}

bool stem_image_supported(const void* x, int es, int W, int C) { return C == 3 && W * 3 * es % 16 == 0 && ((uintptr_t)x & 15) == 0; }

hipError_t launch_stem_image(const ConvArgs& a, int es, const void* x, const int32_t* ids, int H, int W, int pad, void* yq, int Hq, int Wq, hipStream_t s)
{
    if (!stem_pool_supported(a, es, Hq, Wq) || !stem_image_supported(x, es, W, 3)) return hipErrorInvalidValue;
    StemTile t;
    bool small;
    if (!stem_tiles(a, es, Hq, Wq, t, small)) return hipErrorInvalidValue;
    const bool by_value = ids && t.images <= 256;
    const ImageArgs im{x, by_value ? nullptr : ids, (int)by_value, H, 3 * W * es, pad};
    const dim3 grid(stem_blocks(t, es == 2 ? 512 : 768));
    auto launch = [&](auto tab) {
        using Tab = decltype(tab);
        using K = void (*)(Tab, ConvArgs, void*, StemTile, ImageArgs);
        if (by_value) std::memcpy(tab.id, ids, sizeof(int32_t) * (size_t)t.images);
        if (es == 2) EE_LAUNCH(static_cast<K>(stem_pool_bf16_kernel), grid, dim3(256), SI_LDS, s, tab, a, yq, t, im);
        else if (small) EE_LAUNCH((static_cast<K>(stem_pool_i8_kernel<ST_SMALL_TW, ST_SMALL_TH>)), grid, dim3(256), (StemImageShape<ST_SMALL_TW, ST_SMALL_TH>::lds_bytes()), s, tab, a, yq, t, im);
        else EE_LAUNCH((static_cast<K>(stem_pool_i8_kernel<ST_TW, ST_TH>)), grid, dim3(256), (StemImageShape<ST_TW, ST_TH>::lds_bytes()), s, tab, a, yq, t, im);
    };
    if (by_value && t.images > 64) launch(ImageIds<256>{});
    else launch(ImageIds<64>{});
    return hipGetLastError();
}

// ---- a folded stride-2 first layer of 2 x 2 taps straight from the images (int8, 3 channels) ------------------------------------
// Without a folded copy of the batch and the launch that makes it.  A workgroup takes R output rows of one image: the 2 R + 2 image rows under them are one contiguous piece of it, copied into LDS
// asynchronously, folded there into super-pixels (a lane: two neighbouring ones, see image_pixels; pixels outside the image become zero by comparison, as they lie inside the piece), and its
// wavefronts walk over the strips with their operands from LDS.  A lane's requantised 16 channels go straight to memory, 1 KB of contiguous bytes a wavefront.
// R: the most of 8, 4, 2 and 1 rows that leaves two workgroups for every CU (a row of super-pixels in R + 1 is folded twice), within the LDS of four workgroups to a CU; one or four per CU instead
// measured alike, but for 304 x 304, 13 samples (four: 9.4 us instead of 7.2).  Bound by latency on a few samples, by HBM on many (128 of 304 x 304: 129 MB written and read in 23 us).
// 32 channels, us, the folded copy and the streaming kernel / this one, both with the time between launches and the 1x1 layer behind: 224 x 224, 1 sample 13.2 / 9.8, 24 19.2 / 14.5, 64 35.4 / 27.5,
// 128 56.8 / 43.9; 304 x 304, 64 59.3 / 42.1.  By itself, 224 x 224 and 64 samples, 6.1 + 11.5 / 10.1.
struct StreamBand {
    int rows, bands, total;             // output rows of a workgroup, workgroups of an image, in all
    int pairs;                          // pairs of super-pixels of a folded row
    unsigned magic_bands, magic_pairs;
    int raw;                            // bytes of LDS for the image rows: whole copies of a wavefront
};
constexpr int BAND_MARGIN = 16;         // in front of the image rows in LDS, and behind them
static int band_lds(const StreamBand& t) { return 2 * BAND_MARGIN + t.raw + (t.rows + 1) * t.pairs * 32; }

template <int NT>
__device__ __forceinline__ void stream_band(const ConvArgs& a, const ImageArgs& im, const StreamBand& t, ImageTab tab)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char stem_lds[];
    const int tid = threadIdx.x, lane = tid & 63, p = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int unit = xcd_unit(blockIdx.x, t.total);
    if (unit < 0) return;
    const int n = (int)fast_div((unsigned)unit, (unsigned)t.bands, t.magic_bands), y0 = (unit - n * t.bands) * t.rows, rows = min(t.rows, a.Ho - y0);
    const int iy0 = 2 * y0 - im.pad, ia = min(max(iy0, 0), im.H - 1), ib = max(min(iy0 + 2 * rows + 2, im.H), ia + 1);     // the rows that exist, at least one
    const int from = (ia * im.row_bytes) & ~15, chunks = (ib * im.row_bytes - from + 15) >> 4;
    const unsigned char* src = image_at(im, tab, n) + from;
    unsigned char* const l_raw = stem_lds + BAND_MARGIN;
    unsigned char* const l_fold = l_raw + t.raw + BAND_MARGIN;
    const unsigned raw0 = lds_addr(l_raw);
    for (int c = 64 * wave; c < chunks; c += 256)
        dma16(raw0 + c * 16, c + lane < chunks ? src + (c + lane) * 16 : (const unsigned char*)a.zeros);
    v4i_r wreg[NT][2];
    v16i_r bias[NT];                                                    // rounding constant included
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) wreg[j][kb] = *(const v4i_r*)((const unsigned char*)a.w + (size_t)(32 * j + p) * a.Kp + kb * 32 + 16 * hi);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const v4i_r b4 = *(const v4i_r*)((const int*)a.bias + 32 * j + 8 * g + 4 * hi);
#pragma unroll
            for (int e = 0; e < 4; ++e) bias[j][4 * g + e] = b4[e];
        }
    }
    const IrClamp cl = ir_clamp(a.shift, a.lo, a.hi);
    const bool relu = ir_relu(a.shift, a.lo, a.hi);
    const int W = im.row_bytes / 3, pitch = t.pairs * 32;
    wait_all_then_barrier<0>();
    for (int i = tid; i < (rows + 1) * t.pairs; i += 256) {
        const int fr = (int)fast_div((unsigned)i, (unsigned)t.pairs, t.magic_pairs), pr = i - fr * t.pairs, ix = 4 * pr - im.pad;
        unsigned px[2][4];
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
            const int iy = iy0 + 2 * fr + dy;
            image_pixels(stem_lds, BAND_MARGIN + min(max(iy, ia), ib - 1) * im.row_bytes - from + 3 * min(ix, W), px[dy]);     // (past the row's end: bytes that do not count)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if ((unsigned)iy >= (unsigned)im.H || (unsigned)(ix + k) >= (unsigned)W) px[dy][k] = 0;
        }
        v4i_r* q = (v4i_r*)(l_fold + fr * pitch + pr * 32);
        q[0] = v4i_r{(int)px[0][0], (int)px[0][1], (int)px[1][0], (int)px[1][1]};
        q[1] = v4i_r{(int)px[0][2], (int)px[0][3], (int)px[1][2], (int)px[1][3]};
    }
    lds_barrier();
    const int m_end = rows * a.Wo;
    const auto y_buf = __builtin_amdgcn_make_buffer_rsrc((unsigned char*)a.y + ((long long)n * a.Ho + y0) * a.Wo * a.ldc, (short)0, m_end * a.ldc, 0x00020000);     // ends with the band: what is past it is dropped
    for (int s = wave; s * 32 < m_end; s += 4) {
        const int m = 32 * s + p, mc = min(m, m_end - 1), oy = (int)fast_div((unsigned)mc, (unsigned)a.Wo, a.magic_wo), ox = mc - oy * a.Wo;
        const unsigned char* first = l_fold + oy * pitch + (ox + hi) * 16;
        const v4i_r x0 = *(const v4i_r*)first, x1 = *(const v4i_r*)(first + pitch);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            v16i_r acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wreg[j][0], x0, bias[j], 0, 0, 0);
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wreg[j][1], x1, acc, 0, 0, 0);
            const v4i_r o = ir_requant_pack(acc, cl, relu);
            const int ch = 32 * j + 16 * hi;
            __builtin_amdgcn_raw_buffer_store_b128(o, y_buf, ch < a.Co ? (unsigned)(m * a.ldc + a.c_off + ch) : 0x80000000u, 0, 0);
        }
    }
}
template <int NT, int N>
__global__ __launch_bounds__(256, 4) void conv_stream_image_i8_kernel(ImageIds<N>, ConvArgs a, ImageArgs im, StreamBand t)
{
    if constexpr (N == 64) request_args<sizeof(ImageIds<64>) + sizeof(ConvArgs) + sizeof(ImageArgs) + sizeof(StreamBand)>();
    stream_band<NT>(a, im, t, (ImageTab)__builtin_amdgcn_kernarg_segment_ptr());
}

static StreamBand band_of(const ConvArgs& a, int row_bytes, int rows)
{
    StreamBand t;
    t.rows = rows;
    t.bands = (a.Ho + rows - 1) / rows;
    t.total = a.M / (a.Ho * a.Wo) * t.bands;
    t.pairs = (a.Wo + 2) / 2;
    t.magic_bands = stem_magic(t.bands);
    t.magic_pairs = stem_magic(t.pairs);
    t.raw = (((2 * rows + 2) * row_bytes + 15 + 15) / 16 + 63) / 64 * 1024;
    return t;
}

bool conv_stream_image_supported(const ConvArgs& a, int es, const void* x, int H, int W, int C, int pad)
{
    return es == 1 && C == 3 && a.Ci == 16 && a.kh == 2 && a.kw == 2 && a.stride == 1 && a.pad == 0 && a.pad_w == 0 && conv_stream_supported(a, 1) && pad >= 0 && pad <= 5 && (long long)H * W * 3 % 16 == 0 &&
           ((uintptr_t)x & 15) == 0 && a.M / (a.Ho * a.Wo) <= 65535 && a.Ho <= 4096 && (long long)a.Wo * a.ldc <= 1 << 24 && band_lds(band_of(a, 3 * W, 1)) <= 64 * 1024;
}

hipError_t launch_conv_stream_image(const ConvArgs& a, const void* x, const int32_t* ids, int H, int W, int pad, hipStream_t s)
{
    if (!conv_stream_image_supported(a, 1, x, H, W, 3, pad)) return hipErrorInvalidValue;
    const int images = a.M / (a.Ho * a.Wo);
    StreamBand t = band_of(a, 3 * W, 1);
    for (int rows = 8; rows > 1; rows /= 2) {
        const StreamBand u = band_of(a, 3 * W, rows);
        if (u.total >= 512 && band_lds(u) <= 40 * 1024) { t = u; break; }
    }
    const bool by_value = ids && images <= 256;
    const ImageArgs im{x, by_value ? nullptr : ids, (int)by_value, H, 3 * W, pad};
    auto launch = [&](auto tab) {
        if (by_value) std::memcpy(tab.id, ids, sizeof(int32_t) * (size_t)images);
        constexpr int N = sizeof(tab.id) / sizeof(int32_t);
        if (a.Co > 32) EE_LAUNCH((conv_stream_image_i8_kernel<2, N>), dim3(xcd_grid(t.total)), dim3(256), band_lds(t), s, tab, a, im, t);
        else EE_LAUNCH((conv_stream_image_i8_kernel<1, N>), dim3(xcd_grid(t.total)), dim3(256), band_lds(t), s, tab, a, im, t);
    };
    if (by_value && images > 64) launch(ImageIds<256>{});
    else launch(ImageIds<64>{});
    return hipGetLastError();
}

}  // namespace ee
