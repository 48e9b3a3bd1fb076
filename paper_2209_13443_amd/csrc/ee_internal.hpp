// Internal declarations of the early-exit serving library (gfx950 only).
#pragma once
#include <utility>
#include <hip/hip_runtime.h>
#include <cstring>
#include <hip/hip_ext.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/ee.h"

namespace ee {

// ---- network description parsed from the blob ------------------------------------------------
enum OpKind { OP_CONV = 0, OP_DWCONV = 1, OP_MAXPOOL = 2, OP_AVGPOOL = 3 };

struct OpDesc {
    int kind, src, dst, res;
    int h_in, w_in, c_in, h_out, w_out, c_out;
    int kh, kw, stride, pad;      // pad: rows of zero padding above and below
    int shift, res_shift, lo, hi;
    float f_lo, f_hi;
    int64_t w_off, b_off;
    int pad_w;                    // columns of zero padding left and right
    int c_off, c_tot;             // the op writes channels [c_off, c_off + c_out) of a tensor of c_tot channels (concatenation)
};

struct ExitDesc {
    int h, w, c, n_cls, gap_shift, frac_bits;
    float logit_scale, thr;
    int64_t w_off, b_off;
};

struct StageDesc {
    int first_op, n_ops, n_tensors, out_tensor;
    int in_h, in_w, in_c, out_h, out_w, out_c;
};

struct NetDesc {
    int dtype = 0, n_classes = 0, in_h = 0, in_w = 0, in_c = 0;
    std::vector<StageDesc> stages;
    std::vector<OpDesc> ops;
    std::vector<ExitDesc> exits;
    int elem_bytes() const { return dtype == EE_I8 ? 1 : 2; }
};

// Validates and decodes a blob.  Returns an ee_status.
int parse_blob(const void* blob, size_t bytes, NetDesc* out);

// ---- slot tables (zero-copy compaction) ----------------------------------------------------------
// Survivors of an exit are never moved: the samples of a batch live in arbitrary slots of the next segment's
// input memory and a table names the slot of every batch row (the GPU analogue of changing only the DMA
// addressing, Sec. III-A / III-B "Overhead").  The host hands a step's two tables (input rows, output rows) to one
// tiny kernel by value, which stores them in device memory; the convolution and pooling kernels read them there.
enum { EE_ZC_MAX_B = 256 };
struct SlotTab { uint16_t s[EE_ZC_MAX_B]; };
// dst[0 .. b) = in, dst[256 .. 256 + b) = out
hipError_t launch_upload_slots(const SlotTab& in, const SlotTab& out, int b, uint16_t* dst, hipStream_t s);

// ---- kernel argument blocks --------------------------------------------------------------------
// Implicit-GEMM convolution: rows = output pixels m = (n, oy, ox), columns = output channels,
// reduction over (r, s, c).  Weights are pre-packed [Co_pad][Kp] with the reduction index the
// loader uses (see pack_weights in ee_api.cpp), zero padded.
struct ConvArgs {
    const void* x; const void* w; const void* bias; const void* res; void* y;
    const void* wo;      // the same weights as ready matrix-instruction operands [32 rows][step of 32 bytes][lane][16] (conv_skinny_kernel), or null
    const void* zeros;   // >= 16 readable zero bytes: what padding taps and rows past the batch read
    int M, H, W, Ci, Ho, Wo, Co;
    int kh, kw, stride, pad;   // pad: rows
    int pad_w;           // columns of padding
    int ldc, c_off;      // the output pixel has ldc channels, of which this layer writes [c_off, c_off + Co)
    int Kp;              // weight row pitch in elements (reduction length, zero padded)
    unsigned magic_howo, magic_wo;   // floor(2^32 / (Ho*Wo)), floor(2^32 / Wo): division by multiply-high
    unsigned tap_rows;   // bit r*kw set for every kernel row r (kh*kw <= 31)
    unsigned magic_spt, magic_kw;    // set by the launchers of the few-pixel kernel: floor(2^32 / steps of a tap), floor(2^32 / kw)
    int plain_step;      // set by the launcher: bytes the source of a row advances per reduction step when no tap needs a check
    int mode;            // 0: Ci % 16 == 0 loader with bounds checks; 1: 4-channel zero-padded input
    int Hp, Wp, kwp;     // mode 1: padded input dims and padded kernel width
    int shift, res_shift, lo, hi;
    float f_lo, f_hi;
    int* gap_sums;       // not null (int8, conv_igemm_kernel, conv_skinny_kernel or conv_taps_kernel, last layer of a segment): also add the per-sample channel sums of the output into gap_sums[n][Co]
    const uint16_t* xs;  // not null: sample n of the input is slot xs[n] of x (device memory; conv_igemm_kernel, conv_skinny_kernel and conv_rows_kernel only)
    const uint16_t* ys;  // not null: sample n of the output is slot ys[n] of y (device memory; those and conv_taps_kernel)
};

// Two chained convolutions in one launch (kernels_pair.hip): c2 is the first layer (its y and res are unused, its
// output stays on chip), the rest describes the 1x1 layer that reads it.
struct PairArgs {
    ConvArgs c2;
    const void* w3; const void* bias3; const void* res; void* y;
    int Co3, Kp3;        // second layer: output channels, weight row pitch in elements
    int shift, res_shift, lo, hi;
    float f_lo, f_hi;
};

// The seam of two bottleneck blocks in one launch (kernels_seam.hip): a 3x3 stride-1 layer with padding 1 (C -> C channels; w0 null: not part of the launch), the 1x1 layer with a
// residual behind it (C -> N1) and the 1x1 layer that reads that one (N1 -> N2).  x is the first of them's input; y1 and y2 are the 1x1 layers' outputs.
struct SeamArgs {
    const void* x; const void* res; void* y1; void* y2;
    const void* w0; const void* b0; const void* w1; const void* b1; const void* w2; const void* b2;    // ready operands (ConvArgs::wo) and padded biases
    int M, H, W, C, N1, N2;
    unsigned magic_hw, magic_w;      // floor(2^32 / (H W)), floor(2^32 / W)
    int pitch0, pitch1, pitch2;      // operand steps of 32 bytes per block of 32 weight rows
    int shift0, lo0, hi0, shift1, res_shift, lo1, hi1, shift2, lo2, hi2;
};

// An inverted-residual block in one launch (kernels_ir.hip): 1x1 expansion -> 3x3 depthwise -> 1x1 projection (+ residual).
// Weights and biases are packed for it when the context is created: expansion rows of Kx bytes (c_in padded with zeros
// to a multiple of 32) for Ce32 channels (the expanded channels padded to a multiple of 32, padding rows zero), the
// depthwise weights as ready matrix-instruction operands [Ce32 / 32][5][lane][16] (diagonal matrices, ir_diag_operands), projection rows
// of Ce32 bytes for NCO * 32 output channels; be and bd include the rounding constants of their shifts.
struct IrArgs {
    const void* x; const void* res; void* y;
    const void* we; const int* be;
    const void* wd; const int* bd;
    const void* wp; const int* bp;
    int B, H, W, Cin, Kx, Ce32, Cout, Ho, Wo, stride, pad;
    int sh_e, lo_e, hi_e, sh_d, lo_d, hi_d, sh_p, lo_p, hi_p, res_shift;
    const uint16_t* ys;  // bottleneck block only; not null: sample n of the output goes to slot ys[n] of y (device memory; B <= EE_ZC_MAX_B)
    int* gap_sums;       // int8; not null: also add the per-sample channel sums of the output into gap_sums[n][Cout]
    const void* ws; const int* bs;   // bottleneck block only; not null: the residual is the 1x1 convolution of x with these operands and biases
    int sh_s, lo_s, hi_s;            // (res is null then), requantised with these
    float f_lo_e, f_hi_e, f_lo_d, f_hi_d, f_lo_p, f_hi_p, f_lo_s, f_hi_s;      // bf16 bottleneck block: the layers' bounds, the biases are floats
};

struct DirectConvArgs {   // one thread per output element; any shape (correctness fallback)
    const void* x; const void* w; const void* bias; const void* res; void* y;
    int M, H, W, Ci, Ho, Wo, Co, kh, kw, stride, pad, shift, res_shift, lo, hi;
    float f_lo, f_hi;
    int pad_w, ldc, c_off;
};

struct PoolArgs {         // depthwise 3x3 and max-pool share the shape block
    const void* x; const void* w; const void* bias; void* y;
    const void* w3;      // int8 3x3 depthwise: weights packed for the dot-product kernel, [C/16][column][4-channel group][channel] dwords (or null)
    int B, H, W, C, Ho, Wo, k, stride, pad, shift, lo, hi;
    float f_lo, f_hi;
    int ldc, c_off;      // pooling: the output pixel has ldc channels, of which this layer writes [c_off, c_off + C)
};

// ---- kernel launches ---------------------------------------------------------------------------------
// Every kernel goes out through EE_LAUNCH.  While a launch is being timed, the pair of events named here is attached
// to the dispatch itself (its own begin and end time stamps, what a kernel trace shows), instead of event records in
// front of and behind it, which would also count the dispatch latency of a stream whose back-to-back launches they break.
extern thread_local hipEvent_t g_launch_start, g_launch_stop;     // null: an ordinary launch
#define EE_LAUNCH(kernel, grid, block, lds_bytes, stream, ...) \
    hipExtLaunchKernelGGL(kernel, grid, block, lds_bytes, stream, ee::g_launch_start, ee::g_launch_stop, 0, __VA_ARGS__)

// ---- which part of the batch runs where ------------------------------------------------------------
// Workgroups go to the 8 XCDs in turn, and a line that a kernel has written stays in the L2 of the XCD that wrote it: reading it from
// another XCD is 2-3 times as slow (12 MB moved by one kernel after the other: 3.8 us when every workgroup reads what its own XCD
// wrote, 9.3 us when it reads what the next one wrote).  So every kernel gives XCD k the k-th eighth of the batch, counted in
// units of its own (tiles, strips, rows, blocks of pixels): xcd_unit is the workgroup's unit, or -1 for a workgroup past its XCD's share.
inline unsigned xcd_grid(long long units) { return (unsigned)((units + 7) / 8 * 8); }
__device__ __forceinline__ int xcd_first(int xcd, int units) { return (int)((unsigned)units * (unsigned)xcd >> 3); }      // units < 2^28
__device__ __forceinline__ int xcd_unit(unsigned block, int units)
{
    const int k = (int)(block & 7), u = xcd_first(k, units) + (int)(block >> 3);
    return u < xcd_first(k + 1, units) ? u : -1;
}

// All of a launch's arguments (BYTES in all, at least), a word of every 64-byte line, requested together at the start of a kernel.  They are in memory that no cache holds when a kernel starts; left to
// itself the compiler loads each where it is first needed, a round trip to that memory per line not asked for before: three or four of them one after the other in front of a kernel's first load.
// MobileNetV2, one image through every segment and head (31 launches) 166.8 -> 161.2 us; bf16 ResNet-50, 5 samples (62 launches) 386.5 -> 382.5.
// BYTES ends inside the explicit arguments: the sum of the structures a kernel begins with, or explicit_args of the kernel's own list.
template <int BYTES>
__device__ __forceinline__ void request_args()
{
    const __attribute__((address_space(4))) int* k = (const __attribute__((address_space(4))) int*)__builtin_amdgcn_kernarg_segment_ptr();
    const int x = [&]<int... LINE>(std::integer_sequence<int, LINE...>) { return (k[16 * LINE] ^ ...); }(std::make_integer_sequence<int, (BYTES + 63) / 64>{});
    asm volatile("" ::"s"(x));
}

// Bytes of a kernel's arguments, laid out one after the other at their alignment
template <typename F> struct explicit_args;
template <typename... A>
struct explicit_args<void(A...)> {
    static constexpr int bytes()
    {
        size_t n = 0;
        ((n = (n + alignof(A) - 1) / alignof(A) * alignof(A) + sizeof(A)), ...);
        return (int)n;
    }
};
static_assert(explicit_args<void(int, void*, short, int)>::bytes() == 24, "padding in front of an argument, none behind the last");

// ---- launchers (defined in the .hip files) -------------------------------------------------------
hipError_t launch_conv_mfma_i8(const ConvArgs& a, hipStream_t s);
hipError_t launch_conv_mfma_bf16(const ConvArgs& a, hipStream_t s);
// asynchronous-copy implicit GEMM (ES = element bytes); tile 0 = chosen by shape, 1..4 forced
template <int ES> hipError_t launch_conv_igemm(const ConvArgs& a, int tile, hipStream_t s);
int conv_igemm_default(const ConvArgs& a, int es, long long blocks);      // its configuration for an untuned launch of that many 64 x 64 tiles
// the fused pair (ES = element bytes); cfg 0 = chosen by shape
template <int ES> hipError_t launch_conv_pair(const PairArgs& p, int cfg, hipStream_t s);
bool conv_pair_supported(int es, int co2, int kh, int kw, int ci, int co3);
// the seam of two bottleneck blocks (int8); cfg: EE_CFG_SEAM | blocks of 32 pixels per wavefront in the narrow layers (1 or 2) | EE_CFG_SEAM_FRONT: with the 3x3 layer.  Stored in the
// table of the pair that ends the block
enum { EE_CFG_SEAM = 0x40000, EE_CFG_SEAM_FRONT = 0x10 };
bool conv_seam_supported(int es, int c, int n1, int n2);
bool conv_seam_config_ok(int cfg, int c, int W, bool front);       // cfg names such a launch, it exists there (front: whether the 3x3 layer can be part of it) and fits LDS
int conv_seam_default(const SeamArgs& a, bool front, bool joint);  // configuration of an untuned launch, or 0: the layers one by one are faster; joint: the last of them by itself would share a launch
hipError_t launch_conv_seam(const SeamArgs& a, int cfg, hipStream_t s);
// stride-1 "same" convolutions with the activation slab of a tile resident in LDS (kernels_slab.hip); cfg as documented there
bool conv_slab_supported(const ConvArgs& a, int es);
template <int ES> hipError_t launch_conv_slab(const ConvArgs& a, int cfg, hipStream_t s);
int conv_slab_default(const ConvArgs& a, int es);      // configuration of an untuned launch it is the faster one for, else 0
// 1x1 layers with resident weights (kernels_rows.hip): tiles of 32 or 64 pixels.  Its configuration words ask for four wavefront groups with
// 256-byte steps on a large tile, which the staged kernel does not have
enum { EE_CFG_ROWS32 = 0x4231, EE_CFG_ROWS64 = 0x4232 };
inline bool cfg_is_rows(int cfg) { return cfg == EE_CFG_ROWS32 || cfg == EE_CFG_ROWS64; }
bool conv_rows_supported(const ConvArgs& a, int es);
bool conv_rows_config_ok(const ConvArgs& a, int cfg, int es);      // cfg names this kernel and runs on that layer
int conv_rows_default(const ConvArgs& a, int es);      // configuration of an untuned launch it is the faster one for, else 0
template <int ES> hipError_t launch_conv_rows(const ConvArgs& a, int cfg, hipStream_t s);
// the same layers over pixels of whole 32-byte runs (bf16: 64), the weights streamed into registers (kernels_taps.hip): tiles of tm blocks of 32 pixels x 32 channels
// for each of nw wavefronts, the reduction shared by kp.  nw 4: tm 2, 3, 4, 5, 7, with kp 2 tm 2 and 4; nw 8: tm 4 and 7; nw 2: tm 2 and 4, with kp 2 and 4 tm 2
// (tm other than 2 and 4 only for whole 128-byte runs); int8 layers without padding: tm 4 with nw 2, 3 and 4.  Its configuration words ask for wavefront groups with 256-byte steps in combinations that the staged
// kernel does not have, like those of kernels_rows.hip
constexpr int taps_cfg(int tm, int nw, int kp)
{
    if (nw == 3) return 0x4531;
    return nw == 2 && kp < 4 ? (kp == 2 ? 0x4434 : tm == 2 ? 0x4234 : 0x4334) : kp == 4 ? 0x4332 : kp == 2 ? (tm == 2 ? 0x2232 : 0x2332) : nw == 8 ? (tm == 4 ? 0x2432 : 0x4432) : 0x31 | (tm <= 4 ? 0x2000 | tm << 8 : tm == 5 ? 0x4300 : 0x4400);
}
constexpr int TAPS_CFGS[] = {taps_cfg(2, 4, 1), taps_cfg(3, 4, 1), taps_cfg(4, 4, 1), taps_cfg(5, 4, 1), taps_cfg(7, 4, 1), taps_cfg(2, 4, 2), taps_cfg(4, 4, 2), taps_cfg(2, 2, 4), taps_cfg(4, 8, 1), taps_cfg(7, 8, 1), taps_cfg(2, 2, 1), taps_cfg(4, 2, 1), taps_cfg(2, 2, 2), taps_cfg(4, 3, 1)};
inline bool cfg_is_taps(int cfg)
{
    for (const int c : TAPS_CFGS)
        if (cfg == c) return true;
    return false;
}
// whether wavefronts share a reduction (another order of a bf16 sum than the staged kernels')
constexpr bool cfg_taps_shares(int cfg) { return cfg == taps_cfg(2, 4, 2) || cfg == taps_cfg(4, 4, 2) || cfg == taps_cfg(2, 2, 2) || cfg == taps_cfg(2, 2, 4); }
bool conv_taps_supported(const ConvArgs& a, int es);
bool conv_taps_config_ok(const ConvArgs& a, int cfg, int es);      // cfg names this kernel and runs on that layer: it covers it, the tile exists for its pixels and fits LDS
int conv_taps_default(const ConvArgs& a, int es);      // configuration of an untuned launch it is the faster one for, else 0
template <int ES> hipError_t launch_conv_taps(const ConvArgs& a, int cfg, hipStream_t s);
enum { EE_CFG_SLAB = 0x10000 };     // configuration words with this bit name the slab kernel
// few output pixels: the reduction split over a workgroup's wavefronts, operands straight from global memory (kernels_skinny.hip)
// Its configuration words are those whose fields ask for wavefront groups (bits 12-15: 2 = tiles of 32 pixels, 4 = of 16) with a step
// field of 1 or 2 (bits 4-7: blocks of channels per workgroup), which the staged kernel does not have; bits 0-3: log2 of the
// wavefronts + 1 (with ring field 2 in bits 8-11), or 4 with ring field 3 for 16 wavefronts.
constexpr int skinny_cfg(int t, int tn, int lw) { return (lw < 4 ? lw + 1 : 4) | tn << 4 | (lw < 4 ? 2 : 3) << 8 | (t == 32 ? 2 : 4) << 12; }
inline bool cfg_is_skinny(int cfg)
{
    const int step = (cfg >> 4) & 15, groups = cfg >> 12;
    return cfg > 0 && (groups == 2 || groups == 4) && (step == 1 || step == 2);
}
bool conv_skinny_config_ok(int cfg);
int conv_skinny_default(const ConvArgs& a, int es);    // configuration of an untuned launch it is the faster one for, else 0
int conv_skinny_order_bf16(const ConvArgs& a);         // the word whose wavefronts share the reduction of a tuned bf16 layer of this size, or 0: the order of the staged kernels
// ee_autotune tries it up to this many output pixels: every operand byte it loads feeds one instruction, so with more it is never the fastest
constexpr long long EE_SKINNY_MAX_ROWS = 8192;
template <int ES> hipError_t launch_conv_skinny(const ConvArgs& a, int cfg, hipStream_t s);
// several independent int8 layers in one launch with one configuration (kernels_group.hip)
enum { EE_GROUP_MAX = 4 };
bool conv_group_config_ok(int cfg);
hipError_t launch_conv_group(const ConvArgs* a, int n, int cfg, hipStream_t s);
enum { EE_CFG_IR_BLOCK = 0x20000 }; // ee_time_layer: the fused inverted-residual block headed by the layer
// streaming kernel for large, thin int8 layers (es = element bytes); hipErrorInvalidValue for a layer it does not cover
bool conv_stream_supported(const ConvArgs& a, int es);
hipError_t launch_conv_stream(const ConvArgs& a, hipStream_t s);
// the folded stride-2 first layer of 2 x 2 taps (a as for the folded copy, a.x unused) from int8 images of H x W x 3 at x with no folded copy: sample n is image n, or ids[n] (host memory the device can read)
bool conv_stream_image_supported(const ConvArgs& a, int es, const void* x, int H, int W, int C, int pad);
hipError_t launch_conv_stream_image(const ConvArgs& a, const void* x, const int32_t* ids, int H, int W, int pad, hipStream_t s);
// 1x1 int8 layers with at most 32 input channels: activations and weights straight from global memory into one
// matrix instruction per 32 x 32 outputs (w: packed rows of 32 bytes, zero padded; bias with the rounding constant)
struct ThinConvArgs {
    const void* x; const void* w; const void* bias; void* y;
    long long M;                 // output pixels of the batch
    int Ci, Co, ldc, c_off, shift, lo, hi;
};
hipError_t launch_conv_thin(const ThinConvArgs& a, hipStream_t s);
bool conv_thin_supported(int es, int kh, int kw, int stride, int pad, int pad_w, int ci, int co, int c_tot, int c_off, bool has_res);
int forced_conv_tile();
hipError_t launch_conv_direct(const DirectConvArgs& a, int dtype, hipStream_t s);
hipError_t launch_pad_input(const void* x, void* y, int B, int H, int W, int C, int Hp, int Wp, int pad, int dtype, hipStream_t s);
// [B][H][W][C<=4] -> [B][Hs][Ws][2][2][4]: zero padding `pad`, then 2 x 2 pixel blocks folded into channels;
// with gather (device-visible) sample n is read from row gather[n] of x
// gather_on_host: gather points to host memory the caller may read now (then up to 256 ids travel in the kernel arguments)
hipError_t launch_space_to_depth(const void* x, void* y, const int32_t* gather, int B, int H, int W, int C, int Hs, int Ws, int pad, int dtype, hipStream_t s,
                                 bool gather_on_host = false);
// [rows][c_bytes] -> [rows][cp_bytes] (both multiples of 4), the tail of every row zero
hipError_t launch_pad_channels(const void* x, void* y, long long rows, int c_bytes, int cp_bytes, hipStream_t s);
hipError_t launch_depthwise(const PoolArgs& a, int dtype, hipStream_t s);
// the fused inverted-residual block (int8); pointers may be null for ir_block_supported
bool ir_block_pools(const IrArgs& a);                  // whether its launch can carry the exit head's pooling
bool ir_block_supported(const IrArgs& a);
int ir_block_out_blocks(int c_out);            // blocks of 32 output channels the kernel is instantiated with (weights are padded to it)
hipError_t launch_ir_block(const IrArgs& a, hipStream_t s);
// bottleneck block (1x1 -> 3x3 -> 1x1 + residual) in one launch; the same argument block: we / be, wd / bd, wp / bp are the three
// layers' operands and biases, Kx = Cin, Ce32 = the middle channels
// first convolution (folded stride-2 layer, 4 x 4 taps over 16-channel super-pixels, 64 output channels: a as for the streaming
// kernel, a.y unused) and the 3x3 / 2 max-pool with padding 1 behind it in one launch; yq: the pooled output [B][Hq][Wq][64]
bool stem_pool_supported(const ConvArgs& a, int es, int Hq, int Wq);
hipError_t launch_stem_pool(const ConvArgs& a, int es, void* yq, int Hq, int Wq, hipStream_t s);
// the same from images of H x W x 3 at x (a.x unused), padded by `pad` in front, with no folded copy: sample n is image n, or ids[n] (host memory the device can read); x and its rows in whole 16-byte chunks
bool stem_image_supported(const void* x, int es, int W, int C);
hipError_t launch_stem_image(const ConvArgs& a, int es, const void* x, const int32_t* ids, int H, int W, int pad, void* yq, int Hq, int Wq, hipStream_t s);
// a 3x3 convolution from 32 to 64 channels and the 3x3 / 2 max-pool (padding 0 or 1) behind it in one launch (int8)
bool conv_pool_supported(const ConvArgs& a, int es, int Hq, int Wq, int pool_pad);
hipError_t launch_conv_pool(const ConvArgs& a, void* yq, int Hq, int Wq, int pool_pad, hipStream_t s);
bool bneck_block_supported(const IrArgs& a);
bool bneck_block_pools(const IrArgs& a);     // with a.gap_sums the launch also pools: only where its rows of sums fit into LDS
hipError_t launch_bneck_block(const IrArgs& a, hipStream_t s);
// its bf16 form (kernels_bneck16.hip): always with a residual, or with the convolution on the shortcut; does not pool
bool bneck_block_bf16_supported(const IrArgs& a);
hipError_t launch_bneck_block_bf16(const IrArgs& a, hipStream_t s);
hipError_t launch_maxpool(const PoolArgs& a, int dtype, hipStream_t s);
hipError_t launch_avgpool(const PoolArgs& a, int dtype, hipStream_t s);

struct HeadArgs {
    const void* act; int B, HW, C, n_cls;
    int gap_shift, frac_bits; float logit_scale;
    const void* wfc; const void* wfo; const void* bfc;      // weights as rows (heads that head_small may take, else null) and as ready operands (head_operands)
    int32_t* sums;       // [B][C] int32 sums (i8) or float means (bf16)
    int32_t* gap_partial;   // bf16: [B][head_gap_splits(B, HW)][C] partial rows where that is more than one, else not used
    void* logits;        // [B][n_cls] int32 / float scratch
    int64_t s_thr; float thr; int last;
    int32_t* label; float* conf; int64_t* score; uint8_t* flag;
    // stream serving: per-slot outcomes written straight into pinned host memory, each with the launch's tag (null otherwise)
    struct HostOutcome* host_out; unsigned tag;
    const uint16_t* slots;   // pooling: not null: sample b of the batch is slot slots[b] of act (device memory)
    const uint32_t* exp2;    // the softmax's table in device memory (segment_small_i8_kernel)
    int es;                  // element bytes
};
// w0: bits 0-43 the score S (int8: S <= n_cls * 2^30 < 2^44; the host derives the confidence 2^30 / S) or the confidence's
// float bits (bf16); w1: bits 0-31 the label, bit 32 the exit flag; bits 44-63 of both: the launch's tag (never 0: a record the
// host has cleared matches no launch)
struct alignas(16) HostOutcome { uint64_t w0, w1; };
constexpr int EE_OUTCOME_TAG_SHIFT = 44;
inline unsigned outcome_tag(unsigned seq) { return seq % 0xFFFFFu + 1u; }
// host side: records [0, b) all carry the tag in both words
inline bool outcomes_ready(const HostOutcome* h, int b, unsigned tag)
{
    for (int k = b - 1; k >= 0; --k)
        if ((unsigned)(__atomic_load_n(&h[k].w0, __ATOMIC_ACQUIRE) >> EE_OUTCOME_TAG_SHIFT) != tag ||
            (unsigned)(__atomic_load_n(&h[k].w1, __ATOMIC_ACQUIRE) >> EE_OUTCOME_TAG_SHIFT) != tag) return false;
    return true;
}
struct Outcome { int64_t score; int32_t label; float conf; uint8_t flag; };
inline bool outcome_exits(const HostOutcome& h) { return (__atomic_load_n(&h.w1, __ATOMIC_RELAXED) >> 32) & 1u; }
inline Outcome decode_outcome(const HostOutcome& h, bool int8)
{
    const uint64_t w0 = __atomic_load_n(&h.w0, __ATOMIC_RELAXED), w1 = __atomic_load_n(&h.w1, __ATOMIC_RELAXED);
    const uint64_t payload = w0 & ((1ull << EE_OUTCOME_TAG_SHIFT) - 1);
    Outcome o;
    o.label = (int32_t)(uint32_t)w1;
    o.flag = (uint8_t)((w1 >> 32) & 1u);
    if (int8) {
        o.score = (int64_t)payload;
        o.conf = (float)(1073741824.0 / (double)o.score);       // as the kernel computes it for the device-side array
    } else {
        o.score = 0;
        const uint32_t bits = (uint32_t)payload;
        std::memcpy(&o.conf, &bits, 4);
    }
    return o;
}
// device address, on the current GPU, of the scratch array that is part of the library image (EE_STATIC_SCRATCH_BYTES bytes)
hipError_t static_scratch(void** out);
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);
constexpr int GAP_SLICE_PIXELS = 4096;      // bf16 pooling keeps partial rows only for images of more pixels
// parts the bf16 pooling splits a sample's pixels into: more than one are partial rows, B + 511 of them at most for the batch
int head_gap_splits(int B, int HW);
hipError_t launch_head_gap(const HeadArgs& a, int dtype, hipStream_t s);
hipError_t launch_head_fc(const HeadArgs& a, int dtype, hipStream_t s);
hipError_t launch_head_softmax(const HeadArgs& a, int dtype, hipStream_t s);
// all of it in one launch, for heads small enough (pooled: a.sums holds the sums already)
bool head_small(const HeadArgs& a, int dtype, bool pooled);
bool head_small_weights(long long row_bytes, int n_cls);      // its condition on the weights
hipError_t launch_head_small(const HeadArgs& a, int dtype, bool pooled, hipStream_t s);

// A small segment and its exit head in one launch (int8, kernels_segment.hip).  Tensors of one sample live in LDS: offsets and bytes per pixel.
enum { EE_SEG_LAYERS = 6, EE_SEG_ROWS = 64, EE_SEG_CHUNKS = 256 };
struct SegChunk { int off, tap; };       // bytes from the patch's corner in the source tensor, tap r * kw + s (31: past the end)
// What never changes is in device memory: the argument segment of a launch is host memory, where every cache line costs a round trip over the bus.
struct alignas(64) SegLayer {
    const void* wo; const int* bias;     // ready operands (ConvArgs::wo), biases with the rounding constant
    int w_off, bias_off, bias_kib;       // where they go in LDS; whole KiB of biases
    int tab;                             // in LDS: the layer's part of the table below
    unsigned tap_rows;                   // bit r * kw of every kernel row r
    int steps, pitch;                    // reduction steps of 32 bytes: of the layer, of a weight row
    int blocks, co;                      // blocks of 32 output channels, output channels (a multiple of 16)
    int src, src_pitch, dst, dst_pitch, res, res_pitch;      // res < 0: none
    int H, W, Ho, Wo, kh, kw, stride, pad, pad_w, cpp;       // cpp: 16-byte chunks per input pixel
    int shift, res_shift, lo, hi;
    unsigned magic_wo, magic_blocks, magic_steps;            // floor(2^32 / d): fast_div
};
struct alignas(64) SegPlan {
    int n;                                                   // layers; 0: the segment is not one of these
    int in_bytes, in_chunks, in_cpp, in_off, in_pitch;       // the input sample
    int fold, fold_off, fold_h, fold_w, fold_pad, img_h, img_w, img_c;      // folded first layer: the super-pixels and the raw image
    int zero_off, sums_off, feat_off, logits_off, exp2_off, lds_bytes, out_bytes;
    int tab_off, tab_kib;
    unsigned magic_cpp, magic_fold_w;
    SegLayer layer[EE_SEG_LAYERS];
    SegChunk tab[EE_SEG_CHUNKS];         // per layer and 16-byte chunk of its reduction (two per step): where it is
};
struct SegRows { int32_t src[EE_SEG_ROWS], dst[EE_SEG_ROWS]; };
// rows (host memory, up to EE_SEG_ROWS samples): input and output row of every sample, by value; else ids / xs and ys (device-visible, may be null)
// plan, dev_plan: the same on the host and on the device
hipError_t launch_segment_small(const SegPlan& plan, const SegPlan* dev_plan, const void* x, void* y, int B, const SegRows* rows, const int32_t* ids, const uint16_t* xs, const uint16_t* ys, const HeadArgs* h, hipStream_t s);

// Stable compaction + refill: the survivors of src[b_act], then the b_incr samples of refill.  dst_off: first destination slot
// of the survivors; ring_rows > 0: dst is a ring of that many slots and destination slots wrap around its end.
hipError_t launch_compact(const uint8_t* flag, const void* src, void* dst, const int32_t* ids_src, int32_t* ids_dst, int b_act,
                          const void* refill, const int32_t* refill_ids, int b_incr, int64_t sample_bytes, int dst_off, int ring_rows,
                          int* b_rem_out, int* b_merged_out, hipStream_t s);
// Admission: pool rows ids[k] -> slots [0, b)
hipError_t launch_admit(const void* pool, void* dst, const int32_t* ids, int b, int64_t sample_bytes, hipStream_t s);

}  // namespace ee
