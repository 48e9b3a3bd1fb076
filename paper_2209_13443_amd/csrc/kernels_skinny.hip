// The matrix-core convolution for few output pixels (skinny_kernel.hpp), one layer per launch.
#include "skinny_kernel.hpp"

namespace ee {

template <int ES, int T, int NW, int TN, bool PLAIN>
__global__ __launch_bounds__(64 * NW, 2) void conv_skinny_kernel(ConvArgs a, int gn, unsigned magic_gn, int nk, int pitch)
{
    request_args<sizeof(ConvArgs) + 16>();
    skinny_tile<ES, T, NW, TN, PLAIN ? SKINNY_PLAIN : SKINNY_ANY>(a, gn, magic_gn, nk, pitch, blockIdx.x);
}

template <int ES, int T, int NW, int TN>
__global__ __launch_bounds__(64 * NW, 2) void conv_skinny_taps_kernel(ConvArgs a, int gn, unsigned magic_gn, int nk, int pitch)
{
    request_args<sizeof(ConvArgs) + 16>();
    skinny_tile<ES, T, NW, TN, SKINNY_TAPS>(a, gn, magic_gn, nk, pitch, blockIdx.x);
}

// ---- launch -----------------------------------------------------------------------------------------------------------
template <int ES, int T, int NW, int TN>
static hipError_t launch_skinny(const ConvArgs& layer, hipStream_t s)
{
    ConvArgs a = layer;
    constexpr int KB = 1024 / T;
    const int gm = (a.M + T - 1) / T, gn = (a.Co + T * TN - 1) / (T * TN);
    const unsigned magic_gn = (unsigned)(0x100000000ull / (unsigned)gn - (gn == 1));
    const int nk = (a.kh * a.kw * a.Ci * ES + KB - 1) / KB, pitch = a.Kp * ES / 32;      // rows are padded to 256 bytes with zeros
    if ((long long)gm * gn > 0x7fffffff || !skinny_reaches(a, ES)) return hipErrorInvalidValue;
    const int mode = skinny_mode(a, ES, T);
    const dim3 grid((unsigned)(gm * gn)), block(64 * NW);
    if (mode == SKINNY_PLAIN) EE_LAUNCH((conv_skinny_kernel<ES, T, NW, TN, true>), grid, block, 0, s, a, gn, magic_gn, nk, pitch);
    else if (mode == SKINNY_TAPS) EE_LAUNCH((conv_skinny_taps_kernel<ES, T, NW, TN>), grid, block, 0, s, a, gn, magic_gn, nk, pitch);
    else EE_LAUNCH((conv_skinny_kernel<ES, T, NW, TN, false>), grid, block, 0, s, a, gn, magic_gn, nk, pitch);
    return hipGetLastError();
}

// log2 of the wavefronts of a configuration word (see skinny_cfg), or -1 when the library has no such kernel
static int skinny_waves(int cfg)
{
    if (!cfg_is_skinny(cfg)) return -1;
    const int tile = cfg & 15, tn = (cfg >> 4) & 15, ns = (cfg >> 8) & 15;
    if (tile < 1 || tile > 4 || !(ns == 2 || (ns == 3 && tile == 4))) return -1;
    const int lw = ns == 3 ? 4 : tile - 1;
    if (cfg >> 12 == 4) return tn == 1 && lw >= 2 ? lw : -1;
    return tn == 1 || lw <= 3 ? lw : -1;
}

bool conv_skinny_config_ok(int cfg) { return skinny_waves(cfg) >= 0; }

// Untuned: the configuration of a launch this kernel is the faster one for, else 0 (asked behind conv_taps_default).  Measured over the layers of the networks at 1-64
// samples with a cold L2: up to 400 tiles of 32 x 32 (one or two per CU) it wins or draws; beyond, operands that are used once per load
// cost more than the staged kernel's chain.  16 x 16 tiles while those of 32 would leave half of the chip idle; four wavefronts are the
// best or within 5 % of it, but for long reductions in a full round, where eight and twice the channels per activation load are.
int conv_skinny_default(const ConvArgs& a, int es)
{
    if (!a.wo || a.mode != 0 || es != 1 || !skinny_reaches(a, es)) return 0;          // bf16 by default: one order of summation, that of the staged kernels
    const long long kbytes = (long long)a.kh * a.kw * a.Ci * es;
    const long long tiles = (long long)((a.M + 31) / 32) * ((a.Co + 31) / 32);
    if (tiles > (kbytes > 128 ? 400 : 200)) return 0;
    if (tiles <= 100 && kbytes > 128) return skinny_cfg(16, 1, 2);
    if (tiles > 200 && kbytes > 640) return skinny_cfg(32, 2, 3);
    return skinny_cfg(32, 1, 2);
}

// bf16, tuned: the word whose wavefronts a layer's reduction is shared by, or 0: the order of summation of the staged kernels.  By the shape alone, so that a timing cannot change an answer.  Measured with
// every configuration over the layers of the ResNet-50, ResNet-18, Inception and MobileNetV2 networks in bf16 at 1-64 samples with a cold L2, sums over a network at 1, 4, 16 and 64 samples against the fastest
// configuration of any order: this rule 1.00-1.02, 1.00-1.01, 1.00-1.01 and 1.00 (ResNet-50), always the staged kernels' order 1.42, 1.16, 1.03 and 1.00, always 16 x 16 tiles and four wavefronts 1.04, 1.09, 1.03, 1.00,
// always 32 x 32 and two 1.17, 1.00, 1.01, 1.00.
int conv_skinny_order_bf16(const ConvArgs& a)
{
    if (!a.wo || a.mode != 0 || a.M > EE_SKINNY_MAX_ROWS || !skinny_reaches(a, 2)) return 0;
    const int kbytes = a.kh * a.kw * a.Ci * 2;
    const long long tiles = (long long)((a.M + 31) / 32) * ((a.Co + 31) / 32);
    if (tiles <= 130) return kbytes >= 128 ? skinny_cfg(16, 1, 2) : 0;
    return tiles <= (kbytes > 2048 ? 600 : kbytes > 128 ? 400 : 0) ? skinny_cfg(32, 1, 1) : 0;
}

template <int ES>
hipError_t launch_conv_skinny(const ConvArgs& a, int cfg, hipStream_t s)
{
    if (a.M <= 0) return hipSuccess;
    if (!a.wo || a.mode != 0 || !conv_skinny_config_ok(cfg)) return hipErrorInvalidValue;
    const int lw = skinny_waves(cfg);
    if (cfg >> 12 == 4) {
        if (lw == 2) return launch_skinny<ES, 16, 4, 1>(a, s);
        if (lw == 3) return launch_skinny<ES, 16, 8, 1>(a, s);
        return launch_skinny<ES, 16, 16, 1>(a, s);
    }
    if (((cfg >> 4) & 15) == 2) {
        if (lw == 0) return launch_skinny<ES, 32, 1, 2>(a, s);
        if (lw == 1) return launch_skinny<ES, 32, 2, 2>(a, s);
        if (lw == 2) return launch_skinny<ES, 32, 4, 2>(a, s);
        return launch_skinny<ES, 32, 8, 2>(a, s);
    }
    if (lw == 0) return launch_skinny<ES, 32, 1, 1>(a, s);
    if (lw == 1) return launch_skinny<ES, 32, 2, 1>(a, s);
    if (lw == 2) return launch_skinny<ES, 32, 4, 1>(a, s);
    if (lw == 3) return launch_skinny<ES, 32, 8, 1>(a, s);
    return launch_skinny<ES, 32, 16, 1>(a, s);
}

template hipError_t launch_conv_skinny<1>(const ConvArgs&, int, hipStream_t);
template hipError_t launch_conv_skinny<2>(const ConvArgs&, int, hipStream_t);

}  // namespace ee
