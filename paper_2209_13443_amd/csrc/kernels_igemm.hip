// The staged implicit-GEMM convolution (igemm_kernel.hpp), one layer per launch.
#include "igemm_kernel.hpp"

namespace ee {

// Two wavefronts per SIMD as the least (here and in the other kernels of one layer, of layers side by side and of a pair; fused blocks, seams and the convolution with its pool have bounds of their own): a wavefront then has at most 256 registers, and the compiler keeps the accumulators where
// ordinary instructions read them; allowed 512 it put them into the other half of the file, an instruction per value away (1x1, 64 -> 256, 56x56, 64 samples 17.1 -> 15.2 us).
template <int ES, int BM, int BN, int KS, int KSPL, bool PLAIN>
__global__ __launch_bounds__(256 * KSPL, 2) void conv_igemm_kernel(ConvArgs a, int gm, int gn, unsigned magic_gn, int ns)
{
    igemm_tile<ES, BM, BN, KS, KSPL, PLAIN>(a, gm, gn, magic_gn, ns, blockIdx.x);
}

// ---- launch ------------------------------------------------------------------------------------------------
template <int ES, int BM, int BN, int KS, int KSPL>
static hipError_t launch_igemm_tile(const ConvArgs& a, bool plain, int ns, hipStream_t s)
{
    const int gm = (a.M + BM - 1) / BM, gn = (a.Co + BN - 1) / BN;
    const dim3 grid(xcd_grid(gm) * (unsigned)gn);
    const unsigned magic_gn = (unsigned)(0x100000000ull / (unsigned)gn - (gn == 1));
    ns = ns < 2 ? 2 : (ns > 4 ? 4 : ns);
    while (ns > 2 && igemm_lds_bytes<ES, BM, BN, KS, KSPL>(a, ns) > 160 * 1024) --ns;      // the deepest ring that fits
    const size_t lds_bytes = igemm_lds_bytes<ES, BM, BN, KS, KSPL>(a, ns);
    // more than 64 KiB of dynamic LDS has to be granted once per kernel
    static const hipError_t granted = [] {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_igemm_kernel<ES, BM, BN, KS, KSPL, true>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_igemm_kernel<ES, BM, BN, KS, KSPL, false>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        return e;
    }();
    if (granted != hipSuccess) return granted;
    if (lds_bytes > 160 * 1024) return hipErrorInvalidValue;
    if (plain)
        EE_LAUNCH((conv_igemm_kernel<ES, BM, BN, KS, KSPL, true>), grid, dim3(256 * KSPL), lds_bytes, s, a, gm, gn, magic_gn, ns);
    else
        EE_LAUNCH((conv_igemm_kernel<ES, BM, BN, KS, KSPL, false>), grid, dim3(256 * KSPL), lds_bytes, s, a, gm, gn, magic_gn, ns);
    return hipGetLastError();
}

// The configuration of an untuned launch, from the size of the problem alone.  Measured with every configuration over the layers of the
// ResNet-50 / ResNet-18, MobileNetV2 and Inception networks at 1-256 samples, each launch behind the layer in front of it and with a cold
// L2; the rule stays within 3-8 % of the best configuration over a network:
//   reductions up to 640 bytes: a tile is over in a few steps and what counts is copies in flight, i.e. many small workgroups on a CU:
//     64-byte steps, 64 x 128 tiles once there are two rounds of 64 x 64 ones, which a bf16 residual tile's LDS would cost (64 x 64 there);
//   longer ones: while the 64 x 64 tiles do not fill the chip, the steps are a serial chain and the fewest, longest win; then tiles grow
//     with the number of them (blocks: 64 x 64 tiles of the output), 128 x 128 from four per CU; channels that would leave half of a
//     128-channel tile empty take 64-channel ones.
int conv_igemm_default(const ConvArgs& a, int es, long long blocks)
{
    const int kbytes = a.kh * a.kw * a.Ci * es;
    const bool narrow = a.Co <= 64;
    if (kbytes <= 640) {
        if (kbytes > 256 && blocks < 256) return 0x423;
        if (narrow) return a.kh * a.kw == 1 || blocks < 1024 ? 0x313 : 0x212;
        if (es == 2 && (a.res || kbytes <= 128)) return 0x313;
        return blocks >= 512 ? 0x214 : 0x313;
    }
    if (blocks < 256) return 0x333;
    if (blocks < 512) return kbytes > 1280 ? 0x334 : 0x323;
    if (narrow) return 0x222;
    if (blocks < 1024) return kbytes > 1280 ? 0x324 : 0x322;
    if (es == 2 && a.res) return 0x313;
    if ((a.Co + 127) / 128 * 128 - a.Co >= 64) return 0x322;
    return blocks < 2048 || kbytes > 1280 ? 0x221 : 0x222;
}

// cfg: bits 0-3 tile (1: 128x128, 2: 128x64, 3: 64x64, 4: 64x128), bits 4-7 reduction step (1: 64, 2: 128, 3: 256 bytes), bits 8-11 ring
// stages (2..4), bits 12-15 wavefront groups splitting the reduction inside a workgroup (0 or 1: none, 2, 4); 0 in the first three
// = by shape.  Not every combination exists: hipErrorInvalidValue for one that does not (or does not fit LDS).
template <int ES>
hipError_t launch_conv_igemm(const ConvArgs& a_in, int cfg, hipStream_t s)
{
    if (a_in.M <= 0) return hipSuccess;
    const int kbytes = a_in.kh * a_in.kw * a_in.Ci * ES;
    const int by_shape = conv_igemm_default(a_in, ES, (long long)((a_in.M + 63) / 64) * ((a_in.Co + 63) / 64));
    if (cfg == 0) cfg = by_shape;
    int tile = cfg & 15, ksel = (cfg >> 4) & 15, ns = (cfg >> 8) & 15, kspl = (cfg >> 12) & 15;
    if (tile == 0) tile = by_shape & 15;
    if (ksel == 0) ksel = kbytes % 128 == 0 ? 2 : 1;
    if (ns == 0) ns = 2;
    const int ks = ksel == 3 ? 256 : (ksel == 2 ? 128 : 64);
    // PLAIN: every reduction step of a row is one contiguous, always valid run of ks bytes: a 1x1 kernel whose
    // pixel is a multiple of the step (the address advances by the step), or an unpadded stride-1 kernel whose
    // kernel row is exactly one step (the address advances by one image row)
    ConvArgs a = a_in;
    const bool plain_1x1 = a.kh == 1 && a.kw == 1 && a.pad == 0 && a.pad_w == 0 && kbytes % ks == 0;
    const bool plain_rows = !plain_1x1 && a.pad == 0 && a.pad_w == 0 && a.stride == 1 && a.kw * a.Ci * ES == ks;
    const bool plain = plain_1x1 || plain_rows;
    a.plain_step = plain_rows ? a.W * a.Ci * ES : ks;
    if (kspl >= 2) {          // measured to pay only for small tiles with the longest step
        if (kspl == 2 && ks == 256 && tile == 3) return launch_igemm_tile<ES, 64, 64, 256, 2>(a, plain, ns, s);
        if (kspl == 2 && ks == 256 && tile == 4) return launch_igemm_tile<ES, 64, 128, 256, 2>(a, plain, ns, s);
        if (kspl == 4 && ks == 256 && tile == 3) return launch_igemm_tile<ES, 64, 64, 256, 4>(a, plain, ns, s);
        return hipErrorInvalidValue;
    }
    if (ks == 256) {
        if (tile == 1) return launch_igemm_tile<ES, 128, 128, 256, 1>(a, plain, ns, s);
        if (tile == 2) return launch_igemm_tile<ES, 128, 64, 256, 1>(a, plain, ns, s);
        if (tile == 4) return launch_igemm_tile<ES, 64, 128, 256, 1>(a, plain, ns, s);
        return launch_igemm_tile<ES, 64, 64, 256, 1>(a, plain, ns, s);
    }
    if (ks == 128) {
        if (tile == 1) return launch_igemm_tile<ES, 128, 128, 128, 1>(a, plain, ns, s);
        if (tile == 2) return launch_igemm_tile<ES, 128, 64, 128, 1>(a, plain, ns, s);
        if (tile == 4) return launch_igemm_tile<ES, 64, 128, 128, 1>(a, plain, ns, s);
        return launch_igemm_tile<ES, 64, 64, 128, 1>(a, plain, ns, s);
    }
    if (tile == 1) return launch_igemm_tile<ES, 128, 128, 64, 1>(a, plain, ns, s);
    if (tile == 2) return launch_igemm_tile<ES, 128, 64, 64, 1>(a, plain, ns, s);
    if (tile == 4) return launch_igemm_tile<ES, 64, 128, 64, 1>(a, plain, ns, s);
    return launch_igemm_tile<ES, 64, 64, 64, 1>(a, plain, ns, s);
}

template hipError_t launch_conv_igemm<1>(const ConvArgs&, int, hipStream_t);
template hipError_t launch_conv_igemm<2>(const ConvArgs&, int, hipStream_t);

}  // namespace ee
