// Several independent int8 convolutions in one launch: the branches of a concatenating block, a block's first layer and the convolution
// on its shortcut.
//
// Each of them alone is a launch of a few microseconds of work behind 1.7 us of dispatch, 1-2 us of ramp (first operands from the last-level
// cache) and a tail in which the chip runs empty; together they share those.  The workgroups of the layers follow one another in the
// grid (per XCD, so that every layer keeps its eighths of the batch), or, where all of them read one input and have reductions of one length, take turns in rounds over the same part of the
// batch: the input, 51 MB in front of a first layer and its shortcut, comes from memory once and out of the XCD's L2 for the others (ResNet-50, 256 -> 128 and 256 -> 512 / 2 and so on, 64 slots, 10,000
// requests 55.5 -> 54.1 ms).  Reductions of other lengths in turns leave the long ones for the end: Inception-style stream 29.1 -> 30.0 ms, static batches of ResNet-18 6.2 -> 6.45.  Every workgroup runs the tile of the single-layer kernels
// (igemm_kernel.hpp, skinny_kernel.hpp: same arithmetic, same results) with its layer's arguments, picked out of the kernel-argument
// segment with scalar loads.  All layers of a launch share one configuration.
#include "igemm_kernel.hpp"
#include "skinny_kernel.hpp"

namespace ee {

struct GroupMember {
    ConvArgs a;
    int gm, gn;
    unsigned magic_gn;
    int first;           // where the layer's share of a round begins (in workgroups of eight: one per XCD); skinny tiles: workgroups of the layers in front
    int share;           // its workgroups of a round
    int nk, pitch;
};
struct ConvGroup { GroupMember m[EE_GROUP_MAX]; };
static_assert(sizeof(GroupMember) % 4 == 0);

// the member a workgroup belongs to (slot: its number in units of GroupMember::first), uniform
__device__ __forceinline__ int group_pick(const ConvGroup& g, int n, int slot)
{
    int i = 0;
#pragma unroll
    for (int k = 1; k < EE_GROUP_MAX; ++k) i = k < n && slot >= g.m[k].first ? k : i;
    return i;
}

// member i of the launch's first argument
__device__ __forceinline__ GroupMember group_member(int i)
{
    typedef const __attribute__((address_space(4))) unsigned* words_t;
    constexpr int W = sizeof(GroupMember) / 4;
    const words_t p = (words_t)__builtin_amdgcn_kernarg_segment_ptr() + i * W;
    union { GroupMember m; unsigned w[W]; } u;
#pragma unroll
    for (int k = 0; k < W; ++k) u.w[k] = p[k];
    GroupMember m = u.m;
    // device memory all of them (the compiler knows that of ordinary kernel arguments, not of these)
    auto global = [](auto*& q) {
        using P = std::remove_reference_t<decltype(q)>;
        q = (P)(__attribute__((address_space(1))) std::remove_pointer_t<P>*)(unsigned long long)q;
    };
    global(m.a.x); global(m.a.w); global(m.a.bias); global(m.a.res); global(m.a.y); global(m.a.wo); global(m.a.zeros);
    global(m.a.gap_sums); global(m.a.xs); global(m.a.ys);
    return m;
}

// round: workgroups (of eight) of a round, in which every layer has its share of tiles, all of the same part of the batch
template <int BM, int BN, int KS, bool PLAIN>
__global__ __launch_bounds__(256, 2) void conv_group_kernel(ConvGroup g, int n, int ns, unsigned round, unsigned magic_round)
{
    const unsigned slot = blockIdx.x >> 3, t = fast_div(slot, round, magic_round);
    const int at = (int)(slot - t * round);
    const GroupMember m = group_member(group_pick(g, n, at));
    igemm_tile<1, BM, BN, KS, 1, PLAIN>(m.a, m.gm, m.gn, m.magic_gn, ns, (t * (unsigned)m.share + (unsigned)(at - m.first)) << 3 | (blockIdx.x & 7));
}

template <int T, int NW, int TN, bool PLAIN>
__global__ __launch_bounds__(64 * NW, 2) void conv_group_skinny_kernel(ConvGroup g, int n)
{
    const GroupMember m = group_member(group_pick(g, n, (int)blockIdx.x));
    skinny_tile<1, T, NW, TN, PLAIN ? SKINNY_PLAIN : SKINNY_ANY>(m.a, m.gn, m.magic_gn, m.nk, m.pitch, blockIdx.x - (unsigned)m.first);
}

template <int T, int NW, int TN>
__global__ __launch_bounds__(64 * NW, 2) void conv_group_skinny_taps_kernel(ConvGroup g, int n)
{
    const GroupMember m = group_member(group_pick(g, n, (int)blockIdx.x));
    skinny_tile<1, T, NW, TN, SKINNY_TAPS>(m.a, m.gn, m.magic_gn, m.nk, m.pitch, blockIdx.x - (unsigned)m.first);
}

// ---- launch ------------------------------------------------------------------------------------------------
template <int BM, int BN, int KS>
static hipError_t launch_group_tile(const ConvArgs* a, int n, int ns, hipStream_t s)
{
    ConvGroup g{};
    bool plain = true;
    for (int i = 0; i < n; ++i) plain &= a[i].kh == 1 && a[i].kw == 1 && a[i].pad == 0 && a[i].pad_w == 0 && a[i].Ci % KS == 0;
    size_t lds_bytes = 0;
    for (int i = 0; i < n; ++i) {
        GroupMember& m = g.m[i];
        m.a = a[i];
        m.a.plain_step = KS;
        m.gm = (a[i].M + BM - 1) / BM; m.gn = (a[i].Co + BN - 1) / BN;
        m.magic_gn = (unsigned)(0x100000000ull / (unsigned)m.gn - (m.gn == 1));
    }
    bool alike = true;                                      // one input, reductions of one length
    for (int i = 1; i < n; ++i) alike &= a[i].x == a[0].x && a[i].kh * a[i].kw * a[i].Ci == a[0].kh * a[0].kw * a[0].Ci;
    auto tiles = [&](int i) { return (long long)xcd_grid(g.m[i].gm) / 8; };      // of pixels, on an XCD
    long long least = tiles(0), rounds = 0, round = 0;
    for (int i = 1; i < n; ++i) least = std::min(least, tiles(i));
    for (int i = 0; i < n; ++i) {
        const long long per_round = alike ? std::max(1ll, (tiles(i) + least / 2) / std::max(1ll, least)) : tiles(i);
        rounds = std::max(rounds, (tiles(i) + per_round - 1) / per_round);
        g.m[i].first = (int)round;
        g.m[i].share = (int)(per_round * g.m[i].gn);
        round += g.m[i].share;
    }
    const long long total = rounds * round;
    if (total > 0xfffffff) return hipErrorInvalidValue;
    const unsigned magic_round = (unsigned)(0x100000000ull / (unsigned)round - (round == 1));
    for (;; --ns) {                                         // the deepest ring that fits
        lds_bytes = 0;
        for (int i = 0; i < n; ++i) lds_bytes = std::max(lds_bytes, igemm_lds_bytes<1, BM, BN, KS, 1>(a[i], ns));
        if (ns == 2 || lds_bytes <= 160 * 1024) break;
    }
    static const hipError_t granted = [] {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_group_kernel<BM, BN, KS, true>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_group_kernel<BM, BN, KS, false>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        return e;
    }();
    if (granted != hipSuccess) return granted;
    if (lds_bytes > 160 * 1024) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total * 8);
    if (plain) EE_LAUNCH((conv_group_kernel<BM, BN, KS, true>), grid, dim3(256), lds_bytes, s, g, n, ns, (unsigned)round, magic_round);
    else EE_LAUNCH((conv_group_kernel<BM, BN, KS, false>), grid, dim3(256), lds_bytes, s, g, n, ns, (unsigned)round, magic_round);
    return hipGetLastError();
}

template <int T, int NW, int TN>
static hipError_t launch_group_skinny(const ConvArgs* a, int n, hipStream_t s)
{
    constexpr int KB = 1024 / T;
    ConvGroup g{};
    bool plain = true, taps = true;                         // every member 1x1 without padding; of whole steps to a tap
    long long total = 0;
    for (int i = 0; i < n; ++i) {
        if (!a[i].wo || !skinny_reaches(a[i], 1)) return hipErrorInvalidValue;
        GroupMember& m = g.m[i];
        m.a = a[i];
        m.gm = (a[i].M + T - 1) / T; m.gn = (a[i].Co + T * TN - 1) / (T * TN);
        m.magic_gn = (unsigned)(0x100000000ull / (unsigned)m.gn - (m.gn == 1));
        m.first = (int)total;
        m.nk = (a[i].kh * a[i].kw * a[i].Ci + KB - 1) / KB;
        m.pitch = a[i].Kp / 32;
        total += (long long)m.gm * m.gn;
        const int mode = skinny_mode(m.a, 1, T);
        plain &= mode == SKINNY_PLAIN;
        taps &= mode != SKINNY_ANY;
    }
    if (total > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total), block(64 * NW);
    if (plain) EE_LAUNCH((conv_group_skinny_kernel<T, NW, TN, true>), grid, block, 0, s, g, n);
    else if (taps) EE_LAUNCH((conv_group_skinny_taps_kernel<T, NW, TN>), grid, block, 0, s, g, n);
    else EE_LAUNCH((conv_group_skinny_kernel<T, NW, TN, false>), grid, block, 0, s, g, n);
    return hipGetLastError();
}

bool conv_group_config_ok(int cfg)
{
    for (const int sk : {skinny_cfg(16, 1, 2), skinny_cfg(16, 1, 3), skinny_cfg(32, 1, 2), skinny_cfg(32, 1, 3), skinny_cfg(32, 2, 2), skinny_cfg(32, 2, 3)})
        if (cfg == sk) return true;
    const int tile = cfg & 15, ksel = (cfg >> 4) & 15, ns = (cfg >> 8) & 15;
    return cfg > 0 && !(cfg >> 12) && tile >= 1 && tile <= 4 && ksel >= 1 && ksel <= 3 && ns >= 2 && ns <= 4;
}

// cfg: a configuration word of the staged kernel (without wavefront groups) or of the one for few pixels; hipErrorInvalidValue for
// one that is not instantiated here
hipError_t launch_conv_group(const ConvArgs* a, int n, int cfg, hipStream_t s)
{
    if (n < 1 || n > EE_GROUP_MAX || cfg <= 0 || (cfg >> 16)) return hipErrorInvalidValue;
    for (int i = 0; i < n; ++i)
        if (a[i].M <= 0 || a[i].mode != 0) return hipErrorInvalidValue;
    if (cfg == skinny_cfg(16, 1, 2)) return launch_group_skinny<16, 4, 1>(a, n, s);
    if (cfg == skinny_cfg(16, 1, 3)) return launch_group_skinny<16, 8, 1>(a, n, s);
    if (cfg == skinny_cfg(32, 1, 2)) return launch_group_skinny<32, 4, 1>(a, n, s);
    if (cfg == skinny_cfg(32, 1, 3)) return launch_group_skinny<32, 8, 1>(a, n, s);
    if (cfg == skinny_cfg(32, 2, 2)) return launch_group_skinny<32, 4, 2>(a, n, s);
    if (cfg == skinny_cfg(32, 2, 3)) return launch_group_skinny<32, 8, 2>(a, n, s);
    const int tile = cfg & 15, ksel = (cfg >> 4) & 15, ns = (cfg >> 8) & 15;
    if (cfg >> 12 || ns < 2 || ns > 4) return hipErrorInvalidValue;
#define EE_GROUP_TILE(T_, BM_, BN_) \
    if (tile == T_) return ksel == 1 ? launch_group_tile<BM_, BN_, 64>(a, n, ns, s) : ksel == 2 ? launch_group_tile<BM_, BN_, 128>(a, n, ns, s) \
                         : ksel == 3 ? launch_group_tile<BM_, BN_, 256>(a, n, ns, s) : hipErrorInvalidValue;
    EE_GROUP_TILE(1, 128, 128) EE_GROUP_TILE(2, 128, 64) EE_GROUP_TILE(3, 64, 64) EE_GROUP_TILE(4, 64, 128)
#undef EE_GROUP_TILE
    return hipErrorInvalidValue;
}

}  // namespace ee
