// Launcher of the bf16-piece convolution (conv_split.h): the instances, and the rule that picks one or
// leaves the layer to the fp32 pipeline (conv_mfma_fast.hip).
#include "conv_split.h"
#include "runtime_cache.h"

#include <algorithm>

namespace im2win {

// Fills the parameters for tiles of TN pixels: the strip width that needs the fewest patch positions.
// False when the patch does not fit what the instance reserves or an offset does not fit 31 bits.
template <int HF, int WF, int CFG>
static bool split_params(SplitParams &Q, const MfmaParams &P, const Shape &sh, bool implicit, size_t *lds)
{
    using KC = SplitK<HF, WF, CFG>;
    using T = SplitTile<KC::SHAPE>;
    constexpr int TM = T::WGM * T::FM * 32, TN = T::WGN * T::FN * 32;
    constexpr int smax = split_positions<HF, WF, CFG>() - 2;
    // (Both calls ask for what either needs, so that they take the same kernel and give the same bits.)
    if (sh.s > 65536) return false;
    // (Strided layers of which only 8 channels at a time fit stay on the fp32 pipeline.  In us, fp32 pipeline / pieces: 3x3 stride 2
    // 128 -> 128 at 56x56, N=32 68 / 79; 64 -> 64 at 112x112, N=128 309 / 319; 256 -> 256 at 28x28, N=64 110 / 131; 90 -> 26 at 41x41,
    // N=86 46 / 54; 5x5 stride 2 64 -> 64 at 56x56, N=16 29 / 61; 96 -> 128 at 48x48, N=64 170 / 187.  Not everywhere: 3x3 56 -> 201 at
    // 94x94, N=28 251 / 125, 5x5 48 -> 96 at 56x56, N=128 208 / 151, which the estimates below do not tell from the others.)
    if (CFG == 2 && HF == WF && HF <= 5 && HF != 4 && sh.s > 1) return false;
    const int rstep = std::max(1, HF / sh.s);
    long long best = -1, best_img = 0;
    int tried = 0;
    for (int want : {512, 64, 48, 32, 28, 24, 16, 12, 8}) {
        const int ns = (sh.Wo - 1) / want + 1;
        if (ns == tried) continue;   // (the widths follow from the number of strips)
        tried = ns;
        const int w = (sh.Wo - 1) / ns + 1, wl = sh.Wo - (ns - 1) * w;
        if (wl < 1 || wl < w / 2) continue;
        const long long PW = (long long)(w - 1) * sh.s + WF;
        if (std::min<long long>(sh.Wi, (long long)(wl - 1) * sh.s + WF - sh.p) < 4) continue;   // runs of at least four words
        long long need = 0, imgs = 0, items = 0;
        for (int ww : {w, wl}) {
            const long long R = std::min<long long>((TN + ww - 2) / ww + 1, (long long)sh.N * sh.Ho);
            const long long I = std::min<long long>((R + sh.Ho - 2) / sh.Ho + 1, sh.N);
            const long long pw = (long long)(ww - 1) * sh.s + WF, rows = (R - 1) * sh.s + HF + (I - 1) * std::max(0, HF - sh.s);
            const long long reads = (R - I + (rstep - 1) * I) / rstep + I;
            need = std::max(need, rows * PW);
            imgs = std::max(imgs, I);
            items = std::max(items, KC::CG * std::max(rows * ((pw + 3) / 4), reads * ((pw * HF + 3) / 4)));
        }
        if (need > smax || items > KC::JQ * KC::PW * 64 || (best >= 0 && need >= best)) continue;
        best = need; best_img = imgs;
        Q.w = w; Q.wl = wl; Q.nstrips = ns; Q.PW = (int)PW;
    }
    if (best < 0) return false;
    const unsigned long long plane = implicit ? (unsigned long long)sh.Hi * sh.Wi : (unsigned long long)sh.Ho * sh.rowlen;
    const unsigned long long larger = std::max((unsigned long long)sh.Hi * sh.Wi, (unsigned long long)sh.Ho * sh.rowlen);
    if ((unsigned long long)best_img * sh.Ci * larger * 4ull >= (1ull << 31)) return false;
    if ((unsigned long long)sh.K * 4ull * TM >= (1ull << 31)) return false;
    if (((unsigned long long)sh.Co * best_img + 64ull) * (unsigned long long)sh.Ho * sh.Wo * 4ull >= kNoStore) return false;
    const long long LF = (long long)(sh.Ho - 1) * sh.s + HF;
    if (LF > INT32_MAX / 2) return false;
    Q.src = P.win; Q.flt = P.flt; Q.out = P.out;
    Q.N = sh.N; Q.Ci = sh.Ci; Q.Ho = sh.Ho; Q.Wo = sh.Wo; Q.Co = sh.Co; Q.s = sh.s; Q.K = sh.K;
    Q.Hi = sh.Hi; Q.Wi = sh.Wi; Q.p = sh.p; Q.rowlen = sh.rowlen;
    Q.plane = (uint32_t)plane; Q.howo = P.howo; Q.src_elems = P.win_elems; Q.out_elems = P.out_elems;
    Q.tiles_m = (sh.Co + TM - 1) / TM;
    const uint32_t rows = (uint32_t)(sh.N * sh.Ho);
    const uint32_t tiles_s = (rows * (uint32_t)Q.w + TN - 1) / TN;
    Q.tiles_l = (rows * (uint32_t)Q.wl + TN - 1) / TN;
    Q.nblocks = (tiles_s * (uint32_t)(Q.nstrips - 1) + Q.tiles_l) * (uint32_t)Q.tiles_m;
    Q.LF = (int)LF; Q.npos = (int)best;
    Q.d_w = make_fastdiv((uint32_t)Q.w); Q.d_wl = make_fastdiv((uint32_t)Q.wl); Q.d_ho = make_fastdiv((uint32_t)sh.Ho);
    Q.rstep = rstep; Q.GF = (sh.Ho - 1 + rstep - 1) / rstep + 1;
    Q.d_rs = make_fastdiv((uint32_t)rstep); Q.d_gf = make_fastdiv((uint32_t)Q.GF); Q.d_pw = make_fastdiv((uint32_t)Q.PW); Q.d_lf = make_fastdiv((uint32_t)LF);
    Q.d_tm = make_fastdiv((uint32_t)Q.tiles_m); Q.d_ns = make_fastdiv((uint32_t)Q.nstrips); Q.d_ns1 = make_fastdiv((uint32_t)std::max(1, Q.nstrips - 1));
    *lds = 2 * (size_t)(2 * KC::KS) * split_a_plane(TM) + (size_t)KC::CG * (smax + 2) * 48 + kPassBytes;
    return true;
}

template <int HF, int WF, int CFG, bool IMP>
__global__ __launch_bounds__((split_threads<HF, WF, CFG>()), (split_threads<HF, WF, CFG>() / 256)) void conv_split_kernel(SplitParams P)
{
    extern __shared__ __align__(16) unsigned char smem[];
    conv_split_body<HF, WF, CFG, IMP>(P, smem);
}

template <int HF, int WF, int CFG, bool IMP>
static hipError_t launch_split_t(const SplitParams &Q, size_t lds, int dev, int ncu, hipStream_t st, LaunchPlan *plan)
{
    constexpr int NT = split_threads<HF, WF, CFG>();
    const uint32_t grid = std::min(Q.nblocks, (uint32_t)ncu);   // one workgroup per compute unit; it takes every grid-th tile
    if (plan) {
        plan_record(plan, dim3(grid), NT, lds, "conv_split_kernel<%d, %d, %d, %s>", HF, WF, CFG, IMP ? "true" : "false");
        return hipSuccess;
    }
    void (*kern)(SplitParams) = &conv_split_kernel<HF, WF, CFG, IMP>;
    static KernelCache kc;
    const hipError_t e = allow_dynamic_lds(kc, reinterpret_cast<const void *>(kern), lds, dev);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), lds, st, Q);
    return hipGetLastError();
}

// What the layer takes on the fp32 matrix cores, in us: 64x64 tiles of the pipelined kernel, whose 3x3 and 5x5 instances cut leftover
// tiles into halves or sixteenths and which runs over tile boundaries where K is short and the channels are whole tiles (10 % off, root
// mean square, on 1440 layers).  Strips longer than its instances take (images of a few pixels a row, wide strides) leave the layer to the
// generic kernels, at a quarter of the rate: 7x7 stride 2 20 -> 59 channels 55x55 N=27 105 us, pieces 27.  By sizes alone, so that both
// calls take the same body.
template <int HF, int WF>
static double fp32_estimate(const MfmaParams &P, const Shape &sh, uint32_t blocks, int ncu)
{
    constexpr int CB = HF == 3 && WF == 3 ? 8 : HF == 5 ? 4 : HF == 7 && WF == 7 ? 2 : HF == 4 ? 4 : HF * WF == 7 ? 8 : 16;
    constexpr int LONGEST = HF * WF == 3 ? 256 : HF == 7 && WF == 7 ? 1024 : HF == 5 || HF == 4 ? 768 : 512;
    constexpr uint32_t RESIDENT = (HF == 3 && WF == 3) || (HF == 1 && WF == 7) ? 3 : 2;   // workgroups per compute unit
    const double r = (double)blocks / ncu, up = (double)((blocks + ncu - 1) / ncu);
    if (P.S > LONGEST) return 4.0 + std::max(0.5 * (r + up), 0.6) * (double)sh.K * 0.055;
    const int nkb = (sh.Ci + CB - 1) / CB;
    const bool whole = sh.Ci % CB == 0, pieces = HF == 3 && WF == 3 && sh.Ci % 16 == 0;
    const double k = (double)(nkb * CB * HF * WF);
    if (HF == 3 && WF == 3 && few_tiles_in_sixteenths(P, blocks, ncu))   // (13 % off, in two calls)
        return 3.1 + sh.Ci * (0.027 + (16 * blocks > (uint32_t)ncu ? 0.031 * (double)((P.npix + 15) / 16) * ((P.Co + 15) / 16) / ncu : 0.0));
    if (HF == WF && HF <= 5 && sh.Ci >= 8 && (uint32_t)((sh.npix + 31) / 32) * (uint32_t)((sh.Co + 31) / 32) <= (uint32_t)ncu)
        return 3.4 + (double)((sh.Ci + 7) / 8 * 8 * HF * WF) * 0.0048;   // quarter tiles
    double rounds = 0.9 * up + 0.1 * std::max(r, up > 1.5 ? 0.0 : 0.84);
    if (whole && nkb % 2 == 0 && nkb <= 12 && sh.Co % MB == 0 && blocks >= 3 * RESIDENT * (uint32_t)ncu) {
        rounds = r;
    } else if (HF == WF && (HF == 3 || HF == 5)) {
        const uint32_t left = blocks % (uint32_t)ncu;
        if (pieces && left <= (uint32_t)ncu / 8) rounds = (double)(blocks / ncu) + (left ? 0.42 : 0.0);
        else if (left <= (uint32_t)ncu / 2) rounds = (double)(blocks / ncu) + (left ? 0.55 : 0.0);
        else if (pieces && left <= (uint32_t)(ncu / 2 + ncu / 8)) rounds = (double)(blocks / ncu) + 0.65;
    }
    // (One K block, at most 32 channels and more than four rounds: a tile ends with the stores of two waves of four, and others begin beside it.
    // 8 -> 23 45x45 N=78 18.4 us, 20.7 in pieces; twelve such layers 1.03 to 1.17 times as fast as in pieces, eighteen of three to four rounds 0.90 to 1.01.)
    const bool brief = HF == 3 && WF == 3 && nkb == 1 && P.S <= 256 && sh.Co <= 32 && blocks > 4 * (uint32_t)ncu;
    return 3.75 + rounds * (k * 0.0151 + (brief ? 0.72 : 0.92));
}

// hipErrorNotSupported where no tile shape fits or the fp32 pipeline is the faster one.
template <int HF, int WF, bool IMP>
static hipError_t launch_split(const MfmaParams &P, const Shape &sh, uint32_t blocks, hipStream_t st, LaunchPlan *plan)
{
    int dev = 0, ncu = 0;
    hipError_t e = device_cus(&dev, &ncu);
    if (e != hipSuccess && plan) { e = hipSuccess; ncu = 256; }   // planning without a device: an MI355X's 256 compute units
    if (e != hipSuccess) return e;
    // Which is faster: estimates in us, fitted to 1600 layers of 3x3, 5x5, 7x7, 4x4, 1x7, 7x1, 1x3 and 3x1 filters with 4 to 512 channels, odd
    // sizes and those of usual networks (7 % off, root mean square; the pick takes 1.007 times the best body's time on average, 1.3 at
    // worst).  A body takes its start and end, and per round of tiles the tile's steps and its own start and stores.  Measured, fp32
    // pipeline / wide / narrow / low: 3x3 64 channels 56x56 N=32 62 / 48 / 58 / 57; 3x3 256 channels 14x14 N=128 213 / 140 / 183 / 181;
    // 3x3 512 channels 7x7 N=128 151 / 160 / 101 / 95; 3x3 100 -> 130 29x27 N=61 130 / 99 / 101 / 88; 5x5 96 -> 100 24x24 N=50
    // - / 68 / 94 / 81; 7x7 stride 2 64 -> 20 134x134 N=16 - / 104 / 129 / 74.  Strided 1x7 layers read rows that their windows skip and take a
    // tenth longer, without a workspace above all (16 -> 64 123x123 stride 2 N=106, fp32 / narrow, two calls and workspace-free: 64 / 71 and 68 / 82; 120
    // layers on whose kernel that decides: fp32 1.01 and 1.16 times as fast as the pieces).
    // `mix`: how far a last round that leaves units idle counts in full (it runs at a higher clock).
    auto rounds = [&](uint32_t tiles, double mix) {
        const double r = (double)tiles / ncu, up = (double)((tiles + ncu - 1) / ncu);
        return mix * up + (1.0 - mix) * std::max(r, up > 1.5 ? 0.0 : 0.6);
    };
    const double old = fp32_estimate<HF, WF>(P, sh, blocks, ncu);
    if (old < 9.0) return hipErrorNotSupported;   // (nothing below starts and ends in less)
    SplitParams Q[5];
    size_t lds[5];
    int pick = -1;
    double least = 0.93 * old;
    auto consider = [&](auto cfg) {
        constexpr int CFG = decltype(cfg)::value;
        using KC = SplitK<HF, WF, CFG>;
        using T = SplitTile<KC::SHAPE>;
        constexpr int TM = T::WGM * T::FM * 32, TN = T::WGN * T::FN * 32;
        const double steps = (double)((sh.Ci + 8 * KC::CG - 1) / (8 * KC::CG)) * ((KC::CG * HF * WF + 1) / 2);
        const bool strided = HF == 1 && WF == 7 && sh.s > 1;
        constexpr bool SHORT = HF * WF == 3 || (HF == 4 && WF == 4);   // short K blocks, more patch to a step
        auto time = [&](uint32_t tiles) {
            return KC::SHAPE == kWide     ? 5.3 + rounds(tiles, 0.65) * (SHORT ? 1.15 : 1.0) * (steps * 0.475 + 4.25)
                   : KC::SHAPE == kNarrow ? 4.55 + rounds(tiles, 0.75) * (SHORT ? 1.16 : strided ? 1.12 : 1.0) * (steps * 0.3035 + 2.3)
                                          : 5.05 + rounds(tiles, 0.65) * (SHORT ? 1.3 : HF * WF >= 25 ? 0.94 : 1.0) * (steps * 0.31 + 2.2);
        };
        // (Strips only add tiles: what is too slow without them needs no search of their widths.  On the host, a search for every
        // configuration takes 1.2 to 2 us of a call.)
        if (time((uint32_t)((sh.npix + TN - 1) / TN) * (uint32_t)((sh.Co + TM - 1) / TM)) >= least) return;
        if (!split_params<HF, WF, CFG>(Q[CFG], P, sh, IMP, &lds[CFG])) return;
        const double t = time(Q[CFG].nblocks);
        if (t < least) { least = t; pick = CFG; }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    using C2 = std::integral_constant<int, 2>;
    using C3 = std::integral_constant<int, 3>;
    using C4 = std::integral_constant<int, 4>;
    constexpr bool LONG = HF * WF != 3;                             // (1x3 and 3x1: 0 would be 3 with one item per thread)
    constexpr bool EIGHT = HF == WF && (HF == 3 || HF == 5);       // (the others hold 8 channels in every configuration, or need not)
    if constexpr (LONG) consider(C0{});
    consider(C1{});
    if constexpr (EIGHT) consider(C2{});
    consider(C3{});
    consider(C4{});
    switch (pick) {
        case 0:
            if constexpr (LONG) return launch_split_t<HF, WF, 0, IMP>(Q[0], lds[0], dev, ncu, st, plan);
            return hipErrorNotSupported;
        case 1: return launch_split_t<HF, WF, 1, IMP>(Q[1], lds[1], dev, ncu, st, plan);
        case 2:
            if constexpr (EIGHT) return launch_split_t<HF, WF, 2, IMP>(Q[2], lds[2], dev, ncu, st, plan);
            return hipErrorNotSupported;
        case 3: return launch_split_t<HF, WF, 3, IMP>(Q[3], lds[3], dev, ncu, st, plan);
        case 4: return launch_split_t<HF, WF, 4, IMP>(Q[4], lds[4], dev, ncu, st, plan);
        default: return hipErrorNotSupported;
    }
}

// hipErrorNotSupported where the layer's filter has no instance, no tile shape fits or the fp32 pipeline is the faster one.
hipError_t launch_conv_split(const MfmaParams &P, const Shape &sh, uint32_t blocks, hipStream_t st, bool implicit, LaunchPlan *plan)
{
    auto go = [&](auto hf, auto wf, int least_ci) {
        constexpr int HF = decltype(hf)::value, WF = decltype(wf)::value;
        if (sh.Hf != HF || sh.Wf != WF || sh.Ci < least_ci) return hipErrorNotSupported;
        return implicit ? launch_split<HF, WF, true>(P, sh, blocks, st, plan) : launch_split<HF, WF, false>(P, sh, blocks, st, plan);
    };
    using I1 = std::integral_constant<int, 1>;
    using I3 = std::integral_constant<int, 3>;
    using I4 = std::integral_constant<int, 4>;
    using I5 = std::integral_constant<int, 5>;
    using I7 = std::integral_constant<int, 7>;
    hipError_t e = go(I3{}, I3{}, 8);
    if (e == hipErrorNotSupported) e = go(I5{}, I5{}, 4);
    if (e == hipErrorNotSupported) e = go(I7{}, I7{}, 2);
    if (e == hipErrorNotSupported) e = go(I1{}, I7{}, 8);
    if (e == hipErrorNotSupported) e = go(I7{}, I1{}, 8);
    if (e == hipErrorNotSupported) e = go(I1{}, I3{}, 16);
    if (e == hipErrorNotSupported) e = go(I3{}, I1{}, 16);
    if (e == hipErrorNotSupported) e = go(I4{}, I4{}, 4);
    return e;
}

}  // namespace im2win
