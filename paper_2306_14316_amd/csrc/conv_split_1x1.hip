// bf16-piece convolution (see conv_split.h for the pieces and their precision) of 1x1 layers: the GEMM
// O[Co x pixels] = F[Co x Ci] * I[Ci x pixels], any stride, no padding.
//
// What bounds it: six MFMAs per fp32 product, and beside them the cutting of both operands -- a tile of 128 channels x 128 pixels
// cuts 256 words per 16384 products, 6.5 vector instructions each, half of the time of its MFMAs.  So the cutting has to run beside
// the MFMAs and a tile has to be large: tiles of 64 channels cut each pixel word Co/64 times, which took what the MFMAs save.
// Eight waves, two per SIMD, all of which stage and multiply; half of them multiply first and stage then, the others the other way
// round (see conv_split_stem.hip).  K blocks of 32 channels, two LDS stages, one barrier per block; a workgroup runs its tiles as one
// sequence of K blocks, so the next tile's first block is on its way while a tile ends.
//
// A channel count that is no multiple of eight leaves the last group's missing words zero (RAG: a select per word).
//
// Measured (convolution alone, us, fp32 matrix cores -> tiles of 128 -> of 256 pixels): 256 -> 256 channels 28x28 N=64 62 -> 51 -> 44, 512 -> 512
// 14x14 N=32 37 -> 25 -> 35, N=128 112 -> 92 -> 75, 56x56 N=64 940 -> 627 -> 550 (191 TFLOP/s); 1024 -> 256 14x14 N=64 70 -> 44 -> 63.  A lone tile
// of 128 pixels takes 1.3 us for a K block whose MFMAs take 0.65: a wave's own chain of cutting, writing and reading; of 256 pixels 1.85 for
// 1.3.  Fetching two blocks ahead gave nothing; tiles of 64 x 256 for layers of up to 64 channels 16 against 13 (256 -> 64 56x56 N=8).  Relative
// 2-norm error against 64 bits 7e-8 (fp32 matrix cores 2e-7).
//
// LDS: [channel group of 8][piece][row or pixel][8 channels], one 16-byte read per operand and piece.  A thread fetches eight
// consecutive filter words, and one word of eight channel planes per pixel, lanes on neighbouring pixels: strides and planes of any size
// are only another offset per pixel.
#include "conv_split.h"
#include "runtime_cache.h"

#include <algorithm>

namespace im2win {

struct Split1x1Params : SplitParams {
    uint32_t npix, ntiles;
    int nkb;                  // K blocks of 32 channels
    uint32_t rowstep;         // words of the source from one output row to the next
    FastDiv d_wo, d_howo;
};

// Tiles of 128 channels x 128*FN pixels; a wave owns 64 x 32*FN.
template <int FN>
struct Tile1x1 {
    static constexpr int WGM = 2, TM = 128, TN = 128 * FN;
    // (+64: the four groups of a filter row, which neighbouring lanes write, start in other banks)
    static constexpr uint32_t APL = 3 * TM * 16 + 64, BPL = 3 * TN * 16, BOFF = 4 * APL, STAGE = BOFF + 4 * BPL, PASS = 2 * STAGE;
    static constexpr size_t LDS = PASS + 64;
};

// RAG: Ci is no multiple of eight.
template <int FN, bool RAG, bool IMP>
__global__ __launch_bounds__(512, 2) void conv_split_1x1_kernel(Split1x1Params P)
{
    using T = Tile1x1<FN>;
    constexpr int TM = T::TM, TN = T::TN;
    extern __shared__ __align__(16) unsigned char smem[];
    lds_byte *const L = (lds_byte *)smem;
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % T::WGM, wn = wave / T::WGM;
    const bool late = (wave >> 2) & 1;
    const uint32_t gx = gridDim.x;
    uint32_t first = blockIdx.x, stop = P.ntiles;
    float scale = kScale;

    auto origin = [&](uint32_t t, int &m0, uint32_t &P0) __attribute__((always_inline)) {   // (the M tiles of a pixel tile are neighbours in one L2)
        const uint32_t lb = xcd_swizzle(t, P.ntiles), tn = fdiv(lb, P.d_tm);
        m0 = (int)(lb - tn * (uint32_t)P.tiles_m) * TM;
        P0 = tn * TN;
    };

    // ---- staging.  Filter item: row tid/4, channels 8*(tid%4) ..; pixel items: pixel tid%TN, groups tid/TN + ... of 8 channels
    float wa[8], wb[FN][8];
    const int ar = tid >> 2, ag = tid & 3;
    const int bp = tid % TN, bg = tid / TN;
    uint32_t ft = 0, fvo = 0, bvo[FN];     // tile and offsets of the block being fetched
    int fkb = 0;
    __amdgpu_buffer_rsrc_t rf, rw;
    auto aim = [&](uint32_t t) __attribute__((always_inline)) {
        int m0;
        uint32_t P0;
        origin(t, m0, P0);
        rf = operand_desc(P.flt + (size_t)m0 * P.K, ((size_t)P.Co - (size_t)m0) * P.K);
        fvo = m0 + ar < P.Co ? (uint32_t)(ar * P.K + ag * 8) * 4u : kNoWord;
        const uint32_t img0 = fdiv(P0, P.d_howo);
        const size_t base = (size_t)img0 * P.Ci * P.plane;
        rw = operand_desc(P.src + base, P.src_elems - base);
        const uint32_t px = min(P0 + (uint32_t)bp, P.npix - 1u), img = fdiv(px, P.d_howo), pin = px - img * P.howo;
        const uint32_t m = fdiv(pin, P.d_wo), n = pin - m * (uint32_t)P.Wo;
        const uint32_t at = (img - img0) * (uint32_t)P.Ci * P.plane + m * P.rowstep + n * (uint32_t)P.s;
#pragma unroll
        for (int j = 0; j < FN; ++j) bvo[j] = (at + (uint32_t)((bg + j * (4 / FN)) * 8) * P.plane) * 4u;
    };
    auto fetch = [&]() __attribute__((always_inline)) {   // the block (ft, fkb); then the one after it, or the last again
        const int c0 = fkb * 32;
        const int room = P.Ci - c0;
        const uint32_t vo = ag * 8 < room ? fvo : kNoWord;
        const u32v4 a0 = __builtin_amdgcn_raw_buffer_load_b128(rf, vo, (uint32_t)c0 * 4u, 0), a1 = __builtin_amdgcn_raw_buffer_load_b128(rf, vo, (uint32_t)c0 * 4u + 16u, 0);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t w = e < 4 ? a0[e & 3] : a1[e & 3];
            wa[e] = __builtin_bit_cast(float, !RAG || ag * 8 + e < room ? w : 0u);   // (the words behind a row's last are the next row's)
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int c = (bg + j * (4 / FN)) * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                wb[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rw, c + (RAG ? e : 0) < room ? bvo[j] : kNoWord, (uint32_t)(c0 + e) * P.plane * 4u, 0));
        }
        if (++fkb == P.nkb) {
            if (ft + gx < stop) { ft += gx; aim(ft); fkb = 0; }
            else fkb = P.nkb - 1;
        }
    };
    auto stage = [&](uint32_t at) __attribute__((always_inline)) {
        bf16x8 c[3];
        split8(wa, scale, c[0], c[1], c[2]);
#pragma unroll
        for (int k = 0; k < 3; ++k) *(lds_bf16x8 *)(L + at + (uint32_t)ag * T::APL + (uint32_t)(k * TM + ar) * 16u) = c[k];
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            split8(wb[j], scale, c[0], c[1], c[2]);
#pragma unroll
            for (int k = 0; k < 3; ++k) *(lds_bf16x8 *)(L + at + T::BOFF + (uint32_t)(bg + j * (4 / FN)) * T::BPL + (uint32_t)(k * TN + bp) * 16u) = c[k];
        }
    };

    // ---- multiplication of one K block: two steps.  The second's operands are read as the registers of each piece come free, the h pieces
    // last, behind whose read the products of the m pieces run.  (A second set for the h pieces would spill.)
    floatx16 acc[2][FN], acs[2][FN];
    auto multiply = [&](uint32_t at) __attribute__((always_inline)) {
        struct Piece { bf16x8 a[2], b[FN]; };
        Piece ph, pm, pl;
        const uint32_t pa = at + (uint32_t)h * T::APL + (uint32_t)(wm * 64 + l32) * 16u;
        const uint32_t pb = at + T::BOFF + (uint32_t)h * T::BPL + (uint32_t)(wn * 32 * FN + l32) * 16u;
        auto read = [&](int s, int k, Piece &x) __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < 2; ++f) x.a[f] = *(const lds_bf16x8 *)(L + pa + 2 * s * T::APL + (k * TM + f * 32) * 16);
#pragma unroll
            for (int n = 0; n < FN; ++n) x.b[n] = *(const lds_bf16x8 *)(L + pb + 2 * s * T::BPL + (k * TN + n * 32) * 16);
        };
        auto mul = [&](floatx16 (&c)[2][FN], const Piece &x, const Piece &y) __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int n = 0; n < FN; ++n) c[f][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.a[f], y.b[n], c[f][n], 0, 0, 0);
        };
        read(0, 1, pm); read(0, 0, ph); read(0, 2, pl);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            __builtin_amdgcn_sched_barrier(0);
            mul(acs, pm, pm);
            mul(acs, pl, ph);
            mul(acs, ph, pl);
            __builtin_amdgcn_sched_barrier(0);
            if (s == 0) read(1, 2, pl);
            __builtin_amdgcn_sched_barrier(0);
            mul(acs, pm, ph);
            mul(acs, ph, pm);
            __builtin_amdgcn_sched_barrier(0);
            if (s == 0) read(1, 1, pm);
            __builtin_amdgcn_sched_barrier(0);
            mul(acc, ph, ph);
            __builtin_amdgcn_sched_barrier(0);
            if (s == 0) read(1, 0, ph);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int n = 0; n < FN; ++n)
#pragma unroll
                for (int v = 0; v < 16; ++v) { acc[f][n][v] = 0.0f; acs[f][n][v] = 0.0f; }
    };

    uint32_t lo = 0xffffffffu, hi = 0;   // (uniform) first and last tile with an infinite or NaN output
    auto store = [&](auto secondc, uint32_t t, int nb) __attribute__((always_inline)) {   // (nb: the wave's block of 32 pixels)
        int m0;
        uint32_t P0;
        origin(t, m0, P0);
        m0 += wm * 64;
        const uint32_t pix = P0 + (uint32_t)((wn * FN + nb) * 32 + l32);
        const bool live = pix < P.npix;
        const uint32_t img0 = fdiv(P0, P.d_howo), img = fdiv(min(pix, P.npix - 1u), P.d_howo);
        const uint32_t pin = min(pix, P.npix - 1u) - img * P.howo;
        const __amdgpu_buffer_rsrc_t ro = output_desc(P.out, P.out_elems, ((size_t)img0 * P.Co + (size_t)min(m0, P.Co - 1)) * P.howo);
        const uint32_t howo4 = P.howo * 4u;
        const uint32_t voff = live ? ((img - img0) * (uint32_t)P.Co * P.howo + pin + (uint32_t)(4 * h) * P.howo) * 4u : kNoStore;
        const int room = P.Co - m0 - 4 * h;
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            float v[16], big = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                v[r] = (acc[f][nb][r] + acs[f][nb][r]) * (decltype(secondc)::value ? 1.0f / (kScale2 * kScale2) : 1.0f / (kScale * kScale));
                big = __builtin_elementwise_maximum(big, __builtin_fabsf(v[r]));
            }
            if constexpr (decltype(secondc)::value) {
                settle_outputs<1, 1, IMP, 16, 1>(P, ro, voff + (uint32_t)(32 * f) * howo4, live, room - 32 * f, img, m0 + 4 * h + 32 * f, pin,
                                                 [&](int, int r, float &a) __attribute__((always_inline)) { a = acc[f][nb][r]; return v[r]; });
            } else {
                if (__builtin_amdgcn_ballot_w64(live && !finite(big))) {
                    // (the small products of an infinity are NaN: the sum of the h*h products stands for the output)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float x = acc[f][nb][r];
                        v[r] = finite(x) ? v[r] : x;
                    }
                    lo = min(lo, t);
                    hi = t;
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int dj = 32 * f + 8 * (r >> 2) + (r & 3);
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v[r]), ro, dj < room ? voff : kNoStore, (uint32_t)dj * howo4, 0);
                }
            }
        }
    };

    // One pass over the tiles first, first + gx, ... below stop; LATE: the wave stages before it multiplies.  After the last block the
    // last one is staged again.
    auto tiles = [&](auto secondc, auto latec) __attribute__((always_inline)) {
        uint32_t at = 0;
        for (uint32_t t = first; t < stop; t += gx) {
            clear();
            for (int kb = 0; kb < P.nkb; ++kb) {
                auto next = [&]() __attribute__((always_inline)) { stage(at ^ T::STAGE); fetch(); };
                if constexpr (decltype(latec)::value) next();
                multiply(at);
                if constexpr (!decltype(latec)::value) next();
                at ^= T::STAGE;
                lds_barrier();
            }
#pragma unroll
            for (int nb = 0; nb < FN; ++nb) store(secondc, t, nb);
        }
    };
    auto pass = [&](auto secondc) __attribute__((always_inline)) {
        ft = first;
        fkb = 0;
        aim(ft);
        fetch();
        stage(0);
        fetch();
        lds_barrier();
        if constexpr (decltype(secondc)::value) tiles(secondc, std::false_type{});
        else if (late) tiles(secondc, std::true_type{});
        else tiles(secondc, std::false_type{});
    };
    static_assert(T::PASS % 16 == 0, "");
    pass(std::false_type{});
    // a second pass over the tiles, from the first to the last that has an infinite or NaN output (see conv_split.h)
    if (lane == 0) *(lds_u32v2 *)(L + T::PASS + wave * 8) = u32v2{lo, hi};
    lds_barrier();
    uint32_t from = 0xffffffffu, to = 0;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const u32v2 v = *(const lds_u32v2 *)(L + T::PASS + w * 8);
        from = min(from, v[0]);
        to = max(to, v[1]);
    }
    first = __builtin_amdgcn_readfirstlane(from);
    if (first == 0xffffffffu) return;
    stop = __builtin_amdgcn_readfirstlane(to) + 1u;
    scale = kScale2;
    pass(std::true_type{});
}

template <int FN, bool RAG>
static hipError_t launch_1x1_t(Split1x1Params P, bool implicit, int dev, int ncu, hipStream_t st, LaunchPlan *plan)
{
    using T = Tile1x1<FN>;
    const unsigned long long imgs = std::min<unsigned long long>((unsigned long long)T::TN / P.howo + 2, (unsigned long long)P.N);
    const unsigned long long larger = std::max((unsigned long long)P.Hi * P.Wi, (unsigned long long)P.Ho * P.rowlen);   // (both calls take the same kernel)
    if (imgs * P.Ci * larger * 4ull >= (1ull << 31) || (unsigned long long)P.K * 4ull * T::TM >= (1ull << 31)) return hipErrorNotSupported;
    if (((unsigned long long)P.Co * imgs + 128ull) * P.howo * 4ull >= kNoStore) return hipErrorNotSupported;
    P.tiles_m = (P.Co + T::TM - 1) / T::TM;
    P.d_tm = make_fastdiv((uint32_t)P.tiles_m);
    P.ntiles = ((P.npix + T::TN - 1) / T::TN) * (uint32_t)P.tiles_m;
    const uint32_t grid = std::min(P.ntiles, (uint32_t)ncu);   // one workgroup per compute unit; it takes every grid-th tile
    if (plan) {
        plan_record(plan, dim3(grid), 512, T::LDS, "conv_split_1x1_kernel<%d, %s, %s>", FN, tf(RAG), tf(implicit));
        return hipSuccess;
    }
    void (*kern)(Split1x1Params) = implicit ? &conv_split_1x1_kernel<FN, RAG, true> : &conv_split_1x1_kernel<FN, RAG, false>;
    static KernelCache kc[2];
    const hipError_t e = allow_dynamic_lds(kc[implicit], reinterpret_cast<const void *>(kern), T::LDS, dev);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(512), T::LDS, st, P);
    return hipGetLastError();
}

// hipErrorNotSupported where the fp32 kernel (conv_mfma_1x1.hip) is the faster one or the layer is outside its conditions.
hipError_t launch_conv_split_1x1(const float *src, const float *flt, float *out, const Shape &sh, hipStream_t st, bool implicit, LaunchPlan *plan)
{
    if (sh.Hf != 1 || sh.Wf != 1 || sh.p != 0) return hipErrorNotSupported;
    int dev = 0, ncu = 0;
    hipError_t e = device_cus(&dev, &ncu);
    if (e != hipSuccess && plan) { e = hipSuccess; ncu = 256; }   // planning without a device: an MI355X's 256 compute units
    if (e != hipSuccess) return e;
    Split1x1Params P = {};
    P.src = src; P.flt = flt; P.out = out;
    P.N = sh.N; P.Ci = sh.Ci; P.Ho = sh.Ho; P.Wo = sh.Wo; P.Co = sh.Co; P.s = sh.s; P.K = sh.K;
    P.Hi = sh.Hi; P.Wi = sh.Wi; P.p = 0; P.rowlen = sh.rowlen;
    P.plane = implicit ? (uint32_t)(sh.Hi * sh.Wi) : (uint32_t)((size_t)sh.Ho * sh.rowlen);
    P.rowstep = implicit ? (uint32_t)sh.s * (uint32_t)sh.Wi : (uint32_t)sh.rowlen;
    P.howo = (uint32_t)(sh.Ho * sh.Wo); P.npix = (uint32_t)sh.npix; P.nkb = (sh.Ci + 31) / 32;
    P.src_elems = (size_t)sh.N * sh.Ci * P.plane; P.out_elems = (size_t)sh.npix * sh.Co;
    P.d_wo = make_fastdiv((uint32_t)sh.Wo); P.d_howo = make_fastdiv(P.howo);
    if (sh.s > 65536) return hipErrorNotSupported;
    // Which is faster, in us: fitted to 1300 layers, the pieces' tiles of 128 and 256 pixels 6 and 8 % off (root mean square), the fp32 kernel's 13 %
    // (the pick takes 1.002 times the best one's time on average).  `mix`: how far a last round that leaves units idle counts in full.  Layers that
    // the fp32 1x1 kernel does not take (Ci no multiple of 8, Co none of 4) ran the generic kernels, which take up to eight times as long:
    // in us, generic two calls / workspace-free / pieces: 43 -> 100 channels 28x28 N=29 28 / 27 / 8.6, 285 -> 94 8x5 N=58 20 / 126 / 16, 870 -> 102
    // 16x16 stride 2 N=8 59 / 391 / 40, 226 -> 19 44x44 N=6 16 / 93 / 15.  Up to sixteen channels they may be the faster ones (a block of the pieces is
    // 32 channels long) and have an estimate too, fitted to 1166 layers (8 % off the geometric mean of both calls; the pick takes 1.003 times
    // the best one's time on average; 985 layers of 17 to 200 channels are all faster in pieces):
    // 8 -> 6 63x63 N=37 9.4 / 9.6 / 17.7, 7 -> 19 184x184 N=156 365 / 374 / 491, 16 -> 9 77x76 N=102 41 / 41 / 58, 10 -> 10 on 84 images of one pixel 15 / 21 / 5.6; up to four
    // they stay there.  The price of one rule for both calls is 229 rows of 1624 -> 90 channels, in two calls 88 us generic, 102 here.  Measured, fp32 / 128 / 256 pixels, the
    // one that runs in brackets: 256 -> 256 28x28 N=64 62 / 51 / [44], 14x14 N=32 [12.7] / 14.4 / 21, N=128 34 / 27 / [25]; 512 -> 512 14x14 N=32
    // 37 / [25] / 35, N=64 64 / 45 / [39], N=128 112 / 92 / [75], 56x56 N=64 940 / 627 / [550]; 1024 -> 256 14x14 N=64 70 / [44] / 63, N=128 122 / 85 / [70].
    auto rounds = [&](double r, double mix) {
        const double up = (double)(long long)(r + 0.9999);
        return mix * up + (1.0 - mix) * std::max(r, up > 1.5 ? 0.0 : 0.6);
    };
    auto tiles = [&](int tm, int tn) { return (double)((P.npix + tn - 1) / tn) * ((sh.Co + tm - 1) / tm) / ncu; };
    const bool ragged = sh.Ci % 8 != 0, fp32 = !ragged && sh.Co % 4 == 0;
    const double t1 = 3.15 + rounds(tiles(128, 128), 0.45) * (P.nkb * (ragged ? 1.58 : 1.47) + 2.2);
    const double t2 = 3.65 + rounds(tiles(128, 256), 0.45) * (P.nkb * (ragged ? 2.49 : 2.33) + (ragged ? 5.65 : 5.1));
    if (fp32) {
        const double r = tiles(64, 64), up = (double)(long long)(r + 0.9999);
        if (std::min(t1, t2) > 0.9 * (3.56 + (0.25 * up + 0.75 * std::max(r, up > 1.5 ? 0.0 : 1.0)) * (sh.Ci * 0.0213 + 0.28))) return hipErrorNotSupported;
    } else if (sh.Ci <= 16) {
        // tiles of 64 x 64 in K blocks of eight channels (vector loads where the blocks are whole), `rows` of the output to a tile; 0.3 us
        // is added, as the pieces take some less than t1 in a single round
        const double r = std::max(tiles(64, 64) - 1.0, 0.0), kb = (sh.Ci + 7) / 8, rows = std::min(std::min(64, (62 + sh.Wo) / sh.Wo + 1), (int)((P.npix + sh.Wo - 1) / sh.Wo));
        const double generic = 4.68 + kb * ((ragged ? 2.0 : 0.3) + 0.1 * rows) +
                               r * (0.26 + kb * ((ragged ? 0.54 : 0.29) + 0.015 * rows + 0.05 * (sh.s - 1)) + 0.54 * std::min(sh.Co, 64) / 64.0);
        if (sh.Ci <= 4 || std::min(t1, t2) > generic) return hipErrorNotSupported;
    }
    if (t2 < t1) {
        e = sh.Ci % 8 ? launch_1x1_t<2, true>(P, implicit, dev, ncu, st, plan) : launch_1x1_t<2, false>(P, implicit, dev, ncu, st, plan);
        if (e != hipErrorNotSupported) return e;
    }
    return sh.Ci % 8 ? launch_1x1_t<1, true>(P, implicit, dev, ncu, st, plan) : launch_1x1_t<1, false>(P, implicit, dev, ncu, st, plan);
}

}  // namespace im2win
