// bf16-piece convolution (see conv_split.h for the pieces and their precision) of layers with three input channels:
// 7x7 at stride 2, 11x11 at stride 4, 3x3 at strides 1 and 2.  K is 27 to 363, the pixels are many, and what
// the piece kernel of the deeper layers spends per tile on its filter stages, its start and its stores would cost more
// than the MFMAs of such a tile.
//
// What bounds it: the six products per fp32 product on the matrix cores and the streams of the im2win tensor and the
// output are of the same size (7x7, 128 images of 224x224, 64 channels: 72 us at the bf16 peak, 117 us of memory).
// So everything else has to run beside them:
//   - the filter is stationary: a wave cuts its 32 rows (its Q-th of K) into pieces once and keeps them in registers,
//     an MFMA reads its pixel operand only;
//   - a wave stages (cuts words into pieces and writes them to LDS) as well as multiplies.  Two or three waves share
//     a SIMD; in each period half of them multiply first and stage then, the others the other way round, so that the
//     vector ALU works for one while the matrix pipe works for the other (3x3 with one block of channels: workgroups
//     of four waves, one per SIMD, and two workgroups to a unit).  Pixel stages are double-buffered: one barrier per tile;
//   - where K does not fit a wave's registers, Q waves share a 32x32 block: each takes its part of K and hands the
//     others the sums of the channels that they store, through LDS, a period later.
//
// Measured (convolution alone, us, fp32 matrix cores -> here): 7x7, 128 images of 224x224, 64 channels 256 -> 199 (workspace-free 287 ->
// 213), 96 channels 530 -> 338; 11x11 stride 4, 128 images of 227x227, 96 channels 240 -> 172, 64 channels 184 -> 139.  Without the staging
// the first takes 172 (MFMAs fed from LDS alone, on such operands, run at 70 % of the peak: the clock falls to 1.65-1.9 GHz under them); matrix pipes
// busy 63 and 51 % of the cycles.  All waves in one order 221; stores under a branch, so that a wait for words waits for stores too, 227.
// Relative 2-norm error against 64 bits 7e-8 for both (fp32 matrix cores 2.2e-7 and 2.4e-7).
//
// LDS image of the pixels, [channel][piece][chunk of 16 bytes], eight values of K per chunk, so that a pixel operand is
// one 16-byte read per piece:
//   7x7: a chunk is one column of a window -- seven consecutive words of the im2win tensor -- and a zero (11 steps of 16
//     values of K instead of 9.2; windows start 28 bytes apart in the tensor's own order, which no 16-byte read can
//     take).  Even and odd columns lie apart: neighbouring windows, two columns apart, are then neighbouring chunks,
//     where 32 bytes between them would use half of the banks;
//   3x3: a chunk is two columns, each of three words and a zero; windows start eight bytes apart and the fourth column is masked (3 steps);
//   11x11: the tensor's own order; windows start 88 bytes apart and their 121 words are 15 chunks and one word, whose
//     chunk is masked (24 steps instead of 22.7).
#include "conv_split.h"
#include "runtime_cache.h"

#include <algorithm>

namespace im2win {

struct StemParams : SplitParams {
    uint32_t npix, ntiles;
    int chf;                // chunks of a full output row
    FastDiv d_wo, d_howo, d_chf;
};

// HF x HF windows; R blocks of 32 rows, Q parts of K, PX runs of 32*B pixels: one wave each.
// B = 4: a lane's four pixels are neighbours and their outputs leave in one store (of any 4-byte alignment).
template <int HF_, int R_, int Q_, int PX_, int B_>
struct Stem {
    static constexpr int HF = HF_, R = R_, Q = Q_, PX = PX_, B = B_;
    static constexpr bool WIDE = B == 4;
    static constexpr bool COLS = HF == 7, PAIRS = HF == 3;   // chunks are columns, pairs of columns
    static constexpr int KHW = HF * HF, NW = R * Q * PX, NT = 64 * NW, TN = 32 * PX * B;
    static constexpr int STEPS = COLS ? 11 : (PAIRS ? 3 : 24), SPQ = (STEPS + Q - 1) / Q;
    // chunks per channel and piece
    static constexpr int CAP = COLS ? (PX == 4 ? 336 : 176) : (PAIRS ? (B == 4 ? 284 : 140) : (PX == 2 ? 392 : 256));
    static constexpr uint32_t PCB = CAP * 16, CHB = 3 * PCB, STAGE = 3 * CHB;
    static constexpr uint32_t ODD = PCB / 2;                 // COLS: odd columns
    static constexpr int OWN = 16 / Q;                       // accumulators a wave stores
    static constexpr uint32_t RED = Q > 1 ? (uint32_t)(R * PX * Q * (Q - 1)) * (OWN / 4) * 1024u : 0u;
    static constexpr uint32_t PASS = 2 * STAGE + 2 * RED;
    static constexpr size_t LDS = PASS + NW * 8;
    static constexpr int JX = (3 * CAP + NT - 1) / NT;       // chunks a thread stages per tile, at most
    static_assert(LDS <= 160 * 1024 && (Q == 1 || B == 1) && (B == 1 || B == 4), "");
    // chunk (channel, index) that lane half h of step i multiplies; index: the column, the pair of columns or the chunk of the window; -1: none
    static constexpr int chan(int i, int h) { return COLS ? (i < 7 ? h : 2) : (PAIRS ? i : (i < 18 ? i / 6 : (i - 18) / 2)); }
    static constexpr int index(int i, int h)
    {
        if (COLS) return i < 7 ? i : (2 * (i - 7) + h < 7 ? 2 * (i - 7) + h : -1);
        if (PAIRS) return h;
        return i < 18 ? 2 * (i % 6) + h : 12 + 2 * (i % 2) + h;   // (11x11: the fourth quarter takes what the first three leave)
    }
    // filter word (u*HF + v) that value e of a chunk stands for; -1: none
    static constexpr int tap(int idx, int e)
    {
        if (idx < 0) return -1;
        if (COLS) return e < HF ? e * HF + idx : -1;
        if (PAIRS) return e % 4 < HF && 2 * idx + e / 4 < HF ? (e % 4) * HF + 2 * idx + e / 4 : -1;
        const int t = 8 * idx + e;
        return t < KHW ? (t % HF) * HF + t / HF : -1;
    }
};

template <class F, int... I>
__device__ __forceinline__ void stem_for(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// The largest magnitude of a wave's sums, NaN if there is one.
template <class V>
__device__ __forceinline__ float largest(const V &v)
{
    constexpr int n = sizeof(V) / 4;
    float m = __builtin_fabsf(v[0]);
#pragma unroll
    for (int i = 1; i < n; ++i) m = __builtin_elementwise_maximum(m, __builtin_fabsf(v[i]));
    return m;
}

template <class T, bool IMP>
__device__ __forceinline__ void conv_stem_body(const StemParams &P, unsigned char *smem)
{
    constexpr int HF = T::HF, SPQ = T::SPQ, Q = T::Q, JX = T::JX;
    constexpr uint32_t PCB = T::PCB, CHB = T::CHB;
    lds_byte *const L = (lds_byte *)smem;
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (waves 4 apart share a SIMD: the parts of K of one block lie on different ones, and so do the halves of the order.
    // Four waves: one to a SIMD, all in one order, and the waves of the unit's second workgroup beside them)
    const int ks = wave % Q, px = (wave / Q) % T::PX, rb = wave / (Q * T::PX);
    const bool late = T::NW > 4 && ((wave >> 2) & 1);
    const int m0 = ((int)blockIdx.y * T::R + rb) * 32;   // the wave's first output channel
    const uint32_t gx = gridDim.x;

    uint32_t first = xcd_swizzle(blockIdx.x, gx), stop = P.ntiles;   // (per round, an XCD's workgroups take neighbouring tiles)
    float scale = kScale;

    struct Tile { uint32_t P0, Pend, q0, q1; int n0, ch0, total; };   // rows q0 .. q1 of all images; chunks of the first row, of all
    auto tile_of = [&](uint32_t t) __attribute__((always_inline)) {
        Tile o;
        o.P0 = t * T::TN;
        o.Pend = min(o.P0 + T::TN, P.npix) - 1u;
        o.q0 = fdiv(o.P0, P.d_wo);
        o.q1 = fdiv(o.Pend, P.d_wo);
        o.n0 = (int)(o.P0 - o.q0 * (uint32_t)P.Wo);
        const int n1 = (int)(o.Pend - o.q1 * (uint32_t)P.Wo);
        auto chunks = [&](int pixels) __attribute__((always_inline)) {
            const int cols = (pixels - 1) * P.s + HF;
            return T::COLS ? (cols + 1) & ~1 : (T::PAIRS ? (cols + 1) >> 1 : (cols * HF + 7) >> 3);
        };
        o.ch0 = chunks((o.q0 == o.q1 ? n1 + 1 : P.Wo) - o.n0);
        o.total = o.q0 == o.q1 ? o.ch0 : o.ch0 + (int)(o.q1 - o.q0 - 1u) * P.chf + chunks(n1 + 1);
        return o;
    };

    // ---- staging: a thread's chunks of a tile, from memory into registers and, cut up, into LDS
    float words[JX][8];
    uint32_t dest[JX];       // LDS byte offset in the stage; kNoWord: none
    auto fetch = [&](uint32_t t) __attribute__((always_inline)) {
        const Tile o = tile_of(t);
        const uint32_t img0 = fdiv(o.q0, P.d_ho);
        const size_t base = (size_t)img0 * 3u * P.plane;
        const size_t left = (P.src_elems - base) * 4u;
        const uint32_t bytes = left < 0x7fffffffull ? (uint32_t)left : 0x7fffffffu;
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(P.src + base), 0, bytes, 0x00020000);
        auto load1 = [&](uint32_t vo) __attribute__((always_inline)) {
            return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rw, vo, 0, 0));
        };
#pragma unroll
        for (int j = 0; j < JX; ++j) {
            const int id = tid + T::NT * j;
            const bool live = id < 3 * o.total;
            const int r = (id >= o.total ? 1 : 0) + (id >= 2 * o.total ? 1 : 0);
            const int x = id - r * o.total;
            const int i = x < o.ch0 ? 0 : 1 + (int)fdiv((uint32_t)(x - o.ch0), P.d_chf);
            const int c = i == 0 ? x : x - o.ch0 - (i - 1) * P.chf;   // chunk within the row
            const uint32_t q = o.q0 + (uint32_t)i;
            const uint32_t img = fdiv(q, P.d_ho);
            const int m = (int)(q - img * (uint32_t)P.Ho);
            const uint32_t pl = ((img - img0) * 3u + (uint32_t)r) * P.plane;
            const int col0 = (i == 0 ? o.n0 : 0) * P.s;               // column of the row's first word
            dest[j] = live ? (uint32_t)r * CHB + (T::COLS ? (uint32_t)(x & 1) * T::ODD + (uint32_t)(x >> 1) * 16u : (uint32_t)x * 16u) : kNoWord;
            if constexpr (IMP) {
                const int hh = m * P.s - P.p;
                if constexpr (T::COLS) {
                    const int ww = col0 + c - P.p;
                    const bool ok = live && ww >= 0 && ww < P.Wi;
#pragma unroll
                    for (int u = 0; u < HF; ++u)
                        words[j][u] = load1(ok && hh + u >= 0 && hh + u < P.Hi ? (pl + (uint32_t)((hh + u) * P.Wi + ww)) * 4u : kNoWord);
                } else if constexpr (T::PAIRS) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int ww = col0 + 2 * c + e / 4 - P.p, u = e % 4;
                        words[j][e] = u == HF ? 0.0f
                            : load1(live && ww >= 0 && ww < P.Wi && hh + u >= 0 && hh + u < P.Hi ? (pl + (uint32_t)((hh + u) * P.Wi + ww)) * 4u : kNoWord);
                    }
                } else {
                    int k = (8 * c) / HF, u = 8 * c - k * HF;
                    k += col0 - P.p;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const bool ok = live && k >= 0 && k < P.Wi && hh + u >= 0 && hh + u < P.Hi;
                        words[j][e] = load1(ok ? (pl + (uint32_t)((hh + u) * P.Wi + k)) * 4u : kNoWord);
                        const bool wrap = ++u == HF;
                        u = wrap ? 0 : u;
                        k += wrap ? 1 : 0;
                    }
                }
            } else {
                constexpr uint32_t W = T::COLS ? HF : (T::PAIRS ? 6 : 8);   // words of a chunk
                const uint32_t off = pl + (uint32_t)(m * P.rowlen + col0 * HF) + (uint32_t)c * W;
                if constexpr (T::COLS) {
                    // (a row's last column of an odd number is read past the row: kept from the tensor's end)
                    const uint32_t vo = live && (off + HF) * 4u <= bytes ? off * 4u : kNoWord;
                    const u32v4 a = __builtin_amdgcn_raw_buffer_load_b128(rw, vo, 0, 0);
                    const u32v3 b = __builtin_amdgcn_raw_buffer_load_b96(rw, vo, 16, 0);
#pragma unroll
                    for (int u = 0; u < HF; ++u) { const uint32_t w = u < 4 ? a[u & 3] : b[(u & 3) % 3]; words[j][u] = __builtin_bit_cast(float, w); }
                } else {
                    const bool over = live && (off + W) * 4u > bytes;   // a row's last chunk, at the tensor's end
                    float w[8];
                    if (__builtin_amdgcn_ballot_w64(over)) {
#pragma unroll
                        for (uint32_t e = 0; e < W; ++e) w[e] = load1(live && (off + e + 1u) * 4u <= bytes ? (off + e) * 4u : kNoWord);
                    } else {
                        const uint32_t vo = live ? off * 4u : kNoWord;
                        const u32v4 a = __builtin_amdgcn_raw_buffer_load_b128(rw, vo, 0, 0);
#pragma unroll
                        for (int e = 0; e < 4; ++e) { const uint32_t x = a[e]; w[e] = __builtin_bit_cast(float, x); }
                        if constexpr (T::PAIRS) {
                            const u32v2 b = __builtin_amdgcn_raw_buffer_load_b64(rw, vo, 16, 0);
#pragma unroll
                            for (int e = 0; e < 2; ++e) { const uint32_t x = b[e]; w[4 + e] = __builtin_bit_cast(float, x); }
                        } else {
                            const u32v4 b = __builtin_amdgcn_raw_buffer_load_b128(rw, vo, 16, 0);
#pragma unroll
                            for (int e = 0; e < 4; ++e) { const uint32_t x = b[e]; w[4 + e] = __builtin_bit_cast(float, x); }
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) words[j][e] = !T::PAIRS ? w[e] : (e % 4 == HF ? 0.0f : w[e / 4 * HF + e % 4]);
                }
            }
            if constexpr (T::COLS) words[j][7] = 0.0f;
        }
    };
    auto stage = [&](uint32_t at) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < JX; ++j) {
            bf16x8 c[3];
            split8(words[j], scale, c[0], c[1], c[2]);
            if (dest[j] != kNoWord) {
#pragma unroll
                for (int k = 0; k < 3; ++k) *(lds_bf16x8 *)(L + at + dest[j] + k * PCB) = c[k];
            }
        }
    };

    // ---- the filter, in registers
    bf16x8 a[SPQ][3];
    auto load_filter = [&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        const int row = m0 + l32;
        const size_t base = (size_t)min(m0, P.Co - 1) * P.K;   // (uniform)
        const __amdgpu_buffer_rsrc_t rf = operand_desc(P.flt + base, (size_t)P.Co * P.K - base);
        stem_for([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value, s = q * SPQ + i;
            float w[8];
            int half = h;   // (opaque, one step at a time: as invariants of the passes the offsets would be kept, and spilled)
            asm volatile("" : "+v"(half));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                constexpr int none = -1;
                const int t0 = s < T::STEPS ? T::tap(T::index(s, 0), e) : none, t1 = s < T::STEPS ? T::tap(T::index(s, 1), e) : none;
                const uint32_t o0 = t0 < 0 ? kNoWord : (uint32_t)(T::chan(s, 0) * T::KHW + t0) * 4u;
                const uint32_t o1 = t1 < 0 ? kNoWord : (uint32_t)(T::chan(s, 1) * T::KHW + t1) * 4u;
                const uint32_t o = half ? o1 : o0;
                w[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rf, row < P.Co && o != kNoWord ? o + (uint32_t)(l32 * P.K) * 4u : kNoWord, 0, 0));
            }
            split8(w, scale, a[i][0], a[i][1], a[i][2]);
        }, std::make_integer_sequence<int, SPQ>{});
    };

    auto pixel = [&](int blk) __attribute__((always_inline)) {   // the lane's pixel in a block, from the tile's first
        return (uint32_t)(px * 32 * T::B + l32 * T::B + blk);
    };

    // ---- multiplication: a 32x32 block of the wave's over its part of K
    auto multiply = [&](auto qc, uint32_t t, int blk, uint32_t at) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, n = T::STEPS - q * SPQ < SPQ ? T::STEPS - q * SPQ : SPQ;
        const Tile o = tile_of(t);
        const uint32_t pix = min(o.P0 + pixel(blk), o.Pend);
        const uint32_t row = fdiv(pix, P.d_wo);
        const int i = (int)(row - o.q0), nn = (int)(pix - row * (uint32_t)P.Wo);
        const uint32_t lb = i == 0 ? 0u : (uint32_t)(o.ch0 + (i - 1) * P.chf) * (T::COLS ? 8u : 16u);   // (columns: two to a step of 16 bytes)
        const uint32_t b = at + lb + (uint32_t)(nn - (i == 0 ? o.n0 : 0)) * (T::COLS ? 16u : (uint32_t)P.s * (T::PAIRS ? 8u : HF * 2u));
        uint32_t base[3];   // COLS: of the pair steps, of the third channel, of its last step; otherwise one
        if constexpr (T::COLS) {
            base[0] = b + (uint32_t)h * CHB;
            base[1] = b + 2u * CHB + (uint32_t)h * T::ODD;
            base[2] = h ? at + 2u * CHB + PCB - 16u : b + 2u * CHB + 3u * 16u;   // (zeros)
        } else {
            base[0] = base[1] = base[2] = b + (uint32_t)h * 16u;
        }
        auto read = [&](auto ic, auto kc, bf16x8 (&x)[3]) __attribute__((always_inline)) {   // piece k of step i's pixels
            constexpr int s = q * SPQ + decltype(ic)::value, k = decltype(kc)::value;
            uint32_t from;
            if constexpr (T::COLS) {
                if constexpr (s < 7) from = base[0] + (s & 1) * T::ODD + (s >> 1) * 16u;
                else if constexpr (s < 10) from = base[1] + (s - 7) * 16u;
                else from = base[2];
                x[k] = *(const lds_bf16x8 *)(L + from + k * PCB);
            } else {
                from = base[0] + (uint32_t)T::chan(s, 0) * CHB + (uint32_t)T::index(s, 0) * 16u;
                const u32v2 lo = *(const lds_u32v2 *)(L + from + k * PCB), hi = *(const lds_u32v2 *)(L + from + k * PCB + 8u);
                x[k] = __builtin_bit_cast(bf16x8, u32v4{lo[0], lo[1], hi[0], hi[1]});
            }
        };
        auto mask = [&](auto ic, bf16x8 &x) __attribute__((always_inline)) {
            constexpr int s = q * SPQ + decltype(ic)::value;
            if constexpr (!T::COLS && T::tap(T::index(s, 1), 7) < 0) {   // the chunk that the window ends in
                u32v4 w = __builtin_bit_cast(u32v4, x);
                if constexpr (!T::PAIRS) {
                    w[0] &= h ? 0xffffu : 0xffffffffu;
                    w[1] = h ? 0u : w[1];
                }
#pragma unroll
                for (int d = 2; d < 4; ++d) w[d] = h ? 0u : w[d];
                x = __builtin_bit_cast(bf16x8, w);
            }
        };
        floatx16 acc, acs;
#pragma unroll
        for (int v = 0; v < 16; ++v) { acc[v] = 0.0f; acs[v] = 0.0f; }
        bf16x8 x[2][3];
        using K0 = std::integral_constant<int, 0>;
        using K1 = std::integral_constant<int, 1>;
        using K2 = std::integral_constant<int, 2>;
        read(K0{}, K0{}, x[0]); read(K0{}, K1{}, x[0]); read(K0{}, K2{}, x[0]);
        // A step's operands are read during the step before it, between its MFMAs.
        stem_for([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            if constexpr (i < n) {
                using IN = std::integral_constant<int, i + 1>;
                const bf16x8 (&f)[3] = a[i];
                bf16x8 (&p)[3] = x[i & 1], (&pn)[3] = x[(i + 1) & 1];
                mask(ic, p[0]); mask(ic, p[1]); mask(ic, p[2]);
                __builtin_amdgcn_sched_barrier(0);
                acs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[2], p[0], acs, 0, 0, 0);
                if constexpr (i + 1 < n) read(IN{}, K0{}, pn);
                __builtin_amdgcn_sched_barrier(0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0], p[0], acc, 0, 0, 0);
                if constexpr (i + 1 < n) read(IN{}, K1{}, pn);
                __builtin_amdgcn_sched_barrier(0);
                acs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[1], p[0], acs, 0, 0, 0);
                if constexpr (i + 1 < n) read(IN{}, K2{}, pn);
                __builtin_amdgcn_sched_barrier(0);
                acs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[1], p[1], acs, 0, 0, 0);
                acs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0], p[1], acs, 0, 0, 0);
                acs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0], p[2], acs, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }, std::make_integer_sequence<int, SPQ>{});
        floatx16 sum;
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v] = acc[v] + acs[v];
        if (__builtin_amdgcn_ballot_w64(!finite(largest(sum)))) {
            // (the small products of an infinity are NaN: the sum of the h*h products stands for it)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float big = acc[v];
                sum[v] = finite(big) ? sum[v] : big;
            }
        }
        return sum;
    };

    // ---- the wave's share of a block's outputs: registers OWN*ks .. of the sums, all of them scaled
    uint32_t lo = 0xffffffffu, hi = 0;   // (uniform) first and last tile with an infinite or NaN output
    // The lane's number again, worked out at each use: what depends on it alone would be kept through the loops, and a three-block workgroup
    // (168 registers to a wave) then reloads filter words in them (11x11, N=128 227x227 96 channels 176 -> 187 us).  11x11 in eight waves has
    // the registers (64 channels 132, so 137).
    auto fresh_lane = [&]() __attribute__((always_inline)) {
        int l = lane;
        if constexpr (Q < 4 || T::NW > 8) asm volatile("" : "+v"(l));
        return l;
    };
    auto first_channel = [&](int l) __attribute__((always_inline)) { return (T::OWN == 16 ? 0 : ks * (T::OWN / 4) * 8) + (l >> 5) * 4; };   // of the block
    // (7x7 in two parts has registers for the comparisons with the channels left: N=128 224x224 80 channels 294, worked out again 302)
    auto room_of = [&](int j0) __attribute__((always_inline)) {
        if constexpr (Q == 2) return P.Co - m0 - first_channel(lane);
        else return P.Co - m0 - j0;
    };
    auto settled = [&](auto bc, const __amdgpu_buffer_rsrc_t &ro, uint32_t voff, bool live, int j0, uint32_t img, uint32_t pin, auto &&sum) __attribute__((always_inline)) {
        settle_outputs<HF, HF, IMP, T::OWN, decltype(bc)::value>(P, ro, voff, live, P.Co - m0 - j0, img, m0 + j0, pin, [&](int b, int r, float &acc) __attribute__((always_inline)) {
            acc = sum(b, r);
            return acc * (1.0f / (kScale2 * kScale2));
        });
    };
    auto store = [&](auto secondc, auto fullc, uint32_t t, bool there, int blk, const auto &v) __attribute__((always_inline)) {
        const uint32_t P0 = t * T::TN, Pend = min(P0 + T::TN, P.npix) - 1u;
        const uint32_t pix = P0 + pixel(blk);
        const bool live = there && pix <= Pend;
        const uint32_t img0 = fdiv(P0, P.d_howo), img = fdiv(min(pix, Pend), P.d_howo);
        const uint32_t pin = min(pix, Pend) - img * P.howo;
        const __amdgpu_buffer_rsrc_t ro = output_desc(P.out, P.out_elems, ((size_t)img0 * P.Co + (size_t)min(m0, P.Co - 1)) * P.howo);
        const int j0 = first_channel(fresh_lane()), room = room_of(j0);
        uint32_t at = (((img - img0) * (uint32_t)P.Co + (uint32_t)j0) * P.howo + pin) * 4u;
        asm("" : "+v"(at));   // (computed by all lanes: no branch here either)
        const uint32_t voff = live ? at : kNoStore;
        if constexpr (decltype(secondc)::value) {
            settled(std::integral_constant<int, 1>{}, ro, voff, live, j0, img, pin, [&](int, int r) __attribute__((always_inline)) { return v[r]; });
        } else {
            // Every wave issues every store, the lanes that must not pass an offset that no descriptor covers: with their number fixed
            // the wait for the next tile's words counts past them instead of waiting for them.
            const uint32_t howo4 = P.howo * 4u;
            float o[T::OWN];
#pragma unroll
            for (int r = 0; r < T::OWN; ++r) o[r] = v[r] * (1.0f / (kScale * kScale));
            if (__builtin_amdgcn_ballot_w64(live && !finite(largest(o)))) { lo = min(lo, t); hi = t; }
#pragma unroll
            for (int r = 0; r < T::OWN; ++r) {
                const int dj = 8 * (r >> 2) + (r & 3);
                const uint32_t vo = decltype(fullc)::value || dj < room ? voff : kNoStore;
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, o[r]), ro, vo, (uint32_t)dj * howo4, 0);
            }
        }
    };

    // The same for the four neighbouring pixels of a lane, 16 bytes per channel (all inside the layer or all outside, in one plane).
    auto store_wide = [&](auto secondc, auto fullc, uint32_t t, const floatx16 (&v)[T::B]) __attribute__((always_inline)) {
        const uint32_t P0 = t * T::TN, Pend = min(P0 + T::TN, P.npix) - 1u;
        const uint32_t pix = P0 + pixel(0);
        const bool live = pix <= Pend;
        const uint32_t img0 = fdiv(P0, P.d_howo), img = fdiv(min(pix, Pend), P.d_howo);
        const uint32_t pin = min(pix, Pend) - img * P.howo;
        const __amdgpu_buffer_rsrc_t ro = output_desc(P.out, P.out_elems, ((size_t)img0 * P.Co + (size_t)min(m0, P.Co - 1)) * P.howo);
        const int j0 = first_channel(fresh_lane()), room = room_of(j0);
        uint32_t at = (((img - img0) * (uint32_t)P.Co + (uint32_t)j0) * P.howo + pin) * 4u;
        asm("" : "+v"(at));   // (computed by all lanes: no branch here either)
        const uint32_t voff = live ? at : kNoStore;
        if constexpr (decltype(secondc)::value) {
            settled(std::integral_constant<int, T::B>{}, ro, voff, live, j0, img, pin, [&](int b, int r) __attribute__((always_inline)) { return v[b][r]; });
        } else {
            const uint32_t howo4 = P.howo * 4u;
            float odd = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dj = 8 * (r >> 2) + (r & 3);
                u32v4 w;   // (element by element: a bit cast applied to a vector element reads element 0)
#pragma unroll
                for (int b = 0; b < T::B; ++b) {
                    const float o = v[b][r] * (1.0f / (kScale * kScale));
                    odd = __builtin_elementwise_maximum(odd, __builtin_fabsf(o));
                    w[b] = __builtin_bit_cast(uint32_t, o);
                }
                store_quad(w, ro, decltype(fullc)::value || dj < room ? voff : kNoStore, (uint32_t)dj * howo4);
            }
            if (__builtin_amdgcn_ballot_w64(live && !finite(odd))) { lo = min(lo, t); hi = t; }
        }
    };

    // Sums of the channels that other waves store go to LDS, [block][owner][source][quad][lane]; the wave's own stay.
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
    constexpr uint32_t QUADS = T::OWN / 4, SLOT = QUADS * 1024u;
    auto block_at = [&]() __attribute__((always_inline)) { return 2u * T::STAGE + (uint32_t)(rb * T::PX + px) * (Q * (Q - 1)) * SLOT + (uint32_t)fresh_lane() * 16u; };
    float own[T::OWN];
    auto hand_over = [&](auto qc, const floatx16 &sum, uint32_t red) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        const uint32_t block = block_at();
        stem_for([&](auto dc) __attribute__((always_inline)) {
            constexpr int d = decltype(dc)::value;
            if constexpr (d == q) {
#pragma unroll
                for (int r = 0; r < T::OWN; ++r) own[r] = sum[d * T::OWN + r];
            } else {
#pragma unroll
                for (uint32_t w = 0; w < QUADS; ++w) {
                    f32x4 v;
                    v.x = sum[d * T::OWN + w * 4]; v.y = sum[d * T::OWN + w * 4 + 1]; v.z = sum[d * T::OWN + w * 4 + 2]; v.w = sum[d * T::OWN + w * 4 + 3];
                    *(lds_f32x4 *)(L + block + red + (uint32_t)(d * (Q - 1) + (q < d ? q : q - 1)) * SLOT + w * 1024u) = v;
                }
            }
        }, std::make_integer_sequence<int, Q>{});
    };
    auto finish = [&](auto secondc, auto fullc, uint32_t t, bool there, uint32_t red) __attribute__((always_inline)) {
        const uint32_t block = block_at();
#pragma unroll
        for (int s = 0; s < Q - 1; ++s)
#pragma unroll
            for (uint32_t w = 0; w < QUADS; ++w) {
                const f32x4 v = *(const lds_f32x4 *)(L + block + red + (uint32_t)(ks * (Q - 1) + s) * SLOT + w * 1024u);
                own[w * 4] += v.x; own[w * 4 + 1] += v.y; own[w * 4 + 2] += v.z; own[w * 4 + 3] += v.w;
            }
        store(secondc, fullc, t, there, 0, own);
    };

    if (T::COLS && tid < 6) *(lds_bf16x8 *)(L + (uint32_t)(tid / 3) * T::STAGE + 2u * CHB + (uint32_t)(tid % 3) * PCB + PCB - 16u) = bf16x8{};

    // One pass over the tiles first, first + gx, ... below stop.  LATE: the wave stages before it multiplies.  FULL: all 32 channels of
    // the wave exist.  (Loops of their own, without a branch around a load or a store: the wait for a tile's words then counts past the
    // stores behind them.  7x7, 128 images: 227 us with branches.)  Past the last tile the last one's words are staged again.
    auto tiles = [&](auto secondc, auto latec, auto fullc, auto qc) __attribute__((always_inline)) {
        constexpr bool LATE = decltype(latec)::value;
        uint32_t at = 0, red = 0;
        for (uint32_t t = first; t < stop; t += gx) {
            auto next = [&]() __attribute__((always_inline)) {
                stage(at ^ T::STAGE);
                fetch(t + 2 * gx < stop ? t + 2 * gx : t);
            };
            if constexpr (LATE) next();
            if constexpr (Q > 1) {
                const floatx16 sum = multiply(qc, t, 0, at);
                finish(secondc, fullc, t == first ? t : t - gx, t != first, red ^ T::RED);
                hand_over(qc, sum, red);
            } else if constexpr (T::WIDE) {
                floatx16 sum[T::B];
#pragma unroll
                for (int b = 0; b < T::B; ++b) sum[b] = multiply(qc, t, b, at);
                store_wide(secondc, fullc, t, sum);
            } else {
#pragma unroll
                for (int b = 0; b < T::B; ++b) store(secondc, fullc, t, true, b, multiply(qc, t, b, at));
            }
            if constexpr (!LATE) next();
            at ^= T::STAGE;
            red ^= T::RED;
            lds_barrier();
        }
        if constexpr (Q > 1) finish(secondc, fullc, first + (stop - 1u - first) / gx * gx, true, red ^ T::RED);
    };
    auto run = [&](auto secondc, auto qc) __attribute__((always_inline)) {
        load_filter(qc);
        fetch(first);
        stage(0);
        fetch(first + gx < stop ? first + gx : first);
        lds_barrier();
        using Yes = std::true_type;
        using No = std::false_type;
        if constexpr (decltype(secondc)::value) {
            tiles(secondc, No{}, No{}, qc);
        } else if (m0 + 32 <= P.Co) {
            if (late) tiles(secondc, Yes{}, Yes{}, qc);
            else tiles(secondc, No{}, Yes{}, qc);
        } else {
            if (late) tiles(secondc, Yes{}, No{}, qc);
            else tiles(secondc, No{}, No{}, qc);
        }
    };
    auto pass = [&](auto secondc) __attribute__((always_inline)) {
        if (first >= stop) return;
        if constexpr (Q == 1) run(secondc, std::integral_constant<int, 0>{});
        else stem_for([&](auto qc) __attribute__((always_inline)) { if (ks == decltype(qc)::value) run(secondc, qc); }, std::make_integer_sequence<int, Q>{});
    };
    pass(std::false_type{});
    // a second pass over the tiles, from the first to the last that has an infinite or NaN output (see conv_split.h)
    if (lane == 0) *(lds_u32v2 *)(L + T::PASS + wave * 8) = u32v2{lo, hi};
    lds_barrier();
    uint32_t from = 0xffffffffu, to = 0;
#pragma unroll
    for (int w = 0; w < T::NW; ++w) {
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

template <int HF, int R, int Q, int PX, int B, bool IMP>
__global__ __launch_bounds__(64 * R * Q * PX, R * Q * PX < 8 ? 2 : R * Q * PX / 4) void conv_split_stem_kernel(StemParams P)
{
    extern __shared__ __align__(16) unsigned char smem[];
    conv_stem_body<Stem<HF, R, Q, PX, B>, IMP>(P, smem);
}

template <int HF, int R, int Q, int PX, int B = 1>
static hipError_t launch_stem_t(StemParams P, bool implicit, hipStream_t st, LaunchPlan *plan)
{
    using T = Stem<HF, R, Q, PX, B>;
    int dev = 0, ncu = 0;
    hipError_t e = device_cus(&dev, &ncu);
    if (e != hipSuccess && plan) { e = hipSuccess; ncu = 256; }   // planning without a device: an MI355X's 256 compute units
    if (e != hipSuccess) return e;
    // chunks that a tile may need: P0 anywhere in a row, rows of Wo pixels (the strides here are below HF: most rows, most columns)
    const long long rows = std::min<long long>((T::TN + P.Wo - 2) / P.Wo + 1, T::TN);
    const long long cols = ((long long)T::TN - rows) * P.s + rows * HF;
    const long long chunks = T::COLS ? cols + rows + 2 : (T::PAIRS ? cols / 2 + rows + 1 : (cols * HF) / 8 + rows + 1);   // (each row is rounded up; zeros; reads past the last)
    if (chunks > T::CAP) return hipErrorNotSupported;
    const unsigned long long imgs = std::min<unsigned long long>((unsigned long long)T::TN / P.howo + 2, (unsigned long long)P.N);
    // (of the larger of both calls' sources, so that they take the same kernel and give the same bits)
    const unsigned long long larger = std::max((unsigned long long)P.Hi * P.Wi, (unsigned long long)P.Ho * P.rowlen);
    if (imgs * 3ull * larger * 4ull >= (1ull << 31)) return hipErrorNotSupported;
    if (((unsigned long long)P.Co * imgs + 64ull) * P.howo * 4ull >= kNoStore) return hipErrorNotSupported;
    constexpr uint32_t kPerCu = T::NW < 8 && 2 * T::LDS <= 160 * 1024 ? 2 : 1;
    P.ntiles = (P.npix + T::TN - 1) / T::TN;
    const int mgroups = (P.Co + 32 * R - 1) / (32 * R);
    uint32_t gx = (uint32_t)ncu * kPerCu / (uint32_t)mgroups;
    if (gx >= 8) gx &= ~7u;   // (whole rows of the grid per XCD, whatever blockIdx.y)
    gx = std::max(1u, std::min(gx, P.ntiles));
    if (plan) {
        plan_record(plan, dim3(gx, mgroups), T::NT, T::LDS, "conv_split_stem_kernel<%d, %d, %d, %d, %d, %s>", HF, R, Q, PX, B, tf(implicit));
        return hipSuccess;
    }
    void (*kern)(StemParams) = implicit ? &conv_split_stem_kernel<HF, R, Q, PX, B, true> : &conv_split_stem_kernel<HF, R, Q, PX, B, false>;
    static KernelCache kc[2];
    if ((e = allow_dynamic_lds(kc[implicit], reinterpret_cast<const void *>(kern), T::LDS, dev)) != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(gx, mgroups), dim3(T::NT), T::LDS, st, P);
    return hipGetLastError();
}

// hipErrorNotSupported where the layer has no instance here or the fp32 kernel (conv_mfma_shallow.hip) is the faster one.
hipError_t launch_conv_split_stem(const float *src, const float *flt, float *out, const Shape &sh, hipStream_t st, bool implicit, LaunchPlan *plan)
{
    if (sh.Ci != 3 || sh.Hf != sh.Wf) return hipErrorNotSupported;
    if (!(sh.Hf == 3 && sh.s <= 2) && !(sh.Hf == 7 && sh.s == 2) && !(sh.Hf == 11 && sh.s == 4)) return hipErrorNotSupported;
    StemParams P = {};
    P.src = src; P.flt = flt; P.out = out;
    P.N = sh.N; P.Ci = sh.Ci; P.Ho = sh.Ho; P.Wo = sh.Wo; P.Co = sh.Co; P.s = sh.s; P.K = sh.K;
    P.Hi = sh.Hi; P.Wi = sh.Wi; P.p = sh.p; P.rowlen = sh.rowlen;
    P.plane = implicit ? (uint32_t)(sh.Hi * sh.Wi) : (uint32_t)((size_t)sh.Ho * sh.rowlen);
    P.howo = (uint32_t)(sh.Ho * sh.Wo); P.npix = (uint32_t)sh.npix;
    P.src_elems = (size_t)sh.N * 3u * P.plane; P.out_elems = (size_t)sh.npix * sh.Co;
    const int cols = (sh.Wo - 1) * sh.s + sh.Wf;
    P.chf = sh.Hf == 7 ? (cols + 1) & ~1 : (sh.Hf == 3 ? (cols + 1) >> 1 : (cols * sh.Hf + 7) >> 3);
    P.d_wo = make_fastdiv((uint32_t)sh.Wo); P.d_ho = make_fastdiv((uint32_t)sh.Ho);
    P.d_howo = make_fastdiv(P.howo); P.d_chf = make_fastdiv((uint32_t)P.chf);
    const int blocks = (sh.Co + 31) / 32;
    int dev = 0, ncu = 0;
    if (device_cus(&dev, &ncu) != hipSuccess) ncu = 256;   // (planning without a device)
    const uint32_t per_cu = P.npix / (uint32_t)ncu;   // pixels
    // Which instance: us, two calls / workspace-free (convolution only).
    if (sh.Hf == 3) {
        // Stride 2: 224x224, padding 1, N=8 16 channels 13.0 / 13.7, here 11.3 / 12.2; 64 channels 15.7 / 16.3, 12.5 / 15.2; N=64 16 channels
        // 74 / 75, 33 / 42; 64 channels 88 / 85, 50 / 57; 96 channels 198 / 180, 91 / 128.  Small layers (500 of all sizes): two calls gain 6 to
        // 40 %; workspace-free, where a workgroup has one or two tiles, up to 7 % is lost (N=77 8x138 124 channels 10.3 / 10.7, here 9.7 / 11.5) and 12 % gained.
        if (sh.s == 2) {
            // An odd count of blocks, three or more: single blocks stage each pixel once per block, pairs leave one block empty.  Pairs where a
            // workgroup has few tiles (in pairs / single: 96 channels, N=1 313x313 9.1 / 10.8, 10.5 / 13.0; 160 channels, N=14 158x127 18.1 / 21.8,
            // 19.7 / 24.6), but not where single ones have a unit each (N=8 51x51 96 channels 6.4 / 7.8, 5.8 / 7.4) or save a second round (N=18 66x66
            // 9.1 / 10.9, 8.2 / 10.2); behind four rounds neither always wins (N=35 191x191 96 channels 40 / 49, 37 / 48; N=57 120x506 127 / 156, 141 / 166).
            const uint32_t tiles = (P.npix + 127) / 128, units = (uint32_t)ncu;
            auto rounds = [&](uint32_t slots, uint32_t groups) { const uint32_t gx = std::max(1u, slots / groups >= 8 ? slots / groups & ~7u : slots / groups); return (tiles + gx - 1) / gx; };
            const uint32_t r1 = rounds(2 * units, (uint32_t)blocks), r2 = rounds(units, (uint32_t)(blocks + 1) / 2);
            const bool single = blocks % 2 && (blocks == 1 || (unsigned long long)tiles * blocks <= units || (r1 == 1 && r2 > 1) || r1 > 4);
            if (single) return launch_stem_t<3, 1, 1, 4>(P, implicit, st, plan);
            return launch_stem_t<3, 2, 1, 4>(P, implicit, st, plan);
        }
        // At stride 1 the output stream is the bound, and with 64 channels the fp32 kernel, whose tiles are half as long, keeps it fuller (N=128
        // 222x222 outputs 369, here 432; tiles of that length here 413, a group of 32 channels each 441).  With an odd number of blocks
        // it runs groups of 32 channels too and is bound by their matrix work: N=128, 222x222 16 channels 278 / 330, here 167 / 194;
        // 96 channels 940 / 1086, 787 / 729; N=16 96 channels 122 / 136, 80 / 95.  Below 2048 pixels per unit, or where a lane's four pixels may
        // lie in two planes (N=128 223x223 96 channels 714 / 755, here 959 / 867), it is the faster; with 32 channels, none of them missing, up to
        // 3072, where it goes over to tiles of 256 pixels (N=201 54x54 24.8 / 29.3, here 28.3 / 31.5; N=109 74x74 25.2 / 30.2, 28.7 / 31.9; 3069
        // pixels per unit 1.01 / 1.14 times as fast here, 3600 1.3; 16 channels, 2048 to 3072 1.1 to 1.4).  (Even counts from four blocks run
        // groups of 32 there as well: N=128, 222x222 128 channels 1220 / 1361, here 1019 / 936; N=16 153 / 169, 99 / 119; but 836 / 966, 1043 / 902
        // off alignment.  Not taken here.)
        // The alignment of the output chooses nothing: 16-byte stores need four bytes.  At 4 or 8 mod 16, fp32 kernel with 4-byte
        // stores -> here: N=128 222x222 16 channels 214 / 248 -> 170 / 197, 96 channels 708 / 746 -> 806 / 738, N=16 96 channels 93 / 99 -> 84 / 99
        // (4-byte stores here 234 / 232, 793 / 1020, 108 / 125).
        if (blocks % 2 == 0 || P.howo % 4u != 0 || per_cu < (sh.Co == 32 ? 3072u : 2048u)) return hipErrorNotSupported;
        return launch_stem_t<3, 1, 1, 4, 4>(P, implicit, st, plan);
    }
    if (sh.Hf == 7) {
        // Up to 64 channels and a tile or less per compute unit the fp32 kernel's shorter start is the faster (where it takes the layer:
        // at most three output rows per 64 pixels): 64 channels, N=1 224x224 10.9 / 11.7, here 11.3 / 13.2; N=2 16.6 / 17.5, here 13.4 / 15.8;
        // 24 channels, N=1 11.2 / 10.5, 11.2 / 12.5; N=2 12.9 / 15.5, 11.4 / 12.6.
        if (blocks <= 2 && per_cu < 64 && sh.Wo > 31) return hipErrorNotSupported;
        // Otherwise at any size (500 layers of all sizes: at least 1.08 times as fast in two calls, 1.02 workspace-free).
        if (blocks == 1) return launch_stem_t<7, 1, 2, 4>(P, implicit, st, plan);
        if (blocks == 3) return launch_stem_t<7, 3, 2, 2>(P, implicit, st, plan);
        // K in one wave or two: one cuts twice the filter words at its start, but nothing is exchanged.  64 channels, N=8 224x224
        // 25.3 / 28.7, in two 22.6 / 27.3; N=32 160x160 35.5 / 39.8, 34.9 / 41.7; N=128 224x224 204 / 217, 234 / 259.
        if (per_cu < 768) return launch_stem_t<7, 2, 2, 2>(P, implicit, st, plan);
        return launch_stem_t<7, 2, 1, 4>(P, implicit, st, plan);
    }
    // Two or more blocks: at any size (331 layers of all sizes: at least 1.37 times as fast as on the fp32 kernels in two calls, 1.14
    // workspace-free).  One block: its own instance from four rounds of the other's tiles, whose one half is empty then; behind five
    // with a full block, whose stores cost it more.
    if (blocks == 1 && per_cu >= (sh.Co > 24 ? 161u : 128u)) {
        // 24 channels, N=8 227x227 15.1 / 25.8, with half of the tile empty (below) 16.3 / 20.4; N=7 273x273 16.9 / 26.6, 17.7 / 24.4; N=16 255x255
        // 21.0 / 31.2, 24.8 / 33.5; N=128 227x227 72 / 131, 132 / 155; fp32 kernel 18.0 / 21.9, 20.7 / 26.0, 25.0 / 31.9, 100 / 136.  8 channels, N=28
        // 155x155 14.5 / 23.6, 16.5 / 23.3; fp32 17.8 / 23.2.  32 channels, N=9 261x261 19.8 / 28.8, 19.4 / 26.1; fp32 22.2 / 27.1.  (Not for narrow images.)
        const hipError_t e = launch_stem_t<11, 1, 4, 2>(P, implicit, st, plan);
        if (e != hipErrorNotSupported) return e;
    }
    if (blocks <= 2) return launch_stem_t<11, 2, 4, 1>(P, implicit, st, plan);
    return launch_stem_t<11, 3, 4, 1>(P, implicit, st, plan);
}

}  // namespace im2win
