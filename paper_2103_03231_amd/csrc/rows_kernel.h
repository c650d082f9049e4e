// rows_kernel.h - the fused per-ray kernel split by network rows (gfx950).
//
// render_kernel.h gives each wave 32 rays and streams every weight through
// LDS to all waves: 256 rays share one copy of the weights, which suits
// frames that fill the chip, but a call of a few thousand rays then occupies
// a few of the 256 CUs, and a lone tile takes 16 layers x 4 barriers-and-copies
// one after the other.  Here a workgroup of 8 waves renders R = 32 CB rays
// (CB = 1 or 2): wave w computes the output rows 32 w .. 32 w + 31 of every
// layer for all R columns.  Its weights come straight from L2 into registers,
// requested one layer (or a few K steps) ahead, each wave its own rows, and the
// activations (the MFMA B operand) pass from layer to layer through LDS in
// 16-byte units that the next layer reads as they are.  What bounds it is the
// L2 read of a whole layer per R rays: small tiles trade that for using more
// CUs.  Measured per layer and workgroup, every CU busy: bf16 R = 32 2,400
// cycles for 128 KiB (53 of the 64 bytes per cycle a CU takes from L2), R = 64
// 3,250 (2,048 of them MFMAs); fp8 R = 32 1,550 for 64 KiB.  fp32 R = 64 is bound
// by its MFMAs (12,288 cycles per layer, 63 % of all) and the epilogues between.
//
// bf16 and fp8 networks run the same MFMA steps on the same packed fragments in
// the same K order as render_kernel.h, so scores, classes and samples are
// bit-identical whichever of the two renders a ray.  Against that kernel's tiles
// of 256 rays, 83 x 61 rays, N = 2, B = 64: 65.4 -> 30 us (tiles of 32); 128 x
// 128, N = 4: 80 -> 66 us (tiles of 64).
//
// fp32 networks run on this kernel alone, on bf16 matrix cores: every fp32
// value is the exact sum of three bf16 values, so a product is six bf16 MFMA
// products (the three left out are below 2^-24 of it, either sign):
// w1 x1 in one fp32 accumulator, w1 x2 + w2 x1 + w2 x2 + w1 x3 + w3 x1 in a
// second, added at the end.  Six steps of 1,024 FLOP per cycle and SIMD against
// 64 for v_mfma_f32_32x32x2_f32: 2.7 times the rate of the fp32 instruction.
// Against fp32 MFMAs in 128-ray tiles: 400 x 400, N = 4, 4,927 -> 2,946 us
// (MFMA pipes 63 % busy, 88 % before), 32 x 32 (tiles of 32 rays: 128 CUs, 32
// before) 410 -> 66.6 us.  The images' error against 64 bits (2-norm, relative)
// falls by 1.8: 7.1e-7 -> 4.0e-7 and 3.4e-7 -> 1.8e-7 (two 400 x 400 images), 2.5e-7
// -> 1.4e-7 (32 x 32); a ray whose N-th and next class are a near-tie may select
// either, with either arithmetic.
#pragma once

#include "render_kernel.h"

namespace donerf {
namespace {

constexpr int kRowThreads = 64 * kRowWaves;

// A layer's 1 KiB fragments as the kernel addresses them, counted from the
// start of its network's stream: the offset of the layer and of wave w's
// first fragment in it.  bf16 / fp8: the chunk-padded streams of layout.h.
// fp32: layout.h rows32_* (three fragments per K step, no padding).
DN_HD constexpr int rows_layer_frags(int net, int kind, int n_bins) {
    return net == kF32 ? rows32_layer_frags(kind, n_bins) : layer_chunks(net, kind, n_bins) * kChunkFrags;
}

// A pointer to weights that the compiler cannot see through: loads that every
// sample makes again are loop-invariant, and hoisted out they would be held in
// registers throughout.  It passes the asm as a pointer to global memory: from a
// generic one the loads would be flat_load, which take a 64-bit address in VGPRs
// each, count as LDS accesses too and so make every wait a wait for all (fp32, 400 x
// 400, N = 4: 3,072 -> 2,982 us; 32 x 32: 72.4 -> 66.8; 128 x 128, bf16, 3 % less).
__device__ __forceinline__ const u32x4* opaque(const u32x4* p) {
    auto q = (const __attribute__((address_space(1))) u32x4*)p;
    asm volatile("" : "+s"(q));
    return (const u32x4*)q;
}

// ------------------------------------------------------------------ fp32 as three bf16

// x = p0 + p1 + p2 exactly, each a bf16: x rounded to nearest, then what is
// left, then the rest (both differences are exact and need at most 16 and 8
// bits; below 2^-110 the last bits of the rest fall under bf16's subnormals).
// Rounding rather than truncating halves the second plane, gives it either sign,
// and so makes the dropped products smaller and unbiased.  Eight values become
// one 16-byte unit per plane.  An infinity (and a finite value that rounds to one,
// from 0x1.ffp127 on) is an infinite p0 and NaN in the others; NaN is three NaN.
__device__ __forceinline__ void split3(const float* f, u32x4 (&o)[3]) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        float x = f[2 * w], y = f[2 * w + 1];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const uint32_t h = pack_bf16x2(x, y);
            o[p][w] = h;
            x -= __uint_as_float(h << 16);
            y -= __uint_as_float(h & 0xFFFF0000u);
        }
    }
}

// A sum from its two accumulators.  Non-finite operands make hi what the fp32
// sum would be (infinite, or NaN) and lo anything, and a hi that overflows may
// meet an infinite lo of the other sign: held to finite values (v_med3_f32
// gives a finite one for NaN), lo leaves such a hi as it is.  The instruction per
// value costs 1 % (400 x 400, N = 4, and 32 x 32 alike); looking for such a lo over
// the wave first (v_maximum3_f32, a branch) costs 0.6 % and 1.9 %.
template <class V>
__device__ __forceinline__ V join(V hi, V lo) {
#pragma unroll
    for (int i = 0; i < (int)(sizeof(V) / 4); ++i)
        hi[i] = hi[i] + __builtin_amdgcn_fmed3f(lo[i], -3.402823466e38f, 3.402823466e38f);
    return hi;
}

// The six products of one K step: a[], b[] hold the three planes.
__device__ __forceinline__ void mma_split32(const u32x4* a, const u32x4* b, f32x16& hi, f32x16& lo) {
    auto m = [](const u32x4& x, const u32x4& y, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c,
                                                       0, 0, 0);
    };
    lo = m(a[2], b[0], lo);
    hi = m(a[0], b[0], hi);
    lo = m(a[0], b[2], lo);
    lo = m(a[1], b[1], lo);
    lo = m(a[1], b[0], lo);
    lo = m(a[0], b[1], lo);
}
__device__ __forceinline__ void mma_split16(const u32x4* a, const u32x4* b, f32x4& hi, f32x4& lo) {
    lo = mma16(a[2], b[0], lo);
    hi = mma16(a[0], b[0], hi);
    lo = mma16(a[0], b[2], lo);
    lo = mma16(a[1], b[1], lo);
    lo = mma16(a[1], b[0], lo);
    lo = mma16(a[0], b[1], lo);
}

// ------------------------------------------------------------------ encoding, one unit at a time

// Slot s of the encoding of v in fourier()'s order and arithmetic: s / 6 the
// frequency pair, s % 3 the coordinate, sine or cosine.
template <int S>
__device__ __forceinline__ float fourier_slot(const float (&v)[3], int g) {
    const float y = v[S % 3] * ((float)(1u << (2 * (S / 6))) * 0.5f * (g ? 2.0f : 1.0f));
    const float r = y - __builtin_rintf(y);
    return S % 6 < 3 ? __builtin_amdgcn_sinf(r) : __builtin_amdgcn_cosf(r);
}

// Argument q of an encoding by pairs (layout.h pair_feature), for fp32 features:
// sincospif avoids multiplying by a rounded pi.
__device__ __forceinline__ void fourier_pair(const float (&v)[3], int q, float& sn, float& co) {
    const int f = q / 3, c = q - 3 * f;
    sincospif((c == 0 ? v[0] : c == 1 ? v[1] : v[2]) * (float)(1u << f), &sn, &co);
}

// ------------------------------------------------------------------ selection over the lanes of a ray

// Top-N of a ray whose classes are spread over LANES neighbouring lanes:
// every lane keeps a best-first list of its own classes, then lists are
// merged pairwise.  Two best-first lists a, b hold the best NCAP of both in
// max(a[k], b[NCAP - 1 - k]), a bitonic sequence that log2(NCAP) stages of
// compare-exchange sort: NCAP + NCAP log2(NCAP) f64 operations per merge
// where inserting one list into the other takes 2 NCAP^2.
// The partners are DPP permutations within a row of 16 lanes: neighbours,
// pairs, and the mirrors of 8 and 16 lanes (which pair the two halves, whose
// lanes hold equal lists by then).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int NCAP, int LANES>
__device__ __forceinline__ void merge_lanes(TopList<NCAP>& top) {
    static_assert(LANES == 8 || LANES == 16, "lanes of a ray lie in one DPP row");
    using TL = TopList<NCAP>;
    sfor<(LANES == 16 ? 4 : 3)>([&](auto M) {
        // quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror
        constexpr int ctrl = CV(M) == 0 ? 0xB1 : CV(M) == 1 ? 0x4E : CV(M) == 2 ? 0x141 : 0x140;
        double w[NCAP];
#pragma unroll
        for (int k = 0; k < NCAP; ++k) w[k] = TL::kmax(top.v[k], dpp_f64<ctrl>(top.v[NCAP - 1 - k]));
#pragma unroll
        for (int h = NCAP / 2; h >= 1; h >>= 1)
#pragma unroll
            for (int k = 0; k < NCAP; ++k)
                if ((k & h) == 0) {
                    const double x = w[k], y = w[k + h];
                    w[k] = TL::kmax(x, y);
                    w[k + h] = TL::kmin(x, y);
                }
#pragma unroll
        for (int k = 0; k < NCAP; ++k) top.v[k] = w[k];
    });
}

// The N best of a ray's B classes in ascending order, lane part of LANES taking
// the blocks part, part + LANES, ... of four classes; block(b): their scores.
template <int NCAP, int LANES, class Block>
__device__ __forceinline__ void lanes_topn(Block&& block, int part, int B, int N, int (&sel)[NCAP]) {
    TopList<NCAP> top;
    top.init();
    for (int b = part; b < B / 4; b += LANES) {
        const u32x4 s = block(b);
#pragma unroll
        for (int j = 0; j < 4; ++j) top.push(__uint_as_float(s[j]), 4 * b + j);
    }
    merge_lanes<NCAP, LANES>(top);
    top.ascending(N, sel);
}

// ------------------------------------------------------------------ the kernel body

// PR: network precision.  CB: 32-ray column blocks.  NCAP: capacity of the
// top-N list (top-N only).  CDF: inverse-CDF placement (B <= 128 and wider
// alike).  DIN: depth-network input.
template <int PR, int CB, int NCAP, bool CDF, int DIN>
struct RowsRender {
    static constexpr int R = 32 * CB;
    static constexpr int CT = 2 * CB;                    // 16-column tiles
    static constexpr bool F32 = PR == kF32;
    static constexpr int PL = F32 ? 3 : 1;               // planes of a unit
    static constexpr int KS_D0 = kDKPad / 16, KS_S0 = kSKPad / 16, KS_H = kHidden / 16;
    // Activations: 32 units of 16 bytes per column and plane.  Two buffers
    // (a layer writes the one it does not read: one barrier per layer) unless
    // they would not fit.
    static constexpr int kActUnits = PL * 32 * R;
    static constexpr int NBUF = kActUnits * 16 * 2 <= 96 * 1024 ? 2 : 1;
    // Scores (or class values) of a ray: unit b holds classes 4 b .. 4 b + 3;
    // the row of a unit is padded by 4 columns so that the lanes of one ray,
    // on neighbouring units, start in other banks.
    static constexpr int kScoreRow = R + 4;
    static constexpr int kPreStride = 65;                // a ray's CDF prefix, odd
    static constexpr int kPoolUnits0 = NBUF * kActUnits;
    static constexpr int kPoolUnits1 = 64 * kScoreRow + (CDF ? (R * kPreStride + 3) / 4 : 0);
    static constexpr int kPoolUnits = kPoolUnits0 > kPoolUnits1 ? kPoolUnits0 : kPoolUnits1;
    static constexpr int SCAP = CDF ? kMaxSamples : NCAP;   // samples a ray's row holds

    struct Shared {
        u32x4 pool[kPoolUnits];
        u32x4 skip[PL * 4 * R];                          // direction skip: 4 units
        float bias[kBiasMax];
        float bins[2 * 256];
        float geo[9][R];                                 // o, r, v = (unified origin - c) / d_max
        float samp[SCAP][2][R];                          // depth, width
        int32_t cls[SCAP][R];
    };
    static_assert(sizeof(Shared) <= 160 * 1024, "one workgroup's LDS");

    const RenderArgs& a;
    Shared& sh;
    int lane, wave, g, col, G, c16;

    // LDS unit of K step ks of a 32x32x16 step, lane group g: the bf16
    // networks number units for their 16x16x32 steps (layout.h
    // chained16_from32), the others in 32x32 order.
    __device__ __forceinline__ int unit32(int ks) const {
        return hid16(PR) ? 4 * (ks >> 1) + 2 * g + (ks & 1) : 2 * ks + g;
    }
    __device__ __forceinline__ u32x4* buf(int b) const { return sh.pool + (NBUF == 2 ? b * kActUnits : 0); }
    // ---- weights.  A wave reads the fragments of its own rows straight from
    // L2, kHeld of them ahead: they travel through one ring of registers that
    // runs on from layer to layer (fragment i of a stage in slot i % kHeld; each
    // one used is replaced by the one kHeld further on, in this stage or the
    // next).  bf16: a whole layer ahead.  fp32: four K steps of three planes.
    static constexpr int kHeld = F32 ? 12 : PR == kBF16 ? 16 : 8;
    u32x4 ring[kHeld];

    // Where fragment i of a wave's rows lies in a stage, counted from the
    // wave's first: fp32 stages are contiguous; bf16 and fp8 hidden layers
    // interleave the two waves of a pass by pairs of fragments, the other
    // layers one by one.
    enum Map { kLinear, kPairs, kSingles };
    static constexpr Map kHidMap = F32 ? kLinear : kPairs, kOneMap = F32 ? kLinear : kSingles;
    DN_HD static constexpr int at(Map m, int i) { return m == kLinear ? i : m == kPairs ? (i / 2) * 4 + i % 2 : 2 * i; }
    // The wave's first fragment in a hidden layer, a first layer or head of KS
    // 16-element steps (row block rb).
    __device__ __forceinline__ int hid0() const {
        return F32 ? wave * 48 : ((wave >> 1) * (PR == kBF16 ? 8 : 4)) * 4 + 2 * (wave & 1);
    }
    __device__ __forceinline__ static int one0(int rb, int KS) {
        return F32 ? 3 * rb * KS : (rb >> 1) * KS * 2 + (rb & 1);
    }
    template <Map M, int SLOT0 = 0>
    __device__ __forceinline__ void preload(const u32x4* w) {
        sfor<kHeld>([&](auto I) { ring[(CV(I) + SLOT0) % kHeld] = w[at(M, CV(I)) * 64 + lane]; });
    }
    // Fragments I .. I + NF - 1 of a stage of F (mapping M, from w) are used:
    // request their successors (the next stage: mapping MN, from wn).
    template <int F, Map M, Map MN, int I, int NF, int SLOT0 = 0>
    __device__ __forceinline__ void refill(const u32x4* w, const u32x4* wn) {
        sfor<NF>([&](auto J) {
            constexpr int i = I + CV(J), n = i + kHeld;
            ring[(i + SLOT0) % kHeld] = n < F ? w[at(M, n) * 64 + lane] : wn[at(MN, n < F ? 0 : n - F) * 64 + lane];
        });
    }

    // ---- layers.  in and out: activation buffers; bv[..] holds the next
    // kBAhead K steps' B operands.
    template <int N>
    __device__ __forceinline__ static void zero(f32x16 (&x)[N]) {
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) x[j][i] = 0.0f;
    }
    static constexpr int kBAhead = F32 ? 1 : CB == 1 ? 3 : 2;

    // KS steps of 16 K on 32x32x16 MFMAs for row block rows, into acc; unit(ks):
    // the LDS unit of step ks for this lane; NC column blocks from cb0 on.  The
    // fragments come from the ring (a stage of KS * PL), whose next stage is wn.
    template <int KS, Map MN, int SLOT0, int NC, class Unit>
    __device__ __forceinline__ void steps32(const u32x4* w, const u32x4* wn, int cb0, const u32x4* in, Unit unit,
                                            f32x16 (&acc)[NC]) {
        f32x16 lo[NC];
        if constexpr (F32) zero(lo);
        u32x4 bv[kBAhead + 1][NC][PL];
        auto read_b = [&](auto K) {
            constexpr int ks = CV(K);
#pragma unroll
            for (int j = 0; j < NC; ++j)
#pragma unroll
                for (int p = 0; p < PL; ++p)
                    bv[ks % (kBAhead + 1)][j][p] = in[(p * 32 + unit(ks)) * R + 32 * (cb0 + j) + col];
        };
        sfor<(kBAhead < KS ? kBAhead : KS)>(read_b);
        sfor<KS>([&](auto K) {
            constexpr int ks = CV(K);
            if constexpr (ks + kBAhead < KS) read_b(std::integral_constant<int, ks + kBAhead>{});
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const u32x4* b = bv[ks % (kBAhead + 1)][j];
                if constexpr (F32) mma_split32(&ring[(3 * ks + SLOT0) % kHeld], b, acc[j], lo[j]);
                else acc[j] = Prec<kBF16>::mma(&ring[(ks + SLOT0) % kHeld], b, acc[j], 127);
            }
            refill<KS * PL, kOneMap, MN, ks * PL, PL, SLOT0>(w, wn);
            __builtin_amdgcn_sched_barrier(0x6);
        });
        if constexpr (F32)
#pragma unroll
            for (int j = 0; j < NC; ++j) acc[j] = join(acc[j], lo[j]);
    }

    // first layers: units in 32x32 order (2 ks + g)
    template <int KS, int SLOT0>
    __device__ __forceinline__ void first_layer(const u32x4* w, const u32x4* wn, BiasAt bias, const u32x4* in,
                                                u32x4* out) {
        f32x16 acc[CB];
        const f32x16 b0 = bias_frag(bias + 32 * wave, g);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[cb] = b0;
        steps32<KS, kHidMap, SLOT0>(w, wn, 0, in, [&](int ks) { return 2 * ks + g; }, acc);
        emit32<PR>(acc, out);
    }

    // the folded positions layer: two fp32 steps of 8 K in every network
    __device__ __forceinline__ void first_layer_pos(const u32x4 (&av)[2], BiasAt bias, const u32x4* in, u32x4* out) const {
        f32x16 acc[CB];
        const f32x16 b0 = bias_frag(bias + 32 * wave, g);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[cb] = b0;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const u32x4 bv = in[(2 * ks + g) * R + 32 * cb + col];
                acc[cb] = Prec<kF32>::mma(&av[ks], &bv, acc[cb], 127);
            }
        emit32<PR>(acc, out);
    }

    // ReLU and rounding of this wave's 32-row block, written as the units of
    // the next layer's input in precision OUT.  With one buffer the rounding
    // comes before the barrier, where the older wave of a SIMD, done first,
    // runs it beside the younger one's MFMAs.
    template <int OUT>
    __device__ __forceinline__ void emit32(const f32x16 (&acc)[CB], u32x4* out) const {
        constexpr int NU = OUT == kFP8 ? 1 : 2;
        u32x4 o[CB][NU][PL];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            if constexpr (F32) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float f[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) f[i] = fmaxf(acc[cb][8 * h + i], 0.0f);
                    split3(f, o[cb][h]);
                }
            } else if constexpr (OUT == kFP8) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_fmed3f(acc[cb][4 * w + i], 0.0f, 448.0f);
                    // the first convert's kept half is overwritten by the second
                    uint32_t x = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], __builtin_bit_cast(int, v[0]), false);
                    o[cb][0][0][w] = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], (int)x, true);
                }
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        o[cb][h][0][w] = relu_bf16x2(acc[cb][8 * h + 2 * w], acc[cb][8 * h + 2 * w + 1]);
            }
        }
        if constexpr (NBUF == 1) {
            // held here: the compiler would sink the rounding past the barrier
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int h = 0; h < NU; ++h)
#pragma unroll
                    for (int p = 0; p < PL; ++p) asm volatile("" : "+v"(o[cb][h][p]));
            lds_barrier();
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int h = 0; h < NU; ++h)
#pragma unroll
                for (int p = 0; p < PL; ++p) {
                    // fp8: elements 16 (wave % 2) .. + 15 of K step wave / 2
                    const int unit = OUT == kFP8 ? 4 * (wave >> 1) + 2 * (wave & 1) + g : unit32(2 * wave + h);
                    out[(p * 32 + unit) * R + 32 * cb + col] = o[cb][h][p];
                }
    }

    // a hidden layer; the next stage (mapping MN) follows at wn; OUT: precision
    // of its output
    template <Map MN, int OUT>
    __device__ __forceinline__ void hidden(const u32x4* w, const u32x4* wn, BiasAt bias, const u32x4* in, u32x4* out,
                                           int sa) {
        if constexpr (PR == kBF16) {
            f32x4 acc[2][CT];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const f32x4 b = *reinterpret_cast<const f32x4*>(bias.s + (bias.off + 32 * wave + 16 * t + 4 * G));
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) acc[t][ct] = b;
            }
            u32x4 bv[kBAhead + 1][CT];
            auto read_b = [&](auto K) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    bv[CV(K) % (kBAhead + 1)][ct] = in[(4 * CV(K) + G) * R + 16 * ct + c16];
            };
            sfor<kBAhead>(read_b);
            sfor<8>([&](auto K) {
                constexpr int ks = CV(K);
                if constexpr (ks + kBAhead < 8) read_b(std::integral_constant<int, ks + kBAhead>{});
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        acc[t][ct] = mma16(ring[2 * ks + t], bv[ks % (kBAhead + 1)][ct], acc[t][ct]);
                refill<16, kHidMap, MN, 2 * ks, 2>(w, wn);
                __builtin_amdgcn_sched_barrier(0x6);
            });
            static_assert(NBUF == 2, "bf16 activations fit twice");
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const f32x4 &x = acc[0][ct], &y = acc[1][ct];
                out[(4 * wave + G) * R + 16 * ct + c16] = u32x4{relu_bf16x2(x[0], x[1]), relu_bf16x2(x[2], x[3]),
                                                                relu_bf16x2(y[0], y[1]), relu_bf16x2(y[2], y[3])};
            }
        } else {
            f32x16 acc[CB];
            const f32x16 b0 = bias_frag(bias + 32 * wave, g);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[cb] = b0;
            if constexpr (F32) {
                steps32<16, MN, 0>(w, wn, 0, in, [&](int ks) { return 2 * ks + g; }, acc);
            } else {
                sfor<4>([&](auto K) {
                    constexpr int ks = CV(K);
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        const u32x4 b[2] = {in[(4 * ks + g) * R + 32 * cb + col], in[(4 * ks + 2 + g) * R + 32 * cb + col]};
                        acc[cb] = Prec<kFP8>::mma(&ring[2 * ks], b, acc[cb], sa);
                    }
                    refill<8, kHidMap, MN, 2 * ks, 2>(w, wn);
                });
            }
            emit32<OUT>(acc, out);
        }
    }
    // six hidden layers from fragment stream w (the wave's first fragment of
    // layer 0), inputs and outputs alternating between the buffers, the first
    // input in buffer 1; the caller publishes the last output
    template <Map MN>
    __device__ __forceinline__ void hidden6(const u32x4* w, const u32x4* wn, int bias_off, const int32_t* ws) {
        constexpr size_t HF = (size_t)rows_layer_frags(PR, kHiddenL, 128) * 64;
        for (int l = 0; l < 5; ++l) {
            hidden<kHidMap, PR>(w + l * HF, w + (l + 1) * HF, BiasAt{sh.bias, bias_off + 256 * l}, buf(1 - (l & 1)),
                                buf(l & 1), ws[l]);
            lds_barrier();
        }
        hidden<MN, PR == kFP8 ? kBF16 : PR>(w + 5 * HF, wn, BiasAt{sh.bias, bias_off + 256 * 5}, buf(0), buf(1), ws[5]);
    }

    // ---- placement from the ray's scores in the pool; N samples per ray to
    // sh.samp and sh.cls
    static constexpr int LPR = kRowThreads / R;   // lanes per ray: 16 or 8
    __device__ __forceinline__ void select_topn() const {
        const int ray = wave * (64 / LPR) + lane / LPR, part = lane % LPR;
        int sel[NCAP];
        lanes_topn<NCAP, LPR>([&](int b) { return sh.pool[b * kScoreRow + ray]; }, part, a.B, a.N, sel);
        if (part == 0) {
#pragma unroll
            for (int k = 0; k < NCAP; ++k)
                if (k < a.N) {
                    const int bin = min(sel[k], a.B - 1);
                    sh.cls[k][ray] = sel[k];
                    sh.samp[k][0][ray] = sh.bins[bin];
                    sh.samp[k][1][ray] = sh.bins[a.B + bin];
                }
        }
    }

    // Inverse CDF (Sec. 5.1): the arithmetic of render_kernel.h's cdf_place
    // (B <= 128) or of its two-sweep form (B > 128), step by step.  bsum: each
    // 4-class block's sum, in the ray's prefix row at b + 1.
    __device__ __forceinline__ float* pre_row(int ray) const {
        return reinterpret_cast<float*>(sh.pool + 64 * kScoreRow) + ray * kPreStride;
    }
    __device__ __forceinline__ void place_cdf() const {
        const int tid = 64 * wave + lane;
        const bool wide = a.B > 128;
        const int NB = wide ? 64 : 32, nb = a.B / 4;
        if (tid < R) {   // prefix in class order; blocks past the last add zeros
            float* p = pre_row(tid);
            float s = 0.0f;
            p[0] = 0.0f;
            for (int b = 0; b < NB; ++b) {
                s = s + (b < nb ? p[b + 1] : 0.0f);
                p[b + 1] = s;
            }
        }
        lds_barrier();
        auto to_depth = [&](float s) { return a.near + exp2f(s * a.log2_span1) - 1.0f; };  // inverse of Eq. 3
        const int NT = 2 * a.N - 1;   // N slice centres, N - 1 inner slice ends
        for (int task = tid; task < NT * R; task += kRowThreads) {
            const int t = task / R, ray = task % R;
            const float* p = pre_row(ray);
            const bool centre = t < a.N;
            const float m = (centre ? a.cdf_u[t] : a.cdf_u[kMaxSamples + t - a.N]) * p[NB];
            // the last block with prefix <= m (prefixes never decrease)
            int b = 0;
            for (int step = NB / 2; step >= 1; step >>= 1) b = p[b + step] <= m ? b + step : b;
            const float lo = p[b];
            float s;
            int k;
            if (b < nb || !wide) {
                const u32x4 u = b < nb ? sh.pool[b * kScoreRow + ray] : u32x4{0u, 0u, 0u, 0u};
                const float w0 = __uint_as_float(u[0]), w1 = __uint_as_float(u[1]), w2 = __uint_as_float(u[2]),
                            w3 = __uint_as_float(u[3]);
                const float r = wide ? m - lo : m, z = wide ? 0.0f : lo;
                const float c1 = wide ? w0 : lo + w0, c2 = c1 + w1, c3 = c2 + w2;
                const int j = (r >= c1 ? 1 : 0) + (r >= c2 ? 1 : 0) + (r >= c3 ? 1 : 0);
                const float base = j == 0 ? z : j == 1 ? c1 : j == 2 ? c2 : c3;
                const float aj = j == 0 ? w0 : j == 1 ? w1 : j == 2 ? w2 : w3;
                const float q = wide ? (r - base) * __builtin_amdgcn_rcpf(aj) : (r - base) / aj;
                const float frac = aj > 0.0f ? fminf(fmaxf(q, 0.0f), 1.0f) : 0.0f;
                k = 4 * b + j;
                s = wide ? ((float)k + frac) * (1.0f / (float)a.B) : ((float)k + frac) / (float)a.B;
            } else {
                k = 4 * b;
                s = m - lo;
            }
            if (centre) {
                sh.samp[t][0][ray] = to_depth(s);
                sh.cls[t][ray] = k;
            } else {
                sh.samp[t - a.N][1][ray] = to_depth(s);   // the slice's inner end, a width below
            }
        }
        lds_barrier();
        if (tid < R) {
            float edge = a.near;
            for (int i = 0; i < a.N; ++i) {
                const float end = i + 1 < a.N ? sh.samp[i][1][tid] : a.dmax;
                sh.samp[i][1][tid] = end - edge;
                edge = end;
            }
        }
    }

    // ---- the whole tile
    __device__ __forceinline__ void run() {
        const int tid = threadIdx.x;
        lane = tid & 63;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        g = lane >> 5;
        col = lane & 31;
        G = lane >> 4;
        c16 = lane & 15;
        // the wave's first fragment of every stage
        constexpr int KIND0 = DIN == kDinEncoded ? kDFirst : kDFirstPos;
        constexpr size_t D0F = rows_layer_frags(PR, KIND0, 128) * 64, HF = rows_layer_frags(PR, kHiddenL, 128) * 64,
                         S0F = rows_layer_frags(PR, kSFirst, 128) * 64;
        const u32x4* dstream = reinterpret_cast<const u32x4*>(a.d_frags);
        const u32x4* sstream = reinterpret_cast<const u32x4*>(a.s_frags);
        const int nrb = a.B / 32, groups = nrb <= 4 ? kRowWaves / nrb : 1;   // depth head: row blocks, waves on one
        const int rb = wave % nrb, cb0 = wave / nrb;
        const u32x4* d0 = dstream + one0(wave, KS_D0) * 64;
        const u32x4* dh = dstream + D0F + hid0() * 64;
        const u32x4* dhead = dstream + D0F + 6 * HF + one0(rb, KS_H) * 64;
        const u32x4* s0 = sstream + one0(wave, KS_S0) * 64;
        const u32x4* shd = sstream + S0F + hid0() * 64;
        const u32x4* shead = sstream + S0F + 6 * HF;

        // this workgroup's tile and its share of the samples
        const bool split_part = blockIdx.x >= a.n_full;
        const uint32_t cpart = blockIdx.x - a.n_full;
        const int nsplit = split_part ? a.split : 1;
        const int part = split_part ? (int)(cpart % (uint32_t)a.split) : 0;
        const uint32_t tile_local = split_part ? cpart / (uint32_t)a.split : 0;
        const uint32_t tile = split_part ? a.n_full + tile_local : blockIdx.x;
        const int k_begin = part * a.N / nsplit;
        const int k_end = (part + 1) * a.N / nsplit;
        const uint32_t ray0 = tile * R;

        // The encoded first layer's KS_D0 steps end at the ring's start again.
        constexpr int D0SLOT = F32 ? 6 : PR == kBF16 ? 10 : 2;
        static_assert((KS_D0 * PL + D0SLOT) % kHeld == 0, "the ring's phase after the first layer");
        u32x4 pos_w[2];
        if constexpr (DIN == kDinEncoded) {
            sfor<(KS_D0 * PL < kHeld ? KS_D0 * PL : kHeld)>(
                [&](auto I) { ring[(CV(I) + D0SLOT) % kHeld] = d0[at(kOneMap, CV(I)) * 64 + lane]; });
            // slots past the first layer's fragments: the first hidden layer's
            if constexpr (KS_D0 * PL < kHeld)
                sfor<kHeld - KS_D0 * PL>([&](auto I) {
                    ring[(KS_D0 * PL + CV(I) + D0SLOT) % kHeld] = dh[at(kHidMap, CV(I)) * 64 + lane];
                });
        } else {
            // two fp32 steps: pass of two row blocks, step, row block
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) pos_w[ks] = dstream[(((wave >> 1) * 2 + ks) * 2 + (wave & 1)) * 64 + lane];
            preload<kHidMap>(dh);
        }
        for (int k = tid; k < a.bias_len; k += kRowThreads) sh.bias[k] = a.bias[k];
        for (int k = tid; k < 2 * a.B; k += kRowThreads) sh.bins[k] = a.bins[k];
        if (tid < R) {
            const uint32_t r = ray0 + tid;
            const Ray ray = camera_ray(a, r < a.total_rays ? r : a.total_rays - 1);
            float ou[3];
            unify(a, ray, ou);
            const float c[3] = {a.cx, a.cy, a.cz};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                sh.geo[k][tid] = ray.o[k];
                sh.geo[3 + k][tid] = ray.r[k];
                sh.geo[6 + k][tid] = (ou[k] - c[k]) / a.dmax;
            }
        }
        lds_barrier();

        // ---- depth-network input and direction skip: unit (ks, g) of column
        // block cb is one task of a wave
        auto store_unit = [&](u32x4* dst, int stride, int unit, int c, const float* f) {
            if constexpr (F32) {
                u32x4 o[3];
                split3(f, o);
#pragma unroll
                for (int p = 0; p < 3; ++p) dst[(p * stride + unit) * R + c] = o[p];
            } else {
                dst[unit * R + c] = Prec<kBF16>::pack(f);
            }
        };
        constexpr int D_TASKS = (DIN == kDinEncoded ? KS_D0 : 2) * CB, K_TASKS = 2 * CB;
        for (int task = wave; task < D_TASKS + K_TASKS; task += kRowWaves) {
            const bool is_skip = task >= D_TASKS;
            const int tk = is_skip ? task - D_TASKS : task;
            const int ks = tk / CB, c = 32 * (tk % CB) + col;
            const float r[3] = {sh.geo[3][c], sh.geo[4][c], sh.geo[5][c]};
            const float v[3] = {sh.geo[6][c], sh.geo[7][c], sh.geo[8][c]};
            float f[8];
            if (is_skip) {
                if constexpr (F32) {
                    const int U = 2 * ks + g;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        fourier_pair(r, min(4 * U + i, 11), f[2 * i], f[2 * i + 1]);
                        if (U == 3) f[2 * i] = i == 0 ? r[0] : i == 1 ? r[2] : 0.0f, f[2 * i + 1] = i == 0 ? r[1] : 0.0f;
                    }
                } else {
                    sfor<2>([&](auto K) {
                        if (ks == CV(K))
                            sfor<8>([&](auto E) {
                                constexpr int s = 8 * CV(K) + CV(E);
                                if constexpr (s < 12) f[CV(E)] = fourier_slot<s>(r, g);
                                else f[CV(E)] = s < 15 && !g ? r[s % 12 % 3] : 0.0f;
                            });
                    });
                }
                // K step 8 of the bf16 networks' 16x16 head reads unit
                // G = 2 g + ks, the others 2 ks + g
                store_unit(sh.skip, 4, hid16(PR) ? 2 * g + ks : 2 * ks + g, c, f);
            } else if constexpr (DIN == kDinEncoded) {
                if constexpr (F32) {
                    const int U = 2 * ks + g;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int q = 4 * U + i;
                        const float x[3] = {q < 30 ? v[0] : r[0], q < 30 ? v[1] : r[1], q < 30 ? v[2] : r[2]};
                        fourier_pair(x, q < 30 ? q : min(q - 30, 11), f[2 * i], f[2 * i + 1]);
                        // the identities, 84 .. 89, then zeros
                        if (q == 42) f[2 * i] = v[0], f[2 * i + 1] = v[1];
                        else if (q == 43) f[2 * i] = v[2], f[2 * i + 1] = r[0];
                        else if (q == 44) f[2 * i] = r[1], f[2 * i + 1] = r[2];
                        else if (q > 44) f[2 * i] = f[2 * i + 1] = 0.0f;
                    }
                } else {
                    sfor<KS_D0>([&](auto K) {
                        if (ks == CV(K))
                            sfor<8>([&](auto E) {
                                constexpr int s = 8 * CV(K) + CV(E);
                                if constexpr (s < 30) f[CV(E)] = fourier_slot<s>(v, g);
                                else if constexpr (s < 42) f[CV(E)] = fourier_slot<s - 30>(r, g);
                                else f[CV(E)] = s < 45 ? (g ? r[s % 3] : v[s % 3]) : 0.0f;
                            });
                    });
                }
                store_unit(buf(0), 32, 2 * ks + g, c, f);
            } else {
                // [u', r, u_c] in fp32: unit (ks, g) holds K 8 ks + 2 e + g
                const float q9[9] = {v[0], v[1], v[2], r[0], r[1], r[2], (sh.geo[0][c] - a.cx) / a.dmax,
                                     (sh.geo[1][c] - a.cy) / a.dmax, (sh.geo[2][c] - a.cz) / a.dmax};
                float q[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = g ? q9[2 * e + 1] : q9[2 * e];
                    const float hi = (e == 0 && g == 0) ? q9[8] : 0.0f;
                    q[e] = ks ? hi : lo;
                }
                buf(0)[(2 * ks + g) * R + c] = Prec<kF32>::pack(q);
            }
        }
        lds_barrier();

        // ---- depth network: input in buffer 0, layer l's output in buffer
        // 1 - l % 2
        if constexpr (DIN == kDinEncoded) first_layer<KS_D0, D0SLOT>(d0, dh, BiasAt{sh.bias, 0}, buf(0), buf(1));
        else first_layer_pos(pos_w, BiasAt{sh.bias, 0}, buf(0), buf(1));
        lds_barrier();
        hidden6<kOneMap>(dh, dhead, 256, a.wscale + 1);
        lds_barrier();
        // ---- depth head: waves over row blocks, then over column blocks.  The
        // ring runs on into the shading network: fp32 its first layer, which
        // the others keep in registers of their own, then its hidden layers.
        {
            // B <= 128: one column block per wave (waves past the last compute
            // the last one again and drop it); B > 128: all of them.
            auto head = [&](auto NCc, int first, bool active) {
                constexpr int NC = CV(NCc);
                f32x16 acc[NC];
                const f32x16 b0 = bias_frag(BiasAt{sh.bias, kDepthHeadBias + 32 * rb}, g);
#pragma unroll
                for (int j = 0; j < NC; ++j) acc[j] = b0;
                steps32<KS_H, F32 ? kOneMap : kHidMap, 0>(dhead, F32 ? s0 : shd, first, buf(1),
                                                          [&](int ks) { return unit32(ks); }, acc);
                lds_barrier();   // the activations are read: the scores take their place
                if (!active) return;
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    const int c = 32 * (first + j) + col;
                    if (a.out_scores && part == 0 && ray0 + c < a.total_rays) {
                        float* dst = a.out_scores + (size_t)(ray0 + c) * a.B + 32 * rb + 4 * g;
#pragma unroll
                        for (int i = 0; i < 16; ++i) dst[8 * (i / 4) + (i % 4)] = acc[j][i];
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int b = 8 * rb + 2 * q + g;
                        float v[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            v[i] = acc[j][4 * q + i];
                            if constexpr (CDF) v[i] = sigmoid<F32>(v[i]);
                        }
                        sh.pool[b * kScoreRow + c] = u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]),
                                                           __float_as_uint(v[2]), __float_as_uint(v[3])};
                        if constexpr (CDF) pre_row(c)[b + 1] = ((v[0] + v[1]) + v[2]) + v[3];
                    }
                }
            };
            if (CB == 1 || nrb <= 4) head(std::integral_constant<int, 1>{}, min(cb0, CB - 1), cb0 < CB && wave < nrb * groups);
            else head(std::integral_constant<int, CB>{}, 0, wave < nrb);
            lds_barrier();
            if constexpr (CDF) place_cdf();
            else select_topn();
            lds_barrier();
        }

        // ---- shading network per sample, composited front to back by the
        // lanes that hold the head's outputs: 16 columns per wave (16x16
        // head) or 32 (fp8 networks)
        constexpr bool H16 = PR != kFP8;
        constexpr int HW = H16 ? CT : CB;                // waves that run the head
        const int hc = H16 ? 16 * wave + c16 : 32 * wave + col;
        const bool composer = wave < HW && (H16 ? G == 0 : g == 0);
        const int s_bias = 7 * 256;
        float T = 1.0f, Cr = 0.0f, Cg = 0.0f, Cb = 0.0f, Dp = 0.0f;
        u32x4 s0w[KS_S0];
        if constexpr (!F32)
#pragma unroll
            for (int ks = 0; ks < KS_S0; ++ks) s0w[ks] = s0[at(kOneMap, ks) * 64 + lane];
        for (int k = k_begin; k < k_end; ++k) {
            // keeps the samples' equal weight loads inside the loop
            const u32x4 *s0k = opaque(s0), *shk = opaque(shd), *hk = opaque(shead);
            // the last head read buffer 1 (its only buffer, if there is one)
            if constexpr (NBUF == 1) lds_barrier();
            // tasks from the last wave down: the first waves run the head
            for (int task = kRowWaves - 1 - wave; task < KS_S0 * CB; task += kRowWaves) {
                const int ks = task / CB, c = 32 * (task % CB) + col;
                const float t = sh.samp[k][0][c];
                float x[3], w[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) x[i] = sh.geo[i][c] + t * sh.geo[3 + i][c];
                warp(a, x, w);
                float f[8];
                if constexpr (F32) {
                    const int U = 2 * ks + g;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int q = 4 * U + i;
                        fourier_pair(w, min(q, 29), f[2 * i], f[2 * i + 1]);
                        if (q == 30) f[2 * i] = w[0], f[2 * i + 1] = w[1];
                        else if (q > 30) f[2 * i] = w[2], f[2 * i + 1] = 0.0f;
                    }
                } else {
                    sfor<KS_S0>([&](auto K) {
                        if (ks == CV(K))
                            sfor<8>([&](auto E) {
                                constexpr int s = 8 * CV(K) + CV(E);
                                if constexpr (s < 30) f[CV(E)] = fourier_slot<s>(w, g);
                                else f[CV(E)] = s == 30 ? (g ? w[2] : w[0]) : (g ? 0.0f : w[1]);
                            });
                    });
                }
                store_unit(buf(0), 32, 2 * ks + g, c, f);
            }
            lds_barrier();
            if constexpr (F32) {
                first_layer<KS_S0, 0>(s0k, shk, BiasAt{sh.bias, s_bias}, buf(0), buf(1));
            } else {
                f32x16 acc[CB];
                const f32x16 b0 = bias_frag(BiasAt{sh.bias, s_bias + 32 * wave}, g);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[cb] = b0;
#pragma unroll
                for (int ks = 0; ks < KS_S0; ++ks)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        const u32x4 bv = buf(0)[(2 * ks + g) * R + 32 * cb + col];
                        acc[cb] = Prec<kBF16>::mma(&s0w[ks], &bv, acc[cb], 127);
                    }
                emit32<PR>(acc, buf(1));
            }
            lds_barrier();
            hidden6<F32 ? kOneMap : kHidMap>(shk, F32 ? s0k : shk, s_bias + 256, a.wscale + 9);
            // the head's first fragments are requested before the barrier
            constexpr int HS = H16 ? 9 : KS_H + 2, HA = F32 ? 1 : HS;   // its K steps, and those held
            u32x4 hw[HS][PL];
            if (wave < HW)
#pragma unroll
                for (int u = 0; u < HA; ++u)
#pragma unroll
                    for (int p = 0; p < PL; ++p) hw[u][p] = hk[(PL * u + p) * 64 + lane];
            lds_barrier();
            if (wave < HW) {
                const u32x4* in = buf(1);
                float h0, h1, h2, h3;
                if constexpr (H16) {
                    f32x4 acc = *reinterpret_cast<const f32x4*>(sh.bias + s_bias + 7 * 256 + 4 * G), lo = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int u = 0; u < 9; ++u) {
                        u32x4 bv[PL];
#pragma unroll
                        for (int p = 0; p < PL; ++p) {
                            if (u + HA < HS) hw[u + HA < HS ? u + HA : 0][p] = hk[(PL * (u + HA) + p) * 64 + lane];
                            bv[p] = u < 8 ? in[(p * 32 + 4 * u + G) * R + hc] : sh.skip[(p * 4 + G) * R + hc];
                        }
                        if constexpr (F32) mma_split16(hw[u], bv, acc, lo);
                        else acc = mma16(hw[u][0], bv[0], acc);
                    }
                    if constexpr (F32) acc = join(acc, lo);
                    h0 = acc[0], h1 = acc[1], h2 = acc[2], h3 = acc[3];
                } else {
                    f32x16 acc = bias_frag(BiasAt{sh.bias, s_bias + 7 * 256}, g);
#pragma unroll
                    for (int ks = 0; ks < HS; ++ks) {
                        const u32x4 bv = ks < KS_H ? in[(2 * ks + g) * R + hc] : sh.skip[(2 * (ks - KS_H) + g) * R + hc];
                        acc = Prec<kBF16>::mma(hw[ks], &bv, acc, 127);
                    }
                    h0 = acc[0], h1 = acc[1], h2 = acc[2], h3 = acc[3];
                }
                const float tk = sh.samp[k][0][hc], dk = sh.samp[k][1][hc];
                const float cr = sigmoid<F32>(h0), cg = sigmoid<F32>(h1), cbl = sigmoid<F32>(h2);
                const float tau = fmaxf(h3, 0.0f) * dk;
                const float wgt = T * one_minus_exp_neg<F32>(tau);
                Cr += wgt * cr;
                Cg += wgt * cg;
                Cb += wgt * cbl;
                Dp += wgt * tk;
                T *= exp_neg<F32>(tau);
            }
        }

        // ---- outputs
        const uint32_t rid = ray0 + hc;
        if (composer && rid < a.total_rays) {
            if (nsplit > 1) {
                float* q = a.partial + ((size_t)(tile_local * R + hc) * nsplit + part) * 5;
                q[0] = Cr;
                q[1] = Cg;
                q[2] = Cb;
                q[3] = Dp;
                q[4] = T;
            } else {
                float* o = a.out_rgb + (size_t)rid * 3;
                o[0] = Cr;
                o[1] = Cg;
                o[2] = Cb;
                if (a.out_depth) a.out_depth[rid] = Dp;
            }
            if (part == 0)
                for (int k = 0; k < a.N; ++k) {
                    if (a.out_bins) a.out_bins[(size_t)rid * a.N + k] = sh.cls[k][hc];
                    if (a.out_samples) {
                        a.out_samples[((size_t)rid * a.N + k) * 2 + 0] = sh.samp[k][0][hc];
                        a.out_samples[((size_t)rid * a.N + k) * 2 + 1] = sh.samp[k][1][hc];
                    }
                }
        }
    }
};

// Tiles of 32 CB rays: the main kernel of fp32 networks (64 rays: with 96 the
// three planes leave no LDS for the tables, with 32 every weight feeds half the
// work), and the tiles of calls too small to fill the chip with the main
// kernel's.
template <int PR, int CB, int NCAP, bool CDF, int DIN>
__global__ void __launch_bounds__(kRowThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
render_rows(const RenderArgs a) {
    using K = RowsRender<PR, CB, NCAP, CDF, DIN>;
    __shared__ typename K::Shared sh;
    K k{a, sh};
    k.run();
}

// A list of 8 pays on the fp32 tiles of 64 rays only: 4 or 16 otherwise.
template <int PR, int CB, bool CDF, int DIN>
hipError_t launch_rows_variant(int ncap, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    const dim3 block(kRowThreads);
    if constexpr (CDF) {
        hipLaunchKernelGGL((render_rows<PR, CB, 16, true, DIN>), grid, block, 0, stream, a);
    } else if (ncap == 4) {
        hipLaunchKernelGGL((render_rows<PR, CB, 4, false, DIN>), grid, block, 0, stream, a);
    } else {
        if constexpr (PR == kF32 && CB == kF32CB) {
            if (ncap == 8) {
                hipLaunchKernelGGL((render_rows<PR, CB, 8, false, DIN>), grid, block, 0, stream, a);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((render_rows<PR, CB, 16, false, DIN>), grid, block, 0, stream, a);
    }
    return hipGetLastError();
}

template <int PR, int CB>
hipError_t launch_rows(int cdf, int ncap, int din, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    if (din == kDinPositions)
        return cdf ? launch_rows_variant<PR, CB, true, kDinPositions>(ncap, a, grid, stream)
                   : launch_rows_variant<PR, CB, false, kDinPositions>(ncap, a, grid, stream);
    return cdf ? launch_rows_variant<PR, CB, true, kDinEncoded>(ncap, a, grid, stream)
               : launch_rows_variant<PR, CB, false, kDinEncoded>(ncap, a, grid, stream);
}

}  // namespace
}  // namespace donerf
