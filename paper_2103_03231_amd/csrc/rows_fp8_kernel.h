// rows_fp8_kernel.h - the fused per-ray kernel of mixed fp8 networks for
// frames that fill the chip (gfx950).
//
// E4M3 layers are short on the matrix cores (a 256 x 256 layer of 128 rays is
// 2,048 cycles of one SIMD) against their epilogue: ReLU, clamp and rounding of
// every value, about 1,800 VALU cycles.  VALU work of one wave costs the MFMAs of
// another nothing (measured: an MFMA stream runs as fast beside a stream of
// v_med3_f32 or v_cvt_pk_fp8_f32 from the SIMD's other wave), but waves that meet
// at one barrier do their epilogues together.  So two independent workgroups
// share a CU, one wave of each per SIMD, and wave priorities keep them apart:
// a wave's priority rises as it gets through a layer's K loop and drops in the
// epilogue, so whichever is ahead keeps the matrix core and the other one's
// epilogue runs beside it.
//
// A workgroup is 4 waves and 128 rays.  Wave w computes rows 64 w .. 64 w + 63 of
// every layer for all 128 columns (eight accumulation chains), its weights read
// from L2 into registers half a layer ahead, the activations passed on through
// LDS (32 KiB of E4M3 in each of two buffers; the heads' bf16 input takes both).
// An activation fragment read from LDS feeds two MFMAs, and no weight passes
// through LDS: half the LDS traffic of 32-ray waves that share a weight stream.
// Ray generation, encoding, selection and compositing go by rays: wave w owns
// rays 32 w .. 32 w + 31, lanes l and l + 32 the same ray, as in render_kernel.h.
//
// Measured against 32-ray waves on a shared weight stream (256-ray tiles, one
// workgroup per CU), in turn on one box: 5 x 400 x 400, N = 4: 1,379 -> 1,320 us
// (MFMA pipes busy 59 -> 67 %); 1920 x 1080, N = 2, 192 classes: 2,270 -> 2,217 us;
// 131,072 rays, N = 16: top-N 768 -> 741 us, inverse CDF 814 -> 734 us (128 classes)
// and 784 -> 754 us (192).  N = 1 with 192 or 256 classes is level (up to 2 % slower
// where a last round leaves two tiles on a few CUs).  With all-zero weights, which
// leave the clock at 2.4 GHz, 1,212 -> 1,073 us against 1,392 us on real ones of the
// same box: about half of what is left above the MFMAs' own time is the power
// limit, the rest epilogues that meet no MFMAs of the other workgroup.  Without the
// priorities 1.5 % slower.
//
// The MFMA steps, fragments and K order are rows_kernel.h's, so a ray's scores,
// classes and samples do not depend on which kernel renders it.
#pragma once

#include "rows_kernel.h"

namespace donerf {
namespace {

template <int NCAP, int PLACE, int DIN>
struct RowsFp8 {
    static constexpr int R = 32 * kF8CB, CB = kF8CB;
    static constexpr int NT = 64 * kF8Waves;
    static constexpr int KS_D0 = kDKPad / 16, KS_S0 = kSKPad / 16, KS_H = kHidden / 16;
    static constexpr bool CDF = PLACE != kPlaceTopN;
    static constexpr int kHalf = 16 * R;   // 16-byte units of one E4M3 buffer

    struct Shared {
        u32x4 pool[2 * kHalf];             // activations; scores of 128 classes
        float bias[2048];                  // of the network that runs
        u32x4 skip[2][NT];                 // each lane's direction skip
    };
    static_assert(sizeof(Shared) <= 80 * 1024, "two workgroups per CU");

    const RenderArgs& a;
    Shared& sh;
    int lane, wave, g, col;

    // ---- weights: a ring of registers as in rows_kernel.h, eight fragments
    // (two K steps of an E4M3 layer) ahead
    static constexpr int kHeld = 8;
    u32x4 ring[kHeld];
    // fragments I .. I + NF - 1 of a stage of F from w (stride st) are used:
    // their successors, the next stage's from wn (stride sn)
    template <int F, int I, int NF, int SLOT0>
    __device__ __forceinline__ void refill(const u32x4* w, int st, const u32x4* wn, int sn) {
        sfor<NF>([&](auto J) {
            constexpr int i = I + CV(J), n = i + kHeld;
            ring[(i + SLOT0) % kHeld] = n < F ? w[n * st * 64 + lane] : wn[(n < F ? 0 : n - F) * sn * 64 + lane];
        });
    }
    // Wave priority from MFMA step s of n: behind, under way, ahead.
    template <int S, int N>
    __device__ __forceinline__ static void priority() {
        if constexpr (S == 3 * N / 16) __builtin_amdgcn_s_setprio(1);
        if constexpr (S == 7 * N / 16) __builtin_amdgcn_s_setprio(2);
        if constexpr (S == 11 * N / 16) __builtin_amdgcn_s_setprio(3);
    }

    __device__ __forceinline__ void load_bias(f32x16 (&acc)[2][CB], int off) const {
        sfor<2>([&](auto Q) {
            const f32x16 b = bias_frag(BiasAt{sh.bias, off + 64 * wave + 32 * CV(Q)}, g);
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[CV(Q)][c] = b;
        });
    }

    // ---- epilogues of the wave's two 32-row blocks
    __device__ __forceinline__ void emit_e4m3(const f32x16 (&acc)[2][CB], u32x4* out) const {
        __builtin_amdgcn_s_setprio(0);
        sfor<2>([&](auto Q) {
            sfor<CB>([&](auto C) {
                const f32x16& x = acc[CV(Q)][CV(C)];
                u32x4 o;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_fmed3f(x[4 * w + i], 0.0f, 448.0f);
                    // the first convert's kept half is overwritten by the second
                    uint32_t p = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], __builtin_bit_cast(int, v[0]), false);
                    o[w] = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], (int)p, true);
                }
                out[(4 * wave + 2 * CV(Q) + g) * R + 32 * CV(C) + col] = o;
            });
        });
    }
    __device__ __forceinline__ void emit_bf16(const f32x16 (&acc)[2][CB], u32x4* out) const {
        sfor<2>([&](auto Q) {
            sfor<CB>([&](auto C) {
                const f32x16& x = acc[CV(Q)][CV(C)];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    u32x4 o;
#pragma unroll
                    for (int w = 0; w < 4; ++w) o[w] = relu_bf16x2(x[8 * h + 2 * w], x[8 * h + 2 * w + 1]);
                    out[(2 * (2 * (2 * wave + CV(Q)) + h) + g) * R + 32 * CV(C) + col] = o;
                }
            });
        });
    }

    // ---- layers
    // A first layer of KS bf16 steps: units 2 ks + g of buffer 0 to E4M3 in
    // buffer 1.
    template <int KS, int SLOT0>
    __device__ __forceinline__ void first_layer(const u32x4* w, const u32x4* wn, int bias) {
        f32x16 acc[2][CB];
        load_bias(acc, bias);
        u32x4 b[3];
        auto rd = [&](auto S) { b[CV(S) % 3] = sh.pool[(2 * (CV(S) / CB) + g) * R + 32 * (CV(S) % CB) + col]; };
        sfor<2>(rd);
        sfor<KS * CB>([&](auto S) {
            constexpr int s = CV(S), ks = s / CB, c = s % CB;
            priority<s, KS * CB>();
            if constexpr (s + 2 < KS * CB) rd(std::integral_constant<int, s + 2>{});
            sfor<2>([&](auto Q) {
                acc[CV(Q)][c] = Prec<kBF16>::mma(&ring[(2 * ks + CV(Q) + SLOT0) % kHeld], &b[s % 3], acc[CV(Q)][c], 127);
            });
            if constexpr (c == CB - 1) refill<2 * KS, 2 * ks, 2, SLOT0>(w, 1, wn, 1);
            __builtin_amdgcn_sched_barrier(0);
        });
        emit_e4m3(acc, sh.pool + kHalf);
    }

    // the folded positions layer: two fp32 steps of 8 K
    __device__ __forceinline__ void first_layer_pos(const u32x4 (&w)[2][2], int bias) {
        f32x16 acc[2][CB];
        load_bias(acc, bias);
        sfor<2>([&](auto K) {
            sfor<CB>([&](auto C) {
                const u32x4 b = sh.pool[(2 * CV(K) + g) * R + 32 * CV(C) + col];
                sfor<2>([&](auto Q) {
                    acc[CV(Q)][CV(C)] = Prec<kF32>::mma(&w[CV(K)][CV(Q)], &b, acc[CV(Q)][CV(C)], 127);
                });
            });
        });
        emit_e4m3(acc, sh.pool + kHalf);
    }

    // the K loop of an E4M3 layer
    __device__ __forceinline__ void hidden_steps(f32x16 (&acc)[2][CB], const u32x4* w, const u32x4* wn, int sn,
                                                 const u32x4* in, int sa) {
        u32x4 b[3][2];
        auto rd = [&](auto S) {
            constexpr int ks = CV(S) / CB, c = CV(S) % CB;
#pragma unroll
            for (int u = 0; u < 2; ++u) b[CV(S) % 3][u] = in[(4 * ks + 2 * u + g) * R + 32 * c + col];
        };
        sfor<2>(rd);
        sfor<4 * CB>([&](auto S) {
            constexpr int s = CV(S), ks = s / CB, c = s % CB;
            priority<s, 4 * CB>();
            if constexpr (s + 2 < 4 * CB) rd(std::integral_constant<int, s + 2>{});
            sfor<2>([&](auto Q) {
                acc[CV(Q)][c] = Prec<kFP8>::mma(&ring[(4 * ks + 2 * CV(Q)) % kHeld], b[s % 3], acc[CV(Q)][c], sa);
            });
            if constexpr (c == CB - 1) refill<16, 4 * ks, 4, 0>(w, 1, wn, sn);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    // The six hidden layers: input in buffer 1, output as bf16 in the whole
    // pool.  wn, sn: the stage that follows.
    __device__ __forceinline__ void hidden6(const u32x4* w, const u32x4* wn, int sn, int bias, const int32_t* ws) {
        constexpr size_t HF = (size_t)layer_chunks(kFP8, kHiddenL, 128) * kChunkFrags * 64;
        for (int l = 0; l < 5; ++l) {
            f32x16 acc[2][CB];
            load_bias(acc, bias + 256 * l);
            hidden_steps(acc, w + l * HF, w + (l + 1) * HF, 1, sh.pool + (l & 1 ? 0 : kHalf), ws[l]);
            emit_e4m3(acc, sh.pool + (l & 1 ? kHalf : 0));
            lds_barrier();
        }
        f32x16 acc[2][CB];
        load_bias(acc, bias + 256 * 5);
        hidden_steps(acc, w + 5 * HF, wn, sn, sh.pool, ws[5]);
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();   // both buffers are read
        emit_bf16(acc, sh.pool);
        lds_barrier();
    }

    // 32 classes (a row block) of the depth head for every column; FIRST: the
    // row block at wn follows (otherwise the ring ends here)
    template <bool FIRST>
    __device__ __forceinline__ void head_block(f32x16 (&acc)[CB], const u32x4* w, const u32x4* wn, int rb) {
        const f32x16 b0 = bias_frag(BiasAt{sh.bias, 7 * 256 + 32 * rb}, g);
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[c] = b0;
        sfor<KS_H>([&](auto K) {
            constexpr int ks = CV(K);
            sfor<CB>([&](auto C) {
                const u32x4 b = sh.pool[(2 * ks + g) * R + 32 * CV(C) + col];
                acc[CV(C)] = Prec<kBF16>::mma(&ring[ks % kHeld], &b, acc[CV(C)], 127);
            });
            if constexpr (FIRST || ks + kHeld < KS_H) refill<KS_H, ks, 1, 0>(w, 2, wn, 2);
            __builtin_amdgcn_sched_barrier(0x6);
        });
    }

    // ---- scores of 128 classes in the pool: unit (class / 4) of each ray
    __device__ __forceinline__ void store_scores(const f32x16 (&acc)[CB], int rbl) const {
        sfor<CB>([&](auto C) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = acc[CV(C)][4 * q + i];
                    if constexpr (CDF) v[i] = sigmoid<false>(v[i]);
                }
                sh.pool[(8 * rbl + 2 * q + g) * R + 32 * CV(C) + col] =
                    u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
            }
        });
    }
    __device__ __forceinline__ f32x4 block(int b, int ray) const {
        return __builtin_bit_cast(f32x4, sh.pool[b * R + ray]);
    }

    // ---- samples of the lane's ray.  Top-N: classes, a byte each.  Inverse CDF:
    // lanes of group 0 hold the depths, of group 1 the widths.
    static constexpr int NP = (NCAP + 3) / 4;
    int cls[NP];
    float td[CDF ? NCAP : 1];

    // Inverse CDF, the arithmetic of rows_kernel.h's place_cdf.  The targets of
    // a lane (group 0: slice centres, group 1: inner slice ends) ascend, so its
    // block and the prefix before it only move forward.  One call resolves the
    // targets whose block is among the nh blocks from b0 on in the pool, or that
    // lie past the last block (last).
    struct Walk {
        int b;        // current block
        float pre;    // sum of the blocks before it
        int done;     // targets resolved
    };
    __device__ __forceinline__ void walk_half(Walk& k, int b0, int nh, bool last, float total, int ray) {
        const bool wide = PLACE == kPlaceCdfWide;
        const int NB = wide ? 64 : 32;
#pragma unroll
        for (int t = 0; t < NCAP; ++t) {
            const float m = (g ? a.cdf_u[kMaxSamples + t] : a.cdf_u[t]) * total;
            if (t >= k.done && t < a.N - g) {
                f32x4 w = {0.0f, 0.0f, 0.0f, 0.0f};
                bool at = false;
                while (k.b < b0 + nh) {
                    w = block(k.b - b0, ray);
                    const float nxt = k.pre + (((w[0] + w[1]) + w[2]) + w[3]);
                    at = !(nxt <= m) || k.b == NB - 1;
                    if (at) break;
                    k.pre = nxt;
                    ++k.b;
                }
                float s = 0.0f;
                int c = 0;
                if (at || (last && !wide)) {
                    if (!at) w = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    const int b = at ? k.b : NB - 1;
                    const float lo = k.pre;
                    const float r = wide ? m - lo : m, z = wide ? 0.0f : lo;
                    const float c1 = wide ? w[0] : lo + w[0], c2 = c1 + w[1], c3 = c2 + w[2];
                    const int j = (r >= c1 ? 1 : 0) + (r >= c2 ? 1 : 0) + (r >= c3 ? 1 : 0);
                    const float base = j == 0 ? z : j == 1 ? c1 : j == 2 ? c2 : c3;
                    const float aj = j == 0 ? w[0] : j == 1 ? w[1] : j == 2 ? w[2] : w[3];
                    const float q = wide ? (r - base) * __builtin_amdgcn_rcpf(aj) : (r - base) / aj;
                    const float frac = aj > 0.0f ? fminf(fmaxf(q, 0.0f), 1.0f) : 0.0f;
                    c = 4 * b + j;
                    s = wide ? ((float)c + frac) * (1.0f / (float)a.B) : ((float)c + frac) / (float)a.B;
                } else if (last) {
                    c = 4 * (NB - 1);
                    s = m - k.pre;
                }
                if (at || last) {
                    td[t] = a.near + exp2f(s * a.log2_span1) - 1.0f;   // inverse of Eq. 3
                    cls[t / 4] |= c << (8 * (t % 4));
                    k.done = t + 1;
                }
            }
        }
    }

    // The lane's indices, through an asm the compiler cannot see through: LDS
    // addresses made from them are made again in each phase, and in each stage of
    // a sample, instead of being held in registers (and spilled) across the tile.
    // Without that in the samples, the ray made again, the dumps before them and
    // weight pointers to global memory (opaque), inverse CDF spilled 24 to 76
    // registers and every wait in the layers was a wait for all loads: 131,072
    // rays, N = 16, inverse CDF, 192 classes 804 -> 754 us; top-N, 128 classes
    // 763 -> 741 us; 5 x 400 x 400, N = 4 1,379 -> 1,347 us.
    __device__ __forceinline__ void set_lane(int l) {
        asm volatile("" : "+v"(l));
        lane = l;
        g = l >> 5;
        col = l & 31;
    }

    __device__ __forceinline__ void run() {
        const int tid = threadIdx.x;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        set_lane(tid & 63);
        constexpr int KIND0 = DIN == kDinEncoded ? kDFirst : kDFirstPos;
        constexpr size_t D0F = rows_layer_frags(kFP8, KIND0, 128) * 64, HF = rows_layer_frags(kFP8, kHiddenL, 128) * 64,
                         S0F = rows_layer_frags(kFP8, kSFirst, 128) * 64;
        // the wave's first fragment of every stage: passes of two row blocks
        const u32x4* ds = reinterpret_cast<const u32x4*>(a.d_frags);
        const u32x4* ss = reinterpret_cast<const u32x4*>(a.s_frags);
        const u32x4* d0 = ds + wave * 2 * KS_D0 * 64;
        const u32x4* dh = ds + D0F + wave * 16 * 64;
        const u32x4* dhead = ds + D0F + 6 * HF;
        const u32x4* s0 = ss + wave * 2 * KS_S0 * 64;
        const u32x4* shd = ss + S0F + wave * 16 * 64;
        const u32x4* shead = ss + S0F + 6 * HF;

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

        constexpr int D0SLOT = 4;   // the 12 fragments of the encoded first layer end at slot 0
        u32x4 pos_w[2][2];
        if constexpr (DIN == kDinEncoded) {
            sfor<kHeld>([&](auto I) { ring[(CV(I) + D0SLOT) % kHeld] = d0[CV(I) * 64 + lane]; });
        } else {
            sfor<2>([&](auto K) {
                sfor<2>([&](auto Q) { pos_w[CV(K)][CV(Q)] = ds[((wave * 2 + CV(K)) * 2 + CV(Q)) * 64 + lane]; });
            });
            sfor<kHeld>([&](auto I) { ring[CV(I)] = dh[CV(I) * 64 + lane]; });
        }
        // biases of the depth network: seven layers, then the head
        for (int k = tid; k < 7 * 256 + a.B; k += NT) sh.bias[k] = a.bias[k < 7 * 256 ? k : kDepthHeadBias + k - 7 * 256];

        // ---- the lane's ray, the depth-network input, the direction skip
        auto rl = [&]() { return 32 * wave + col; };    // ray within the tile
        auto rid = [&]() { return ray0 + (uint32_t)rl(); };
        auto lane_ray = [&]() { return camera_ray(a, rid() < a.total_rays ? rid() : a.total_rays - 1); };
        {
            const Ray ray = lane_ray();
            float ou[3], v[3];
            unify(a, ray, ou);
            v[0] = (ou[0] - a.cx) / a.dmax;
            v[1] = (ou[1] - a.cy) / a.dmax;
            v[2] = (ou[2] - a.cz) / a.dmax;
            float f[kDSlots];
            if constexpr (DIN == kDinEncoded) {
                fourier<5>(v, g, f);
                fourier<2>(ray.r, g, f + 30);
                f[42] = g ? ray.r[0] : v[0];
                f[43] = g ? ray.r[1] : v[1];
                f[44] = g ? ray.r[2] : v[2];
                f[45] = f[46] = f[47] = 0.0f;
#pragma unroll
                for (int ks = 0; ks < KS_D0; ++ks) sh.pool[(2 * ks + g) * R + rl()] = Prec<kBF16>::pack(f + 8 * ks);
            } else {
                // unit (ks, g) holds K 8 ks + 2 e + g of [u', r, u_c]
                const float uc[3] = {(ray.o[0] - a.cx) / a.dmax, (ray.o[1] - a.cy) / a.dmax, (ray.o[2] - a.cz) / a.dmax};
                const float q[8] = {g ? v[1] : v[0],         g ? ray.r[0] : v[2], g ? ray.r[2] : ray.r[1],
                                    g ? uc[1] : uc[0],       g ? 0.0f : uc[2],    0.0f, 0.0f, 0.0f};
                sh.pool[g * R + rl()] = Prec<kF32>::pack(q);
                sh.pool[(2 + g) * R + rl()] = Prec<kF32>::pack(q + 4);
                fourier<2>(ray.r, g, f + 30);
            }
            float fs[kSkipSlots];
#pragma unroll
            for (int k = 0; k < 12; ++k) fs[k] = f[30 + k];
            fs[12] = g ? 0.0f : ray.r[0];
            fs[13] = g ? 0.0f : ray.r[1];
            fs[14] = g ? 0.0f : ray.r[2];
            fs[15] = 0.0f;
            sh.skip[0][64 * wave + lane] = Prec<kBF16>::pack(fs);
            sh.skip[1][64 * wave + lane] = Prec<kBF16>::pack(fs + 8);
        }
        lds_barrier();

        // ---- depth network
        const int nrb = a.B / 32;
        const bool two = nrb > 4;                       // row blocks wave and 4 + wave
        const int rb0 = wave < nrb ? wave : 0, rb1 = 4 + wave < nrb ? 4 + wave : 0;
        const u32x4* h0 = dhead + ((rb0 >> 1) * KS_H * 2 + (rb0 & 1)) * 64;
        const u32x4* h1 = dhead + ((rb1 >> 1) * KS_H * 2 + (rb1 & 1)) * 64;
        if constexpr (DIN == kDinEncoded) first_layer<KS_D0, D0SLOT>(d0, dh, 0);
        else first_layer_pos(pos_w, 0);
        lds_barrier();
        hidden6(dh, h0, 2, 256, a.wscale + 1);

        // ---- depth head and placement: 128 classes at a time in the pool
        set_lane(lane);
        {
            f32x16 acc0[CB], acc1[CB];
            const bool act0 = wave < nrb, act1 = 4 + wave < nrb;
            if (act0) head_block<true>(acc0, h0, h1, rb0);
            if (act1) head_block<false>(acc1, h1, h1, rb1);
            if (a.out_scores && part == 0)
                for (int h = 0; h < (two ? 2 : 1); ++h)
                    if (h ? act1 : act0)
                        sfor<CB>([&](auto C) {
                            const uint32_t r = ray0 + 32 * CV(C) + col;
                            if (r < a.total_rays) {
                                float* dst = a.out_scores + (size_t)r * a.B + 32 * (h ? rb1 : rb0) + 4 * g;
#pragma unroll
                                for (int i = 0; i < 16; ++i)
                                    dst[8 * (i / 4) + (i % 4)] = h ? acc1[CV(C)][i] : acc0[CV(C)][i];
                            }
                        });
            // each half of the classes in turn: stored, then used by f(first
            // block, blocks)
            auto halves = [&](auto f) {
                lds_barrier();
                if (act0) store_scores(acc0, wave);
                lds_barrier();
                f(0, min(a.B, 128) / 4);
                if (two) {
                    lds_barrier();
                    if (act1) store_scores(acc1, wave);
                    lds_barrier();
                    f(32, (a.B - 128) / 4);
                }
            };
#pragma unroll
            for (int i = 0; i < NP; ++i) cls[i] = 0;
            if constexpr (!CDF) {
                TopList<NCAP> top;
                top.init();
                halves([&](int b0, int nh) {
                    for (int b = 0; b < nh; b += 2) {
                        const f32x4 v = block(b + g, rl());
#pragma unroll
                        for (int j = 0; j < 4; ++j) top.push(v[j], 4 * (b0 + b) + j);   // + 4 g: rebase
                    }
                });
                top.rebase(4 * g);
                top.merge_partner();
                int sel[NCAP];
                top.ascending(a.N, sel);
#pragma unroll
                for (int k = 0; k < NCAP; ++k) cls[k / 4] |= (min(sel[k], a.B - 1) & 255) << (8 * (k % 4));
            } else {
                float total = 0.0f;
                halves([&](int, int nh) {
                    for (int b = 0; b < nh; ++b) {
                        const f32x4 v = block(b, rl());
                        total = total + (((v[0] + v[1]) + v[2]) + v[3]);
                    }
                });
                Walk k{0, 0.0f, 0};
#pragma unroll
                for (int t = 0; t < NCAP; ++t) td[t] = 0.0f;
                const int nb = a.B / 4;
                halves([&](int b0, int nh) { walk_half(k, b0, nh, b0 + nh == nb, total, rl()); });
                // group 1: slice ends become widths
                if (g) {
                    float edge = a.near;
#pragma unroll
                    for (int i = 0; i < NCAP; ++i) {
                        const float end = i + 1 < a.N ? td[i] : a.dmax;
                        td[i] = end - edge;
                        edge = end;
                    }
                }
            }
        }
        // sample k: class, depth, width
        auto sample = [&](int k, int& c, float& t, float& d) {
            c = (pick<true>(cls, k >> 2) >> (8 * (k & 3))) & 255;
            if constexpr (!CDF) {
                t = a.bins[c];
                d = a.bins[a.B + c];
            } else {
                float own = td[0];
#pragma unroll
                for (int q = 1; q < NCAP; ++q) {
                    float v = td[q];
                    asm("" : "+v"(v));   // a select chain, not a load at a computed index
                    own = k == q ? v : own;
                }
                const float other = __shfl_xor(own, 32);
                t = g ? other : own;
                d = g ? own : other;
            }
        };

        if (part == 0 && (a.out_bins || a.out_samples))
            for (int k = 0; k < a.N; ++k) {
                int c;
                float t, d;
                sample(k, c, t, d);
                if (g == 0 && rid() < a.total_rays) {
                    const size_t at = (size_t)rid() * a.N + k;
                    if (a.out_bins) a.out_bins[at] = c;
                    if (a.out_samples) {
                        a.out_samples[2 * at] = t;
                        a.out_samples[2 * at + 1] = d;
                    }
                }
            }

        // ---- shading network per sample
        set_lane(lane);
        lds_barrier();   // the depth network's biases and the scores are read
        for (int k = 64 * wave + lane; k < 7 * 256 + 32; k += NT) sh.bias[k] = a.bias[7 * 256 + k];
        sfor<kHeld>([&](auto I) { ring[CV(I)] = s0[CV(I) * 64 + lane]; });
        const Ray ray = lane_ray();   // made again: not held (and spilled) across the depth network
        float T = 1.0f, Cr = 0.0f, Cg = 0.0f, Cb = 0.0f, Dp = 0.0f;
        for (int k = k_begin; k < k_end; ++k) {
            // keeps the samples' equal weight loads inside the loop
            const u32x4 *s0k = opaque(s0), *shk = opaque(shd), *hk = opaque(shead);
            set_lane(lane);
            int c;
            float tk, dk;
            sample(k, c, tk, dk);
            {
                float x[3], w[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) x[i] = ray.o[i] + tk * ray.r[i];
                warp(a, x, w);
                float f[kSSlots];
                fourier<5>(w, g, f);
                f[30] = g ? w[2] : w[0];
                f[31] = g ? 0.0f : w[1];
#pragma unroll
                for (int ks = 0; ks < KS_S0; ++ks) sh.pool[(2 * ks + g) * R + rl()] = Prec<kBF16>::pack(f + 8 * ks);
            }
            lds_barrier();
            set_lane(lane);
            first_layer<KS_S0, 0>(s0k, shk, 0);
            lds_barrier();
            set_lane(lane);
            hidden6(shk, s0k, 1, 256, a.wscale + 9);
            set_lane(lane);
            // head: the wave's own 32 columns, one row block
            f32x16 acc = bias_frag(BiasAt{sh.bias, 7 * 256}, g);
            u32x4 hw[KS_H + 2];
            sfor<6>([&](auto K) { hw[CV(K)] = hk[CV(K) * 64 + lane]; });
            sfor<KS_H + 2>([&](auto K) {
                constexpr int ks = CV(K);
                if constexpr (ks + 6 < KS_H + 2) hw[ks + 6] = hk[(ks + 6) * 64 + lane];
                u32x4 b;
                if constexpr (ks < KS_H) b = sh.pool[(2 * ks + g) * R + rl()];
                else b = sh.skip[ks - KS_H][64 * wave + lane];
                acc = Prec<kBF16>::mma(&hw[ks], &b, acc, 127);
                __builtin_amdgcn_sched_barrier(0x6);
            });
            lds_barrier();   // the activations are read: the next sample's input takes their place
            // compositing: lanes of group 0 hold (r, g, b, sigma)
            const float cr = sigmoid<false>(acc[0]), cg = sigmoid<false>(acc[1]), cbl = sigmoid<false>(acc[2]);
            const float tau = fmaxf(acc[3], 0.0f) * dk;
            const float wgt = T * one_minus_exp_neg<false>(tau);
            Cr += wgt * cr;
            Cg += wgt * cg;
            Cb += wgt * cbl;
            Dp += wgt * tk;
            T *= exp_neg<false>(tau);
        }

        // ---- outputs
        set_lane(lane);
        const uint32_t ro = rid();
        const bool valid = ro < a.total_rays;
        if (g == 0 && valid) {
            if (nsplit > 1) {
                float* q = a.partial + ((size_t)(tile_local * R + rl()) * nsplit + part) * 5;
                q[0] = Cr;
                q[1] = Cg;
                q[2] = Cb;
                q[3] = Dp;
                q[4] = T;
            } else {
                float* o = a.out_rgb + (size_t)ro * 3;
                o[0] = Cr;
                o[1] = Cg;
                o[2] = Cb;
                if (a.out_depth) a.out_depth[ro] = Dp;
            }
        }
    }
};

// The main kernel of fp8 networks.
template <int NCAP, int PLACE, int DIN>
__global__ void __launch_bounds__(64 * kF8Waves) __attribute__((amdgpu_waves_per_eu(2, 2)))
fp8_render_kernel(const RenderArgs a) {
    using K = RowsFp8<NCAP, PLACE, DIN>;
    __shared__ typename K::Shared sh;
    K k{a, sh};
    k.run();
}

template <int PL, int DIN>
hipError_t launch_fp8_variant(int ncap, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    const dim3 block(64 * kF8Waves);
    if (ncap == 4) hipLaunchKernelGGL((fp8_render_kernel<4, PL, DIN>), grid, block, 0, stream, a);
    else if (ncap == 8) hipLaunchKernelGGL((fp8_render_kernel<8, PL, DIN>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((fp8_render_kernel<16, PL, DIN>), grid, block, 0, stream, a);
    return hipGetLastError();
}

template <int PL>
hipError_t launch_fp8(int ncap, int din, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    return din == kDinPositions ? launch_fp8_variant<PL, kDinPositions>(ncap, a, grid, stream)
                                : launch_fp8_variant<PL, kDinEncoded>(ncap, a, grid, stream);
}

}  // namespace
}  // namespace donerf
