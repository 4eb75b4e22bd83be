// Kernels of the pre-norm Transolver block around the Physics-Attention layer
// (the model context of section 3; 8 blocks in the paper's Table 7):
//
//   y   = x + PA(LN1(x))
//   out = y + W_b^T GELU(W_a^T LN2(y) + b_a) + b_b
//
// bf16 activations [N][C] between kernels, float32 arithmetic inside, bf16
// matrix-core operands with float32 accumulation.
//
//   k_layernorm     LN1 of the first block (later blocks get theirs from the
//                   previous block's feed-forward epilogue).
//   k_prep_mlp      W_a (bf16) and W_b (f16) as matrix-core fragments, chunked
//                   by FC hidden units: [F/FC][W_a^T part | W_b part], FC*C
//                   elements each, so one linear copy stages a chunk.
//   k_mlp_residual_pc  one kernel for the rest of the block: y = x + PA
//                   output, LN2, both feed-forward products with GELU (its
//                   tanh form in half precision, gelu2_f16) between them, the
//                   residual, and optionally the next block's LN1.
//
// k_mlp_residual_pc: 32 PT (128, or fewer for a small call) points per workgroup.  A
// producer keeps LN2(y) of its group's points as B fragments (K = channels) in
// registers; the hidden layer is walked in chunks staged in LDS:
//   GEMM1  H^T[f][p] = W_a^T[f][:] . LN2(y)[p][:] + b_a[f]   (A = staged W_a^T)
//   GELU   on packed halves; the 16 x 4 outputs of two hidden tiles are
//          exactly a B fragment of the second product (K slot (g, t) <->
//          hidden unit 32km + 16(t>>2) + 4g + (t&3)), handed to the consumer
//          through LDS in that fragment order;
//   GEMM2  out^T[c][p] += W_b^T[c][:] . h[p][:]   (consumer; A = staged W_b,
//          f16 x f16) into the accumulator of 16 PT points x C/2 channels.
// Output rows of W_b's fragments follow zchan(), so a lane ends up holding the
// eight consecutive channels 32k + 8g .. +7 of its point: the same channels
// it loads for the residual, which keeps the next LayerNorm in registers.
#pragma once
#include "ts3_device.h"
#include "ts3_pass2.h"  // zchan

namespace ts3 {

constexpr float BLOCK_LN_EPS = 1e-5f;

// GELU(x) = x Phi(x) of two values, evaluated on packed halves with the
// tanh form of Hendrycks and Gimpel: Phi(x) ~ (1 + tanh(sqrt(2/pi) (x +
// 0.044715 x^3))) / 2 = 1 / (1 + exp(-2 sqrt(2/pi) (x + 0.044715 x^3))), so
// GELU(x) ~ x / (1 + 2^u) with u = -x (K1 + K2 x^2), K1 = 2 sqrt(2/pi) / ln 2,
// K2 = 0.044715 K1: four packed operations, two exp2 and two reciprocals per
// pair.  The form differs from x Phi(x) by at most 4.7e-4 (absolute); in half
// precision (every operation rounded to f16) the RMS absolute error over
// N(0, 1.5^2) inputs is 4.7e-4 and the worst 3.8e-3 (the f16 rounding of x near
// 8).  The tails need no care: for very negative x, 2^u overflows to infinity
// and the reciprocal gives 0; for large x, 2^u underflows and GELU(x) = x.
// Returns the pair as the f16 B-operand slots of the second product.
__device__ __forceinline__ f16x2 gelu2_f16(float a, float b) {
    const f16x2 x{(_Float16)a, (_Float16)b};
    const f16x2 u = x * ((x * x) * (_Float16)-0.10294280f + (_Float16)-2.30220819f);
    const f16x2 d = __builtin_elementwise_exp2(u) + (_Float16)1.0f;
    f16x2 r;
    r[0] = __builtin_amdgcn_rcph(d[0]);
    r[1] = __builtin_amdgcn_rcph(d[1]);
    return x * r;
}

__device__ __forceinline__ void unpack8(const uint4 &u, float (&v)[8]) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ uint4 pack8(const float (&v)[8]) {
    typedef __attribute__((ext_vector_type(8))) __bf16 b8;
    b8 b;
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = (__bf16)v[i];
    return __builtin_bit_cast(uint4, b);
}

// LayerNorm over C channels of bf16 rows; C/8 lanes per row, 8 channels each.
template <int C>
__global__ __launch_bounds__(256) void k_layernorm(const bf16_t *__restrict__ x, int64_t n,
                                                   const float *__restrict__ gam, const float *__restrict__ bet,
                                                   bf16_t *__restrict__ out) {
    constexpr int LPR = C / 8, RPW = 64 / LPR;
    const int lane = threadIdx.x & 63, sub = lane / LPR, cl = lane % LPR;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    float gv[8], bv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        gv[i] = gam[8 * cl + i];
        bv[i] = bet[8 * cl + i];
    }
    for (int64_t r0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * RPW; r0 < n;
         r0 += waves * RPW) {
        const int64_t row = r0 + sub;
        const int64_t rc = row < n ? row : n - 1;
        float v[8];
        unpack8(*reinterpret_cast<const uint4 *>(x + rc * C + 8 * cl), v);
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) s += v[i];
#pragma unroll
        for (int m = 1; m < LPR; m <<= 1) s += __shfl_xor(s, m);
        const float mean = s * (1.f / C);
        float q = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[i] -= mean;
            q += v[i] * v[i];
        }
#pragma unroll
        for (int m = 1; m < LPR; m <<= 1) q += __shfl_xor(q, m);
        const float rstd = 1.f / sqrtf(q * (1.f / C) + BLOCK_LN_EPS);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = v[i] * rstd * gv[i] + bv[i];
        if (row < n) *reinterpret_cast<uint4 *>(out + row * C + 8 * cl) = pack8(v);
    }
}

// Hidden units per chunk.  At C = 128 a chunk of 32 leaves room for a second workgroup
// per compute unit (68 KB of LDS, 122 registers): its products run while the other
// loads or writes its rows, which take as long as the products there.
template <int C> struct MlpCfg {
    static constexpr int FC = C <= 128 ? 32 : 64, KM = FC / 32, CK = C / 32;
    static constexpr int PART = FC * C;                 // elements of each half of a chunk
};

// Fragments of chunk j (hidden units FC j .. FC j + FC - 1):
//   W_a^T part, index ((ht*CK + kc)*64 + l)*8 + t:
//       W_a[c = 32kc + 8(l>>4) + t][f = FC j + 16ht + (l&15)]
//   W_b part,   index ((ct*KM + km)*64 + l)*8 + t:
//       W_b[f = FC j + 32km + 16(t>>2) + 4(l>>4) + (t&3)][c = zchan(ct, l&15)]
template <int C>
__global__ void k_prep_mlp(const float *__restrict__ Wa, const float *__restrict__ Wb, int F,
                           bf16_t *__restrict__ frag) {
    using Cfg = MlpCfg<C>;
    const int64_t total = (int64_t)(F / Cfg::FC) * 2 * Cfg::PART;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t j = i / (2 * Cfg::PART);
        const int e = (int)(i % (2 * Cfg::PART));
        const int t = e & 7, l = (e >> 3) & 63, r = e >> 9;
        float v;
        if (e < Cfg::PART) {
            const int kc = r % Cfg::CK, ht = r / Cfg::CK;
            const int c = 32 * kc + 8 * (l >> 4) + t;
            const int64_t f = Cfg::FC * j + 16 * ht + (l & 15);
            v = Wa[(int64_t)c * F + f];
        } else {
            const int r2 = r - Cfg::PART / 512;
            const int km = r2 % Cfg::KM, ct = r2 / Cfg::KM;
            const int64_t f = Cfg::FC * j + 32 * km + 16 * (t >> 2) + 4 * (l >> 4) + (t & 3);
            const int c = zchan(ct, l & 15);
            frag[i].bits = __builtin_bit_cast(uint16_t, (_Float16)Wb[f * C + c]);  // f16: the second product
            continue;
        }
        frag[i].bits = __builtin_bit_cast(uint16_t, (__bf16)v);
    }
}

// x, pa  : [n][C] bf16, the block input and its Physics-Attention output
// ln2_*  : LN2 affine [C]; frag: k_prep_mlp output; ba [F], bb [C]
// lnn_*  : the next block's LN1 affine, or NULL (then xn is not written)
// xo     : [n][C] bf16 block output (may alias x: a wave reads and writes the
//          same rows); xn: LN1
//          of xo for the next block (may alias nothing that is read here)
// grid   : ceil(n / (32 PT)) workgroups of 512 threads
//
// Producer and consumer waves, two per SIMD (one of each): groups of 64 points, two
// producers and two consumers each, 128 points per workgroup.
//   each wave   first makes LN2(y) of 16 of the block's points, as B fragments, through
//               LDS, and at the end writes 16 points' output and next LN1 from the sums
//               that the consumers leave there;
//   wave q      (producer, group q >> 1, half q & 1) keeps the group's 64
//               points' fragments and, per chunk j of hidden units (64, or 32 at C =
//               128), runs GEMM1 and the GELU for its half of them, which is one K
//               step of GEMM2 or half of one: it writes that h (f16 B fragments, in
//               fragment order) to the group's h tile;
//   wave q + 4  (consumer) runs GEMM2 of chunk j-1 from that h tile for its half of
//               the channels into a 64 x C/2 output accumulator and issues a quarter
//               of the weight copies.
// Every weight fragment read from LDS feeds four MFMAs (four 16-point tiles).  With
// pairs of waves on 32 points (two MFMAs per fragment) the LDS reads alone took longer
// than the products: 272 KB per chunk, 2,100 cycles at 128 bytes, against 2,048 cycles
// of MFMAs per SIMD; now 160 KB.  The GELU's vector work runs beside the other wave's
// matrix work.  W_a^T and W_b halves of a chunk are staged in separate slots (two
// each): step j reads W_a(j) and W_b(j-1) and copies W_a(j+1) and W_b(j).  One barrier
// per step; NCHUNK + 1 steps.  LDS: 4 x 64C bf16 weight slots + 2 x 8 KB h tiles per
// group (160 KB at C = 256).
//
// PT: 16-point tiles per group (the workgroup takes 32 PT points; the figures above are
// for 4).  A workgroup's steps are one chain, so a call of a few thousand points is
// bound by the points per workgroup: 4,096 points at C = 256 ran 32 workgroups and took
// 44 us, with PT = 1 128 workgroups and 24 us.  mlp_tiles() has the rule.  A point's products and their order do
// not depend on PT, nor does its result.
template <int C, int PT> struct MlpPCCfg {
    static constexpr int FC = MlpCfg<C>::FC, KM = FC / 32, CK = C / 32, CT = C / 16, PTS = 32 * PT;
    static constexpr int HT = FC / 32;                   // a producer's hidden tiles
    static constexpr int CTH = CT / 2;                   // a consumer's channel tiles
    static constexpr int ZLD = C + 4;                    // floats per row of output sums (bank spread)
    static constexpr int PART = FC * C;                 // elements of each half of a chunk
    static constexpr int PART_BYTES = PART * 2;
    static constexpr int PART_COPIES = PART_BYTES / 1024;
    static constexpr int HTILE = PT * KM * 64 * 16;      // bytes: a group's h fragments
    static constexpr int YB = PART_BYTES;                // LN2(y) fragments on their way: past W_a's first slot
    static constexpr int PIPE = 4 * PART_BYTES + 2 * 2 * HTILE, ROWS = PTS * ZLD * 4;
    static constexpr int LDS_BYTES = PIPE > ROWS ? PIPE : ROWS;
    static_assert(YB + 2 * PT * CK * 1024 <= LDS_BYTES, "rows pass through the slots");
    static_assert(PART_COPIES % 4 == 0, "each consumer issues a quarter of a part's copies");
    static_assert(HT == 1 || HT == 2, "a producer's hidden units are half a K step or one");
};

template <int C, int F, int PT>
__global__ __launch_bounds__(512, C <= 128 ? 4 : 1) void k_mlp_residual_pc(
    const bf16_t *x, const bf16_t *__restrict__ pa, int64_t n, const float *__restrict__ ln2_g,
    const float *__restrict__ ln2_b, const bf16_t *__restrict__ frag, const float *__restrict__ ba,
    const float *__restrict__ bb, const float *__restrict__ lnn_g, const float *__restrict__ lnn_b, bf16_t *xo,
    bf16_t *__restrict__ xn) {
    using Cfg = MlpPCCfg<C, PT>;
    constexpr int CK = Cfg::CK, CTH = Cfg::CTH, KM = Cfg::KM, HT = Cfg::HT;
    constexpr int NCHUNK = F / Cfg::FC, PB = Cfg::PART_BYTES, HTILE = Cfg::HTILE;
    static_assert(F % Cfg::FC == 0, "hidden width in whole chunks");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[Cfg::LDS_BYTES];
    unsigned char *const wa_slots = lds;               // W_a^T parts, two slots
    unsigned char *const wb_slots = lds + 2 * PB;      // W_b parts, two slots

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int q = wave & 3, role = wave >> 2;
    const int grp = q >> 1, half = q & 1;
    const int li = lane & 15, g = lane >> 4;
    unsigned char *const hslots = lds + 4 * PB + grp * 2 * HTILE;  // the group's two h tiles

    // A consumer's quarter of part `half` (0: W_a^T, 1: W_b) of chunk j into slot sl.
    auto issue_part = [&](int j, int part, int sl) {
        const unsigned char *src = reinterpret_cast<const unsigned char *>(frag) + ((size_t)(2 * j + part)) * PB;
        const uint32_t base = lds_addr(lds) + (part * 2 + sl) * PB;
#pragma unroll
        for (int c = 0; c < Cfg::PART_COPIES / 4; ++c) {
            const int k = q * (Cfg::PART_COPIES / 4) + c;
            dma16(src + k * 1024 + lane * 16, base + k * 1024);
        }
    };

    // Wave w < 2 PT takes points 16w .. of the block, whole rows, before and after the chunks
    // (one memory round trip each way, no row read twice): lane (li, g) holds channels
    // 32k + 8g .. +7 of point row(w) = blk + 16w + li.
    const bool rows = wave < 2 * PT;
    const int64_t pr = (int64_t)blockIdx.x * Cfg::PTS + wave * 16 + li;
    const int64_t prc = pr < n ? pr : n - 1;
    auto load_row = [&](uint4 (&xv)[CK], uint4 (&pv)[CK]) {
#pragma unroll
        for (int k = 0; k < CK; ++k) {
            xv[k] = *reinterpret_cast<const uint4 *>(x + prc * C + 32 * k + 8 * g);
            pv[k] = *reinterpret_cast<const uint4 *>(pa + prc * C + 32 * k + 8 * g);
        }
    };
    // Normalises v over the row (statistics over its four lanes).
    auto normalise = [&](float (&v)[CK][8], const float *gam, const float *bet) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < CK; ++k)
#pragma unroll
            for (int t = 0; t < 8; ++t) s += v[k][t];
        const float mean = xrow_sum(s) * (1.f / C);
        float qq = 0.f;
#pragma unroll
        for (int k = 0; k < CK; ++k)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                v[k][t] -= mean;
                qq += v[k][t] * v[k][t];
            }
        const float rstd = 1.f / sqrtf(xrow_sum(qq) * (1.f / C) + BLOCK_LN_EPS);
#pragma unroll
        for (int k = 0; k < CK; ++k) {
            const f32x4 g0 = *reinterpret_cast<const f32x4 *>(gam + 32 * k + 8 * g);
            const f32x4 g1 = *reinterpret_cast<const f32x4 *>(gam + 32 * k + 8 * g + 4);
            const f32x4 b0 = *reinterpret_cast<const f32x4 *>(bet + 32 * k + 8 * g);
            const f32x4 b1 = *reinterpret_cast<const f32x4 *>(bet + 32 * k + 8 * g + 4);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                v[k][t] = v[k][t] * rstd * g0[t] + b0[t];
                v[k][t + 4] = v[k][t + 4] * rstd * g1[t] + b1[t];
            }
        }
    };
    if (role == 1) issue_part(0, 0, 0);
    if (rows) {  // LN2(x + pa) as B fragments of tile `wave`, through LDS
        uint4 xv[CK], pv[CK];
        load_row(xv, pv);
        float y[CK][8];
#pragma unroll
        for (int k = 0; k < CK; ++k) {
            float a[8], b[8];
            unpack8(xv[k], a);
            unpack8(pv[k], b);
#pragma unroll
            for (int t = 0; t < 8; ++t) y[k][t] = a[t] + b[t];
        }
        normalise(y, ln2_g, ln2_b);
#pragma unroll
        for (int k = 0; k < CK; ++k)
            *reinterpret_cast<uint4 *>(lds + Cfg::YB + ((wave * CK + k) * 64 + lane) * 16) = pack8(y[k]);
    }
    wait_vmcnt<0>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();  // every tile's fragments and W_a(0) are in LDS
    float *const zrows = reinterpret_cast<float *>(lds);  // after the chunks: [PTS][ZLD] output sums
    constexpr int ZLD = Cfg::ZLD;

    if (role == 0) {
        // ---------------------------------------------------------------- producer
        Frag<bf16_t> yb[PT][CK];
#pragma unroll
        for (int pt = 0; pt < PT; ++pt)
#pragma unroll
            for (int k = 0; k < CK; ++k)
                yb[pt][k].v =
                    *reinterpret_cast<const bf16x8 *>(lds + Cfg::YB + (((grp * PT + pt) * CK + k) * 64 + lane) * 16);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();  // the fragments are in registers, the slots free
#pragma unroll 1
        for (int j = 0; j <= NCHUNK; ++j) {
            if (j < NCHUNK) {
                const unsigned char *wa = wa_slots + (j & 1) * PB;
                f32x4 Hh[HT][PT];
#pragma unroll
                for (int i = 0; i < HT; ++i) {
                    const float4 b = *reinterpret_cast<const float4 *>(ba + Cfg::FC * j + 16 * (HT * half + i) + 4 * g);
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt) Hh[i][pt] = f32x4{b.x, b.y, b.z, b.w};
                }
                // A fragments are read one K step ahead of their products.
                Frag<bf16_t> a1[2][HT];
                auto read1 = [&](int kc, Frag<bf16_t>(&dst)[HT]) {
#pragma unroll
                    for (int i = 0; i < HT; ++i)
                        dst[i].v = *reinterpret_cast<const bf16x8 *>(wa + (((HT * half + i) * CK + kc) * 64 + lane) * 16);
                };
                read1(0, a1[0]);
                __builtin_amdgcn_s_setprio(2);  // GEMM1 first on the matrix core; GEMM2 fills the GELU
#pragma unroll
                for (int kc = 0; kc < CK; ++kc) {
                    if (kc + 1 < CK) read1(kc + 1, a1[(kc + 1) & 1]);
#pragma unroll
                    for (int i = 0; i < HT; ++i)
#pragma unroll
                        for (int pt = 0; pt < PT; ++pt) mma(Hh[i][pt], a1[kc & 1][i], yb[pt][kc]);
                }
                __builtin_amdgcn_s_setprio(0);
                // GELU into the f16 B fragments of GEMM2: K step `half`, or slots 4 half .. +3
                // of the only one.
                unsigned char *ht_out = hslots + (j & 1) * HTILE + (HT == 2 ? half * PT * 1024 : half * 8);
#pragma unroll
                for (int pt = 0; pt < PT; ++pt) {
                    typedef __attribute__((ext_vector_type(2 * HT))) uint32_t uh_t;
                    uh_t u;
#pragma unroll
                    for (int t = 0; t < 4 * HT; t += 2)
                        u[t >> 1] = __builtin_bit_cast(uint32_t, gelu2_f16(Hh[t >> 2][pt][t & 3], Hh[t >> 2][pt][(t & 3) + 1]));
                    *reinterpret_cast<uh_t *>(ht_out + (pt * 64 + lane) * 16) = u;
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __syncthreads();  // h(j) written; W_a(j+1) and W_b(j) staged
        }
    } else {
        // ---------------------------------------------------------------- consumer
        f32x4 Z[CTH][PT];  // channel tiles CTH * half + ct
#pragma unroll
        for (int ct = 0; ct < CTH; ++ct)
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) Z[ct][pt] = f32x4{0.f, 0.f, 0.f, 0.f};
        __syncthreads();  // the fragments are in registers, the slots free
#pragma unroll 1
        for (int j = 0; j <= NCHUNK; ++j) {
            if (j + 1 < NCHUNK) issue_part(j + 1, 0, (j + 1) & 1);
            if (j < NCHUNK) issue_part(j, 1, j & 1);
            if (j > 0) {
                // GEMM2 of chunk j-1, K steps outermost: the two products into one
                // accumulator are CTH * PT apart; the fragment of step q2+2 is read
                // while step q2's products run.
                const unsigned char *wb = wb_slots + ((j - 1) & 1) * PB;
                const unsigned char *hin = hslots + ((j - 1) & 1) * HTILE;
                Frag<f16_t> hb[KM][PT];
                constexpr int NQ = KM * CTH;
                auto bfrag = [&](int q2) {
                    return wb + (((CTH * half + q2 % CTH) * KM + q2 / CTH) * 64 + lane) * 16;
                };
                Frag<f16_t> a2[4];
                a2[0].v = *reinterpret_cast<const f16x8 *>(bfrag(0));
#pragma unroll
                for (int km = 0; km < KM; ++km)
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt)
                        hb[km][pt].v = *reinterpret_cast<const f16x8 *>(hin + ((km * PT + pt) * 64 + lane) * 16);
                a2[1].v = *reinterpret_cast<const f16x8 *>(bfrag(1));
#pragma unroll
                for (int q2 = 0; q2 < NQ; ++q2) {
                    if (q2 + 2 < NQ) a2[(q2 + 2) & 3].v = *reinterpret_cast<const f16x8 *>(bfrag(q2 + 2));
                    const int km = q2 / CTH, ct = q2 % CTH;
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt) mma(Z[ct][pt], a2[q2 & 3], hb[km][pt]);
                }
            }
            wait_vmcnt<0>();  // this wave's copies of the step landed
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __syncthreads();
        }

        // lane (li, g) of tile pt holds channels C/2 half + 32k + 8g + 4i + r in Z[2k + i][pt][r]
#pragma unroll
        for (int ct = 0; ct < CTH; ++ct)
#pragma unroll
            for (int pt = 0; pt < PT; ++pt)
                *reinterpret_cast<f32x4 *>(zrows + (grp * 16 * PT + pt * 16 + li) * ZLD + half * (C / 2) + 32 * (ct >> 1) + 8 * g +
                                           4 * (ct & 1)) = Z[ct][pt];
    }
    // out = x + pa + z + bb and the next block's LN1 of the rounded output
    uint4 xv[CK], pv[CK];
    if (rows) load_row(xv, pv);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();  // the sums are in LDS
    if (!rows) return;
    float o[CK][8];
#pragma unroll
    for (int k = 0; k < CK; ++k) {
        float a[8], b[8];
        unpack8(xv[k], a);
        unpack8(pv[k], b);
        const float *zr = zrows + (wave * 16 + li) * ZLD + 32 * k + 8 * g;
        const f32x4 z0 = *reinterpret_cast<const f32x4 *>(zr), z1 = *reinterpret_cast<const f32x4 *>(zr + 4);
        const f32x4 d0 = *reinterpret_cast<const f32x4 *>(bb + 32 * k + 8 * g);
        const f32x4 d1 = *reinterpret_cast<const f32x4 *>(bb + 32 * k + 8 * g + 4);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            o[k][t] = (a[t] + b[t]) + (z0[t] + d0[t]);
            o[k][t + 4] = (a[t + 4] + b[t + 4]) + (z1[t] + d1[t]);
        }
        const uint4 u = pack8(o[k]);
        if (pr < n) *reinterpret_cast<uint4 *>(xo + pr * C + 32 * k + 8 * g) = u;
        unpack8(u, o[k]);
    }
    if (!lnn_g) return;  // uniform
    normalise(o, lnn_g, lnn_b);
    if (pr < n)
#pragma unroll
        for (int k = 0; k < CK; ++k) *reinterpret_cast<uint4 *>(xn + pr * C + 32 * k + 8 * g) = pack8(o[k]);
}

}  // namespace ts3
