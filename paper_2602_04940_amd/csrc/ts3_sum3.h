// Sums over the points of a part for float32 storage, on bf16 matrix cores with
// three-part operands (Parts):
//     partial[m][c] = sum_p a[p][m] b[p][c],   column C = sum_p a[p][m]
// with a the slice weights of x, computed here (pass 1 with b = x, Eq. (4); the
// backward's dZ pass with b = g), or rows stored earlier (the backward's dW2 pass: a =
// dz, b = x).
//
// One workgroup of eight waves per (part, head), blocks of 64 points.  Waves q and
// q + 4 share a SIMD:
//   producer q  a of the block's points 16q .. 16q+15, as parts to the w tile (two
//               slots): the logits (A = W2'^T parts, the first two resident in
//               registers, the third in LDS), the max-shifted softmax; or the stored
//               rows;
//   consumer q  the previous block's contraction for its own quarter of the
//               channels (A = a^T, B = b^T from transposing LDS reads of its b region).
// One barrier per block.  No wave's sum needs another's, and each runs over the
// part's blocks in order.  The b rows are split into parts once, by the wave with less
// vector work:
//   weights of x, b = x (pass 1)  consumer q, a block ahead (two region slots); the
//                                 producers read the logits' B operand there too
//   weights of x, b = g (dZ)      consumer q, one slot that only it reads; the producers
//                                 load and split x themselves
//   stored rows (dW2)             producer q, with a's (two slots)
// Bound by vector instructions beside the matrix cores' 195 MFMAs per 64 points and SIMD
// (C = 128, M = 64): a split costs 5.5 per element.  1M points took 3.04 ms (pass 1, four
// waves with float32 MFMAs), 3.10 ms (dZ) and 1.62 ms (dW2) before.
#pragma once
#include "ts3_backward.h"  // softmax_tile
#include "ts3_pass1.h"
#include "ts3_rt.h"        // mma_parts

namespace ts3 {

enum Sum3 { SUM3_X, SUM3_G, SUM3_STORED };

template <int C, int M, Sum3 KIND> struct Sum3Cfg {
    static constexpr int MT = M / 16, CK = C / 32, PTS = 64;
    static constexpr int CW = C / 4, CWT = CW / 16;      // a consumer's channels and channel tiles
    static constexpr int WROW = M * 2, BROW = CW * 2;    // bytes per point and part
    static constexpr int WPLANE = 32 * WROW, BPLANE = 32 * BROW;
    static constexpr int W_SLOT = 2 * 3 * WPLANE;        // two 32-point tiles of three parts
    static constexpr int B_REGION = 2 * 3 * BPLANE;      // a consumer's slot
    static constexpr int B_SLOTS = KIND == SUM3_G ? 1 : 2;
    static constexpr int W2LO = KIND == SUM3_STORED ? 0 : MT * CK * 1024;  // the third parts of W2'
    static constexpr int LDS_BYTES = 2 * W_SLOT + B_SLOTS * 4 * B_REGION + W2LO;
    static_assert(LDS_BYTES <= 160 * 1024, "tiles exceed LDS");
    static_assert(CWT >= 1 && MT <= 4, "channels split over four consumers");
};

// b region rows: 16-byte chunk k of row R sits at k ^ swizzle(R), which moves the rows
// 8 apart that a transposing read takes together to other banks.
template <int ROWB> __device__ __forceinline__ int boff(int R, int byte) {
    constexpr int NCH = ROWB / 16;
    return R * ROWB + (((byte >> 4) ^ (NCH >= 4 ? 2 * ((R >> 3) & 1) : 0)) << 4) + (byte & 15);
}
// Fragment of a b region plane: K slot (g, t) = row 8g + t, lane column col0 + (l & 15).
template <int ROWB> __device__ __forceinline__ bf16x8 b_frag(const unsigned char *plane, int g, int col0, int j) {
    Frag<bf16_t> f;
    tr_frag<ROWB>(f, plane + boff<ROWB>(8 * g + (j >> 2), (col0 + 4 * (j & 3)) * 2));
    return f.v;
}

// a: slice weights of the rows a_rows = x [n_tile][C] (w2x: W2' parts
// [H][CK][MT][3][64][8], b2s its bias), or stored rows a_rows [H][n_tile][M].  b_rows:
// [n_tile][C].  Grid: nspan * H.
template <int C, int M, Sum3 KIND>
__global__ __launch_bounds__(512, 1) void k_sum3(const float *__restrict__ a_rows, const float *__restrict__ b_rows,
                                                 int64_t n_tile, int64_t span0, SpanGeo geo, int32_t nspan, int32_t H,
                                                 const bf16_t *__restrict__ w2x, const float *__restrict__ b2s,
                                                 float *__restrict__ partials) {
    using Cfg = Sum3Cfg<C, M, KIND>;
    constexpr int MT = Cfg::MT, CK = Cfg::CK, CW = Cfg::CW, CWT = Cfg::CWT, PTS = Cfg::PTS;
    constexpr int WROW = Cfg::WROW, BROW = Cfg::BROW, WPLANE = Cfg::WPLANE, BPLANE = Cfg::BPLANE;
    constexpr int BSLOT = 4 * Cfg::B_REGION, BS = Cfg::B_SLOTS;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[Cfg::LDS_BYTES];
    unsigned char *const w_lds = lds, *const b_lds = lds + 2 * Cfg::W_SLOT;
    unsigned char *const w2lo = b_lds + BS * BSLOT;

    const int jwg = xcd_remap((int)blockIdx.x, nspan * H);  // a part's heads share an XCD (and its L2)
    const int span_local = jwg / H, h = jwg - span_local * H;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = wave & 3;
    const int li = lane & 15, g = lane >> 4;
    const int64_t p_begin = geo.begin(span_local);
    const int64_t p_end = geo.end(span_local, n_tile);
    const int nblk = (int)((p_end - p_begin + PTS - 1) / PTS);  // a launch's parts are not empty

    // Quarter q of the block's b rows: CHUNKS lanes per row, RPP rows per pass.  Rows
    // past the part's end repeat its last row (finite data against zero weights).
    constexpr int CHUNKS = CW / 8, RPP = 64 / CHUNKS, PASSES = PTS / RPP;
    const int crow = lane / CHUNKS, cch = lane % CHUNKS;
    float br[PASSES][8];
    auto load_b = [&](int j) {
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int64_t p = p_begin + (int64_t)j * PTS + i * RPP + crow;
            rt_load8(br[i], b_rows + (p < p_end ? p : p_end - 1) * C + q * CW + 8 * cch, true);
        }
    };
    auto store_b = [&](int slot) {
        unsigned char *const region = b_lds + slot * BSLOT + q * Cfg::B_REGION;
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int r = i * RPP + crow;
            Parts<3> f;
            split8(br[i], f);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                *reinterpret_cast<bf16x8 *>(region + ((r >> 5) * 3 + k) * BPLANE + boff<BROW>(r & 31, cch * 16)) = f.p[k];
        }
    };
    if constexpr (KIND != SUM3_STORED) {  // the third parts of the head's W2' fragments
        const bf16_t *src = w2x + (size_t)h * MT * CK * 3 * 512;
        for (int i = tid; i < MT * CK * 64; i += 512)
            *reinterpret_cast<bf16x8 *>(w2lo + i * 16) =
                *reinterpret_cast<const bf16x8 *>(src + ((i >> 6) * 3 + 2) * 512 + (i & 63) * 8);
    }
    // Block 0's b rows, which the producers of SUM3_X read in the first step.
    if (KIND == SUM3_X && wave >= 4) {
        load_b(0);
        store_b(0);
        load_b(1);
    }
    __syncthreads();

    if (wave < 4) {
        // ---------------------------------------------------------------- producer
        // Lane (g, li) owns row prow(q & 1, li) of the block's 32-point tile q >> 1.
        // Tile 1's rows are stored negated (see mma_parts_add).
        const int R = prow(q & 1, li);
        const float sign = q >> 1 ? -1.f : 1.f;
        unsigned char *const w_tile = w_lds + (q >> 1) * 3 * WPLANE;
        auto point = [&](int j) { return p_begin + (int64_t)j * PTS + (q >> 1) * 32 + R; };
        auto store_a = [&](int j, const f32x4 (&E)[MT]) {
            unsigned char *dst = w_tile + (j & 1) * Cfg::W_SLOT;
            typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                u32x2 u[3];
#pragma unroll
                for (int r = 0; r < 4; r += 2) {
                    const float a = E[mt][r], b = E[mt][r + 1];
                    const uint32_t hi = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
                    const float a1 = a - __uint_as_float(hi << 16), b1 = b - __uint_as_float(hi & 0xffff0000u);
                    const uint32_t mi = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a1, (__bf16)b1});
                    u[0][r >> 1] = hi;
                    u[1][r >> 1] = mi;
                    u[2][r >> 1] = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)(a1 - __uint_as_float(mi << 16)),
                                                                       (__bf16)(b1 - __uint_as_float(mi & 0xffff0000u))});
                }
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    *reinterpret_cast<u32x2 *>(dst + k * WPLANE + woff<WROW>(R, (mt * 16 + 4 * g) * 2)) = u[k];
            }
        };
        if constexpr (KIND == SUM3_STORED) {
            const float *rows = a_rows + (size_t)h * n_tile * M + 4 * g;
            f32x4 next[MT];
            auto load = [&](int j) {
                const int64_t p = point(j);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    next[mt] = *reinterpret_cast<const f32x4 *>(rows + (p < p_end ? p : p_end - 1) * M + 16 * mt);
            };
            load(0);
            load_b(0);
            for (int j = 0; j <= nblk; ++j) {
                if (j < nblk) {
                    f32x4 E[MT];
                    const float scale = point(j) < p_end ? sign : 0.f;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) E[mt] = scale * next[mt];
                    load(j + 1);
                    store_a(j, E);
                    store_b(j & 1);  // of which block j - 2 was contracted before the last barrier
                    load_b(j + 1);
                }
                __syncthreads();
            }
        } else {
            Parts<2> w2[MT][CK];
            f32x4 bias[MT];
            const bf16_t *src = w2x + ((size_t)h * MT * CK * 3 * 64 + lane) * 8;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int kc = 0; kc < CK; ++kc)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        w2[mt][kc].p[k] = *reinterpret_cast<const bf16x8 *>(src + ((kc * MT + mt) * 3 + k) * 512);
                const float4 b = *reinterpret_cast<const float4 *>(b2s + h * M + mt * 16 + g * 4);
                bias[mt] = f32x4{b.x, b.y, b.z, b.w};
            }
            constexpr bool SHARED = KIND == SUM3_X;  // x parts from the consumers' regions
            float xr[SHARED ? 1 : CK][8];
            auto load = [&](int j, int kc) {
                const int64_t p = point(j);
                rt_load8(xr[SHARED ? 0 : kc], a_rows + (p < p_end ? p : p_end - 1) * C + 32 * kc + 8 * g, true);
            };
            if constexpr (!SHARED)
#pragma unroll
                for (int kc = 0; kc < CK; ++kc) load(0, kc);
            for (int j = 0; j <= nblk; ++j) {
                if (j < nblk) {
                    f32x4 E[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) E[mt] = bias[mt];
#pragma unroll
                    for (int kc = 0; kc < CK; ++kc) {
                        Parts<3> xb;
                        if constexpr (SHARED) {
                            const int c = 32 * kc + 8 * g;
                            const unsigned char *src = b_lds + (j & 1) * BSLOT + (c / CW) * Cfg::B_REGION +
                                                       (q >> 1) * 3 * BPLANE + boff<BROW>(R, (c % CW) * 2);
#pragma unroll
                            for (int k = 0; k < 3; ++k) xb.p[k] = *reinterpret_cast<const bf16x8 *>(src + k * BPLANE);
                        } else {
                            split8(xr[kc], xb);
                            load(j + 1, kc);  // clamped to the part's last row
                        }
                        Parts<3> a[MT];
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) {
                            a[mt].p[0] = w2[mt][kc].p[0];
                            a[mt].p[1] = w2[mt][kc].p[1];
                            a[mt].p[2] = *reinterpret_cast<const bf16x8 *>(w2lo + ((kc * MT + mt) * 64 + lane) * 16);
                        }
                        mma_parts_add<MT, 3, 3>(E, a, xb, false);
                    }
                    softmax_tile<MT>(E, point(j) < p_end ? sign : 0.f);
                    store_a(j, E);
                }
                __syncthreads();
            }
        }
    } else {
        // ---------------------------------------------------------------- consumer
        f32x4 S[CWT][MT], D = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ct = 0; ct < CWT; ++ct)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) S[ct][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        Frag<bf16_t> ones;
        ones8(ones);
        if constexpr (KIND == SUM3_G) load_b(0);
        for (int j = 0; j <= nblk; ++j) {
            if (j > 0) {
                const unsigned char *wt = w_lds + ((j - 1) & 1) * Cfg::W_SLOT;
                const unsigned char *region = b_lds + (BS == 2 ? ((j - 1) & 1) * BSLOT : 0) + q * Cfg::B_REGION;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    Parts<3> a[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            Frag<bf16_t> f;
                            tr_frag<WROW>(f, tr_addr<WROW, false>(wt + (t * 3 + k) * WPLANE, g, mt * 16, li));
                            a[mt].p[k] = f.v;
                        }
#pragma unroll
                    for (int ct = 0; ct < CWT; ++ct) {
                        Parts<3> b;
#pragma unroll
                        for (int k = 0; k < 3; ++k) b.p[k] = b_frag<BROW>(region + (t * 3 + k) * BPLANE, g, ct * 16, li);
                        mma_parts_add<MT, 3, 3>(S[ct], a, b, t == 1);
                    }
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        if (mt == q) {  // wave-uniform
                            f32x4 d{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int k = 2; k >= 0; --k) d = mma_bf16(a[mt].p[k], ones.v, d);
                            D = t == 1 ? D - d : D + d;
                        }
                }
            }
            if constexpr (KIND == SUM3_G) {
                if (j < nblk) {
                    store_b(0);  // this wave's own reads of the region are done
                    load_b(j + 1);
                }
            } else if constexpr (KIND == SUM3_X) {
                if (j + 1 < nblk) {
                    store_b((j + 1) & 1);  // of which only this wave has still read (block j - 1, above)
                    load_b(j + 2);
                }
            }
            __syncthreads();
        }
        // lane (g, li) of tile (mt, ct): slice 16mt + 4g + r, channel q CW + 16ct + li
        float *dst = partials + ((size_t)(span0 + span_local) * H + h) * (size_t)(M * (C + 1));
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float *row = dst + (size_t)(mt * 16 + g * 4 + r) * (C + 1);
#pragma unroll
                for (int ct = 0; ct < CWT; ++ct) row[q * CW + ct * 16 + li] = S[ct][mt][r];
                if (mt == q && li == 0) row[C] = D[r];
            }
    }
}

}  // namespace ts3
