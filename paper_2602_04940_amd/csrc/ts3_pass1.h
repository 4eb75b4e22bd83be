// Pass 1 of the Physics-Attention layer: slice logits, per-head temperature
// softmax and the tile contraction s_raw += w^T x, d += sum_i w_i (paper
// Eq. (1) and Eq. (4), Algorithm 1 tile loop).  The slice weights exist only in
// registers and a per-wave LDS scratch tile.
//
// Work decomposition: one workgroup per (span, head).  A span is Q consecutive
// mesh points; its four waves take 32-point blocks round-robin, each keeping a
// private M x C float32 accumulator of its head in registers, with head h's
// W2' fragments resident.  At the end the four wave accumulators are summed in
// a fixed order and written as the span's partial [M][C+1] (column C holds d).
// Spans are folded in index order later, so the result is a fixed function of
// (x, Q) whatever the tiling.
//
// Per 32-point block and wave (point rows 0..31 of the block):
//   x rows   arrive in a per-wave LDS ring by direct global->LDS copies, two
//            blocks ahead of use; they never pass through registers.
//   logits   L[m][p] = W2'[:, h*M+m] . x[p] + b2'   16x16x32 MFMA, A = W2'^T
//            fragments, B = x^T read from the ring; W2' = W2 * log2(e)/tau so
//            the softmax uses exp2.  Lane (g, li) of point tile pt holds
//            slices 16*mt + 4*g + r of point row prow(pt, li).
//   softmax  over the M slices of each point: in-lane, then two cross-row swaps.
//   w rows   normalised and written to a per-wave LDS tile.
//   contract S[m][c] += sum_p w[p][m] x[p][c] (A = w^T, B = x) and
//            d[m] += sum_p w[p][m] (A = w^T against a ones operand), with
//            ds_read_b64_tr_b16 giving operands whose K slots hold points:
//            slot (g, t) <-> point row 8g+t.
// The block loop is unrolled by the ring depth (every tile
// address is then a fixed per-lane offset plus an immediate), and block b-1's
// contraction (matrix cores) is interleaved with block b's softmax (vector
// ALU).
#pragma once
#include <type_traits>
#include "ts3_device.h"

namespace ts3 {

template <typename T, int C, int M> struct Pass1Cfg {
    static constexpr int CT = C / 16;      // 16-channel tiles
    static constexpr int MT = M / 16;      // 16-slice tiles
    static constexpr int CK = C / 32;      // K32 steps over channels
    static constexpr int WAVES = 4;
    static_assert(sizeof(T) == 2, "float32 storage has its own kernel");
    static constexpr int XROW = C * (int)sizeof(T);    // bytes per point row of x
    static constexpr int WROW = M * (int)sizeof(T);    // bytes per point row of w
    static constexpr int XTILE = 32 * XROW;
    static constexpr int WTILE = 32 * WROW;
    static constexpr int NS = 3;                       // ring depth (x and w tiles)
    static constexpr int ROWS_PER_LOAD = 1024 / XROW;  // rows per 1 KB wave copy
    static constexpr int LOADS = 32 / ROWS_PER_LOAD;   // wave copies per block
    static constexpr int WAVE_BYTES = NS * (XTILE + WTILE);
    static constexpr int XT_BYTES = WAVES * WAVE_BYTES;
    static constexpr int RED_BYTES = WAVES * M * (C + 1) * 4;
    static constexpr int LDS_BYTES = XT_BYTES > RED_BYTES ? XT_BYTES : RED_BYTES;
    static_assert(ROWS_PER_LOAD * XROW == 1024, "x rows must tile a 1 KB copy");
};

// Point row of lane li in point tile pt: bits 0-1 from li, bit 2 from pt,
// bits 3-4 from li >> 2, so point tiles 0 and 1 differ only in row bit 2.
__device__ __forceinline__ int prow(int pt, int li) { return (li & 3) | (pt << 2) | ((li >> 2) << 3); }

// Bank-conflict-free placement inside unpadded tile rows, for the LDS access
// phases measured on gfx950: ds_read_b128 serves 16 lanes per cycle from 64
// banks (256 B), the lanes of a cycle sharing lane bit 5 and the parity of
// lane bits 2, 3 and 4; ds_read_b64 (also the transposing form) serves lanes
// 0-31, then 32-63, from 64 banks; ds_write_b64 serves 16 consecutive lanes
// per cycle from 32 banks (128 B).  A cycle is conflict-free when its lanes
// touch distinct banks.  No swizzle below depends on row bit 2, so rows r and
// r+4 (point tile pt, transpose half) differ by a fixed offset; with 16-bit
// elements a step of the channel, slice or K index then changes the offset by
// an XOR with a constant.
// x rows (16-byte chunks): chunk k of row R sits at k ^ xswz(R).
template <int ROWB> __device__ __forceinline__ int xswz(int R) {
    constexpr int NCH = ROWB / 16;
    const int b0 = R & 1, b1 = (R >> 1) & 1, b3 = (R >> 3) & 1;
    const int f = NCH >= 16 ? ((b0 << 1) | (b1 << 2) | (b3 << 3)) : ((b1 << 1) | (b3 << 2));
    return f & (NCH - 1);
}
template <int ROWB> __device__ __forceinline__ int xoff(int R, int byte) {
    return R * ROWB + (((byte >> 4) ^ xswz<ROWB>(R)) << 4) + (byte & 15);
}
// w rows (8-byte slots): slot s of row R sits at s ^ wswz(R), chosen per row
// width for the 8-byte row stores (rows differing in bits 0, 1, 3, 4 in one
// cycle) and the transpose reads (four rows x four slots x two row groups);
// with 32-byte rows (M = 16) the transpose reads stay two-way.
template <int ROWB> __device__ __forceinline__ int wswz(int R) {
    constexpr int NSL = ROWB / 8;
    const int b0 = R & 1, b1 = (R >> 1) & 1, b3 = (R >> 3) & 1, b4 = (R >> 4) & 1;
    if constexpr (NSL >= 16) return b0 | (b4 << 1) | (b1 << 2) | (b3 << 3);
    else if constexpr (NSL == 8) return b1 | (b4 << 1) | (b3 << 2);
    else return (b3 | (b4 << 1)) & (NSL - 1);
}
template <int ROWB> __device__ __forceinline__ int woff(int R, int byte) {
    return R * ROWB + (((byte >> 3) ^ wswz<ROWB>(R)) << 3) + (byte & 7);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// One 8-slot operand fragment from two transposing LDS reads.  Lane (g, j) of
// each 16-lane row reads row 8g + 4*half + j/4, columns col0 + 4*(j%4) .. +3 of
// a tile; the result gives lane (g, i) column col0 + i of rows 8g .. 8g+7 in
// slots 0..7.  `lo` is the lane's address for half 0; half 1 is 4 rows on.
template <int ROWB>
__device__ __forceinline__ void tr_frag(Frag<bf16_t> &f, const unsigned char *lo) {
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)lo);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(lo + 4 * ROWB));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    f.v = __builtin_bit_cast(bf16x8, v);
}
template <int ROWB, bool XT>
__device__ __forceinline__ const unsigned char *tr_addr(const unsigned char *tile, int g, int col0, int j) {
    const int r = 8 * g + (j >> 2);
    const int byte = (col0 + 4 * (j & 3)) * 2;
    return tile + (XT ? xoff<ROWB>(r, byte) : woff<ROWB>(r, byte));
}
template <int V> using ic = std::integral_constant<int, V>;

// x       : tile base, [n_tile][C] storage elements
// n_tile  : points in this tile (tile starts on a span boundary)
// span0   : global index of the tile's first span
// geo     : the spans and the parts they are summed in
// nspan   : parts in this launch; grid = nspan * H
// w2p     : prepared W2' fragments [H][MT][CK][64 lanes][8]
// b2s     : W2'-scaled bias [H*M]
// partials: [span][H][M][C+1] float32
template <typename T, int C, int M>
__global__ __launch_bounds__(256, 1) void k_slice_accumulate(
    const T *__restrict__ x, int64_t n_tile, int64_t span0, SpanGeo geo, int32_t nspan, int32_t H,
    const T *__restrict__ w2p, const float *__restrict__ b2s, float *__restrict__ partials) {
    using Cfg = Pass1Cfg<T, C, M>;
    constexpr int CT = Cfg::CT, MT = Cfg::MT, CK = Cfg::CK;
    constexpr int XROW = Cfg::XROW, WROW = Cfg::WROW, NS = Cfg::NS;
    constexpr int XTILE = Cfg::XTILE, WTILE = Cfg::WTILE;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[Cfg::LDS_BYTES];

    const int nwg = nspan * H;
    const int jwg = xcd_remap((int)blockIdx.x, nwg);
    const int span_local = jwg / H;
    const int h = jwg - span_local * H;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int li = lane & 15;
    const int g = lane >> 4;

    const int64_t p_begin = geo.begin(span_local);
    const int64_t p_end = geo.end(span_local, n_tile);
    const int nblk = (int)((p_end - p_begin + 31) >> 5);
    const int nmine = nblk > wave ? (nblk - wave + Cfg::WAVES - 1) / Cfg::WAVES : 0;

    unsigned char *const wave_lds = lds + wave * Cfg::WAVE_BYTES;
    unsigned char *const xring = wave_lds;                // NS x tiles
    unsigned char *const wring = wave_lds + NS * XTILE;   // NS w tiles
    const uint32_t xring_lds = lds_addr(xring);

    // Block j of this wave (mesh block wave + 4j) into x slot SL.  Lane l of
    // copy i fills physical chunk l % NCH of row i*ROWS_PER_LOAD + l / NCH, so
    // it reads the logical chunk stored there.  Rows past the span's end
    // repeat its last point (finite data that the zero weights of padding
    // points cancel exactly), which also keeps every wave's copy count uniform.
    constexpr int NCH = XROW / 16;
    auto copy_off = [&](int i) {
        const int R = i * Cfg::ROWS_PER_LOAD + lane / NCH;
        return (uint32_t)(R * XROW + (((lane % NCH) ^ xswz<XROW>(R)) << 4));
    };
    auto issue_x = [&](int j, auto slot) {
        constexpr int SL = decltype(slot)::value;
        const int64_t p0 = p_begin + ((int64_t)(wave + Cfg::WAVES * j) << 5);
        const uint32_t dst = xring_lds + SL * XTILE;
        if (p0 + 32 <= p_end) {
            const void *base = x + p0 * C;
#pragma unroll
            for (int i = 0; i < Cfg::LOADS; ++i) dma16s<0>(copy_off(i), base, dst + i * 1024);
        } else {
#pragma unroll
            for (int i = 0; i < Cfg::LOADS; ++i) {
                const int R = i * Cfg::ROWS_PER_LOAD + lane / NCH;
                const int k = (lane % NCH) ^ xswz<XROW>(R);
                int64_t p = p0 + R;
                p = p < p_end ? p : p_end - 1;
                dma16(reinterpret_cast<const unsigned char *>(x + (size_t)p * C) + k * 16, dst + i * 1024);
            }
        }
    };

    // Head h's W2'^T fragments (A operand: lane row = slice) and bias, resident.
    Frag<T> w2[MT][CK];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int kc = 0; kc < CK; ++kc)
            load8(w2[mt][kc], w2p + ((((size_t)h * MT + mt) * CK + kc) * 64 + lane) * 8);
    f32x4 bias[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const float4 b = *reinterpret_cast<const float4 *>(b2s + h * M + mt * 16 + g * 4);
        bias[mt] = f32x4{b.x, b.y, b.z, b.w};
    }

    f32x4 S[MT][CT];
    f32x4 D[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        D[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) S[mt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    Frag<T> ones;
    ones8(ones);
    // Settle the loads above before the x ring starts: the ring's counts
    // assume its own copies are the only memory operations in flight.
    wait_vmcnt<0>();

    // Max-shifted exp2 of the logits in place; per point the reciprocal row sum (zero
    // for padding points).
    auto softmax_shifted = [&](f32x4 (&L)[MT][2], float (&inv)[2], int valid) {
#pragma unroll
        for (int pt = 0; pt < 2; ++pt) {
            float mx = L[0][pt][0];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx = fmaxf(mx, L[mt][pt][r]);
            mx = xrow_max(mx);
            float sum = 0.f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float e = fast_exp2(L[mt][pt][r] - mx);
                    L[mt][pt][r] = e;
                    sum += e;
                }
            inv[pt] = prow(pt, li) < valid ? fast_rcp(xrow_sum(sum)) : 0.f;
        }
    };
    auto block_valid = [&](int j) {
        const int64_t left = p_end - (p_begin + ((int64_t)(wave + Cfg::WAVES * j) << 5));
        return (int)(left < 32 ? left : 32);
    };

    {
        // bf16 tile addresses as (per-lane base) ^ (tile-index constant) +
        // (immediate): with 16-bit elements a tile step moves whole chunks or
        // slots whose index bits do not overlap the base's, and neither
        // swizzle depends on row bit 2 (point tile pt, transpose half).
        static_assert(sizeof(T) == 2, "the pipelined path is written for 16-bit storage");
        const uint32_t wave_off = (uint32_t)(wave * Cfg::WAVE_BYTES);
        uint32_t xl0 = wave_off + xoff<XROW>(prow(0, li), 16 * g);               // logits B, kc = 0
        uint32_t xt0 = wave_off + xoff<XROW>(8 * g + (li >> 2), 8 * (li & 3));   // x^T, ct = 0
        uint32_t wt0 = wave_off + NS * XTILE + woff<WROW>(8 * g + (li >> 2), 8 * (li & 3));  // w^T, mt = 0
        uint32_t ws0 = wave_off + NS * XTILE + woff<WROW>(prow(0, li), 8 * g);   // w rows, mt = 0
        constexpr int PT_X = 4 * XROW, PT_W = 4 * WROW;  // row + 4

        // Logits of point tile pt for the block in x slot SL.
        auto logits16 = [&](auto slot, int pt, f32x4 (&L)[MT][2]) {
            constexpr int SL = decltype(slot)::value;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) L[mt][pt] = bias[mt];
#pragma unroll
            for (int kc = 0; kc < CK; ++kc) {
                Frag<T> xb;
                xb.v = *reinterpret_cast<const bf16x8 *>(lds + (xl0 ^ (kc << 6)) + SL * XTILE + pt * PT_X);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) mma(L[mt][pt], w2[mt][kc], xb);
            }
        };
        // Contraction operands of the block in slot SL: w^T for every slice
        // tile, x^T for channel tile ct.
        auto read_a = [&](auto slot, Frag<T> (&a)[MT]) {
            constexpr int SL = decltype(slot)::value;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) tr_frag<WROW>(a[mt], lds + (wt0 ^ (mt << 5)) + SL * WTILE);
        };
        auto read_b = [&](auto slot, int ct, Frag<T> &b) {
            constexpr int SL = decltype(slot)::value;
            tr_frag<XROW>(b, lds + (xt0 ^ (ct << 5)) + SL * XTILE);
        };
        auto contract16 = [&](auto slot) {
            Frag<T> a[MT], b;
            read_a(slot, a);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) mma(D[mt], a[mt], ones);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                read_b(slot, ct, b);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) mma(S[mt][ct], a[mt], b);
            }
        };
        auto store_w16 = [&](auto slot, const f32x4 (&E)[MT][2], const float (&inv)[2]) {
            constexpr int SL = decltype(slot)::value;
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
#pragma unroll
            for (int pt = 0; pt < 2; ++pt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    *reinterpret_cast<bf16x4 *>(lds + (ws0 ^ (mt << 5)) + SL * WTILE + pt * PT_W) =
                        bf16x4{(__bf16)(E[mt][pt][0] * inv[pt]), (__bf16)(E[mt][pt][1] * inv[pt]),
                               (__bf16)(E[mt][pt][2] * inv[pt]), (__bf16)(E[mt][pt][3] * inv[pt])};
        };
        // exp2 of point tile pt's logits in place; returns the in-lane sum.
        auto exp_tile = [&](f32x4 (&L)[MT][2], int pt) {
            float sum = 0.f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float e = fast_exp2(L[mt][pt][r]);
                    L[mt][pt][r] = e;
                    sum += e;
                }
            return sum;
        };

        // One block j in slot SL = j % NS, overlapping three streams:
        //   logits of point tile 0, then of tile 1 beside tile 0's exp2;
        //   the previous block's contraction beside tile 1's exp2, the
        //   normalisation and this block's w rows;
        //   then the copy of block j + NS - 1 into the slot just freed.
        auto step = [&](int j, auto slot) {
            constexpr int SL = decltype(slot)::value;
            constexpr int PREV = (SL + NS - 1) % NS;
            // Keep the derived addresses inside the step (recomputed with one
            // XOR each) instead of occupying registers across the loop.
            asm volatile("" : "+v"(xl0), "+v"(xt0), "+v"(wt0), "+v"(ws0));
            const int valid = block_valid(j);
            Frag<T> a[MT], b;
            read_a(ic<PREV>{}, a);  // the previous block's tiles are complete
            read_b(ic<PREV>{}, 0, b);
            wait_vmcnt<(NS - 2) * Cfg::LOADS>();  // block j's rows have landed
            asm volatile("" ::: "memory");
            f32x4 L[MT][2];
            logits16(slot, 0, L);
            __builtin_amdgcn_sched_barrier(0);
            logits16(slot, 1, L);
            float sum0 = exp_tile(L, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, CK, 0);
#pragma unroll
            for (int i = 0; i < MT * CK; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) mma(D[mt], a[mt], ones);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                Frag<T> bn;
                if (ct + 1 < CT) read_b(ic<PREV>{}, ct + 1, bn);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) mma(S[mt][ct], a[mt], b);
                b = bn;
            }
            float sum1 = exp_tile(L, 1);
            sum0 = xrow_sum(sum0);
            sum1 = xrow_sum(sum1);
            const bool ok = softmax_sum_ok(sum0) && softmax_sum_ok(sum1);
            float inv[2] = {prow(0, li) < valid ? fast_rcp(sum0) : 0.f, prow(1, li) < valid ? fast_rcp(sum1) : 0.f};
            store_w16(slot, L, inv);
            interleave_chain<0, MT * (CT + 1), 5, MT - 1, MT, 2, 2 * MT>();
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue_x(j + NS - 1, ic<PREV>{});
            if (__any(!ok)) {
                // Rare: some row's exp2 sum left the safe window; redo the
                // block with the max shift.
                logits16(slot, 0, L);
                logits16(slot, 1, L);
                softmax_shifted(L, inv, valid);
                store_w16(slot, L, inv);
            }
            asm volatile("" ::: "memory");
        };
        // The tiles of "block -1" (slot NS-1) hold zeros, so the first step's
        // contraction of the previous block adds exactly nothing.
        {
            uint4 *zx = reinterpret_cast<uint4 *>(xring + (NS - 1) * XTILE);
            uint4 *zw = reinterpret_cast<uint4 *>(wring + (NS - 1) * WTILE);
            for (int i = lane; i < XTILE / 16; i += 64) zx[i] = uint4{0u, 0u, 0u, 0u};
            for (int i = lane; i < WTILE / 16; i += 64) zw[i] = uint4{0u, 0u, 0u, 0u};
        }
        static_assert(NS == 3, "the unrolled loop below assumes a ring of three");
        issue_x(0, ic<0>{});
        issue_x(1, ic<1>{});
        int j = 0;
        for (; j + 3 <= nmine; j += 3) {
            step(j, ic<0>{});
            step(j + 1, ic<1>{});
            step(j + 2, ic<2>{});
        }
        if (j < nmine) step(j, ic<0>{});
        if (j + 1 < nmine) step(j + 1, ic<1>{});
        wait_vmcnt<0>();
        switch ((nmine + NS - 1) % NS) {  // the last block (slot 2 if there was none)
            case 0: contract16(ic<0>{}); break;
            case 1: contract16(ic<1>{}); break;
            default: contract16(ic<2>{}); break;
        }
    }

    // Fixed-order reduction of the four wave accumulators.
    __syncthreads();
    float *red = reinterpret_cast<float *>(lds);
    float *mine = red + (size_t)wave * M * (C + 1);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = mt * 16 + g * 4 + r;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) mine[m * (C + 1) + ct * 16 + li] = S[mt][ct][r];
            if (li == 0) mine[m * (C + 1) + C] = D[mt][r];
        }
    __syncthreads();
    constexpr int E = M * (C + 1);
    float *dst = partials + ((size_t)(span0 + span_local) * H + h) * E;
    for (int e = threadIdx.x; e < E; e += 256)
        dst[e] = (red[e] + red[E + e]) + (red[2 * E + e] + red[3 * E + e]);
}

}  // namespace ts3
