// Point-wise passes of float32 storage on bf16 matrix cores with three-part operands
// (Parts): pass 2 (k_deslice3, Eq. (5)) and the backward's dx pass (k_bw_dx3).
//
// Both keep their points' rows as B operands in registers and read every A operand
// (weights, cached state, state gradients) from an LDS ring that the workgroup fills
// by direct copies several units ahead: the operands of a head are stored as parts in
// the order in which they are used, so a unit (two K steps of the slice tiles, or one K
// step of the channel tiles) is one contiguous piece. One barrier per unit.
#pragma once
#include "ts3_backward.h"
#include "ts3_pass2.h"
#include "ts3_rt.h"

namespace ts3 {

// Rows of A tiles over K = channels: fragments [H][CK][MT][3][64][8], lane l, slot t =
// src(h, 16*mt + (l&15), 32*kc + 8*(l>>4) + t).
// Rows of A tiles over K = slices: fragments [H][KM][CT][3][64][8], lane l, slot t =
// src(h, channel 16*ct + (l&15), slice 32*km + 16*(t>>2) + 4*(l>>4) + (t&3)), zero past
// M: the order in which a logits tile's registers hold the slices.
template <typename Src>
__device__ __forceinline__ void prep_over_channels(bf16_t *dst, int C, int H, int M, int64_t first, int64_t step, Src src) {
    const int CK = C / 32, MT = M / 16;
    const int64_t total = (int64_t)H * CK * MT * 512;
    for (int64_t i = first; i < total; i += step) {
        const int t = (int)(i & 7), lane = (int)((i >> 3) & 63);
        int64_t r = i >> 9;
        const int64_t at = (r * 3 * 64 + lane) * 8 + t;
        const int mt = (int)(r % MT); r /= MT;
        const int kc = (int)(r % CK), h = (int)(r / CK);
        store_parts(dst, at, src(h, mt * 16 + (lane & 15), kc * 32 + (lane >> 4) * 8 + t), 3);
    }
}
template <typename Src>
__device__ __forceinline__ void prep_over_slices(bf16_t *dst, int C, int H, int M, int64_t first, int64_t step, Src src) {
    const int CT = C / 16, KM = M >= 32 ? M / 32 : 1;
    const int64_t total = (int64_t)H * KM * CT * 512;
    for (int64_t i = first; i < total; i += step) {
        const int t = (int)(i & 7), lane = (int)((i >> 3) & 63);
        int64_t r = i >> 9;
        const int64_t at = (r * 3 * 64 + lane) * 8 + t;
        const int ct = (int)(r % CT); r /= CT;
        const int km = (int)(r % KM), h = (int)(r / KM);
        const int m = km * 32 + (t >> 2) * 16 + (lane >> 4) * 4 + (t & 3);
        store_parts(dst, at, m < M ? src(h, ct * 16 + (lane & 15), m) : 0.f, 3);
    }
}
// Element (h, channel c, slice m) of the second layout.
__device__ __forceinline__ int64_t z3_index(int h, int m, int c, int CT, int KM) {
    const int mm = m & 31, t = (mm >> 4) * 4 + (mm & 3), g = (mm & 15) >> 2;
    return (((((int64_t)h * KM + (m >> 5)) * CT + (c >> 4)) * 3) * 64 + g * 16 + (c & 15)) * 8 + t;
}

// W2' = W2 * scale over K = channels, b2s = b2 * scale (scale = log2(e) / tau).
__global__ void k_prep_w2x(const float *__restrict__ W2, const float *__restrict__ b2, float scale, int C, int H, int M,
                           bf16_t *__restrict__ w2x, float *__restrict__ b2s) {
    const int HM = H * M;
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    prep_over_channels(w2x, C, H, M, tid, (int64_t)gridDim.x * blockDim.x,
                       [&](int h, int m, int c) { return W2[(int64_t)c * HM + h * M + m] * scale; });
    if (tid < HM) b2s[tid] = (b2 ? b2[tid] : 0.f) * scale;
}

// Z + b3 / H over K = slices (each head's weights sum to one, so the heads add b3 once).
__global__ void k_prep_z3(const float *__restrict__ Z, const float *__restrict__ b3, int C, int H, int M,
                          bf16_t *__restrict__ zx) {
    const float bscale = 1.f / (float)H;
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    prep_over_slices(zx, C, H, M, tid, (int64_t)gridDim.x * blockDim.x,
                     [&](int h, int c, int m) { return Z[((int64_t)h * M + m) * C + c] + b3[c] * bscale; });
}

// The dx pass's operands: Z and ds_raw over K = channels, W2 (unscaled) and ds_raw over
// K = slices.
struct BwOperands {
    bf16_t *zr, *ds, *w2t, *dst;
};
__global__ void k_bw_prep(const float *__restrict__ Z, const float *__restrict__ dsr, const float *__restrict__ W2, int C,
                          int H, int M, BwOperands o) {
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    prep_over_channels(o.zr, C, H, M, tid, step, [&](int h, int m, int c) { return Z[((int64_t)h * M + m) * C + c]; });
    prep_over_channels(o.ds, C, H, M, tid, step, [&](int h, int m, int c) { return dsr[((int64_t)h * M + m) * C + c]; });
    prep_over_slices(o.w2t, C, H, M, tid, step, [&](int h, int c, int m) { return W2[(int64_t)c * H * M + h * M + m]; });
    prep_over_slices(o.dst, C, H, M, tid, step, [&](int h, int c, int m) { return dsr[((int64_t)h * M + m) * C + c]; });
}

// The workgroup's operand ring: R slots of SLOT KB; unit u sits in slot u % R and is
// copied R - 1 units ahead of its use.  CP: the least copies that a wave issues per
// unit, which bounds how many may still be in flight when the next unit's are awaited
// (anything else a wave has issued since only makes the wait stricter).
template <int WAVES, int R, int SLOT, int CP> struct Ring3 {
    uint32_t base;  // LDS address of the ring
    int wave, lane, put, get;
    __device__ __forceinline__ Ring3(unsigned char *lds, int wave_, int lane_)
        : base(lds_addr(lds)), wave(wave_), lane(lane_), put(0), get(0) {}
    // N fragments (1 KB each) from src into the next slot; waves past the last
    // fragment copy it again.
    template <int N> __device__ __forceinline__ void issue(const bf16_t *src) {
        constexpr int PER = (N + WAVES - 1) / WAVES;
        static_assert(PER >= CP && N <= SLOT, "slot size and wait count");
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int f = __builtin_amdgcn_readfirstlane(wave + i * WAVES < N ? wave + i * WAVES : N - 1);
            dma16(src + (size_t)f * 512 + lane * 8, base + (uint32_t)(put * SLOT + f) * 1024u);
        }
        put = put + 1 == R ? 0 : put + 1;
    }
    // Waits until the next unit has landed for every wave; the slot of the unit before
    // it is free afterwards.  Returns the unit's byte offset in the ring.
    __device__ __forceinline__ uint32_t next() {
        wait_vmcnt<(R - 2) * CP>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        const uint32_t at = (uint32_t)(get * SLOT) * 1024u;
        get = get + 1 == R ? 0 : get + 1;
        return at;
    }
};

// acc[r][t] += A tile r . B[t] for NR row tiles read from LDS at p (parts 1 KB apart) and
// NT point tiles; part products outermost, so consecutive MFMAs are independent.  With
// EXACT the step's products are summed from zero, the leading ones (of 16-bit
// significands, which the matrix core adds all but exactly) apart from the others, and
// added on the vector unit: the slice weights and dz of the backward, whose errors
// would add up in sums over all points in which the rest cancels.
template <int NR, int NT, bool EXACT = false>
__device__ __forceinline__ void mma_unit(f32x4 (*acc)[NT], const unsigned char *p, int lane, const Parts<3> (&b)[NT]) {
    Parts<3> a[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) a[r].p[k] = *reinterpret_cast<const bf16x8 *>(p + (r * 3 + k) * 1024 + lane * 16);
    using PP = PartProducts<3, 3>;
    f32x4 sum[NR][NT];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) sum[r][t] = EXACT ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[r][t];
#pragma unroll
    for (int q = 0; q < (EXACT ? 5 : 6); ++q)
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) sum[r][t] = mma_bf16(a[r].p[PP::I[q]], b[t].p[PP::J[q]], sum[r][t]);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            acc[r][t] = EXACT ? (acc[r][t] + sum[r][t]) + mma_bf16(a[r].p[0], b[t].p[0], f32x4{0.f, 0.f, 0.f, 0.f}) : sum[r][t];
}
// The same over all of a unit's MT row tiles, two at a time.
template <int MT, int NT>
__device__ __forceinline__ void mma_exact(f32x4 (&acc)[MT][NT], const unsigned char *p, int lane, const Parts<3> (&b)[NT]) {
    constexpr int G = MT < 2 ? 1 : 2;
#pragma unroll
    for (int mt = 0; mt < MT; mt += G) {
        mma_unit<G, NT, true>(&acc[mt], p + mt * 3072, lane, b);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Slices of K step km of a [slices x points] tile (lane (g, li): 16mt + 4g + r of point
// li) as the B operand's parts, slot t = slice 32km + 16(t>>2) + 4g + (t&3).
template <int MT, int NT>
__device__ __forceinline__ void pack_parts(const f32x4 (&E)[MT][NT], int t, int km, Parts<3> &f) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int mt = 2 * km + (i >> 2);
        v[i] = mt < MT ? E[mt < MT ? mt : 0][t][i & 3] : 0.f;
    }
    split8(v, f);
}

// softmax_tile of ts3_backward.h over one point tile of an [MT][NT] array.
template <int MT, int NT> __device__ __forceinline__ void softmax_col(f32x4 (&E)[MT][NT], int t, float scale) {
    f32x4 e[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) e[mt] = E[mt][t];
    softmax_tile<MT>(e, scale);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) E[mt][t] = e[mt];
}

// Point rows as B operands.
template <int NT, int CK>
__device__ __forceinline__ void load_points(const float *x, int64_t n, int C, int64_t p0, int li, int g,
                                            Parts<3> (&xb)[CK][NT]) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int64_t p = p0 + 16 * t + li;
        const float *row = x + (p < n ? p : n - 1) * C + 8 * g;
#pragma unroll
        for (int kc = 0; kc < CK; ++kc) {
            float v[8];
            rt_load8(v, row + 32 * kc, true);
            split8(v, xb[kc][t]);
        }
    }
}

template <int C, int M, int NT> struct Deslice3Cfg {
    static constexpr int MT = M / 16, CT = C / 16, CK = C / 32, KM = M >= 32 ? M / 32 : 1;
    static constexpr int WAVES = 8, PTS = WAVES * 16 * NT;
    static constexpr int N1 = MT * 3, N2 = 12;  // fragments per unit: a K step of W2'; four channel tiles of Z
    static constexpr int SLOT = N1 > N2 ? N1 : N2, R = 6;
    static constexpr int UNITS = CK + KM * (CT / 4);  // per head
    static constexpr int CP = (N1 + WAVES - 1) / WAVES;
};

// Pass 2 for float32 storage: eight waves (two per SIMD, so one wave's softmax runs
// beside the other's products) of 16 * NT points each, persistent over blocks; the ring
// runs on across heads and blocks.  W2' and Z fragments are read from LDS once per
// wave for NT tiles.  Bound by the matrix cores (192 MFMAs per 16 points and head at
// C = 128, M = 64).  As four waves of 32 points reading float32 fragments from L2 per
// wave, 1M points took 4.73 ms.
// x, out: [n][C]; w2x: W2' over channels, zx: Z over slices.
template <int C, int M, int NT>
__global__ __launch_bounds__(512, 1) void k_deslice3(const float *__restrict__ x, int64_t n, int32_t H,
                                                     const bf16_t *__restrict__ w2x, const float *__restrict__ b2s,
                                                     const bf16_t *__restrict__ zx, float *__restrict__ out) {
    using Cfg = Deslice3Cfg<C, M, NT>;
    constexpr int MT = Cfg::MT, CT = Cfg::CT, CK = Cfg::CK, KM = Cfg::KM, UNITS = Cfg::UNITS;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[Cfg::R * Cfg::SLOT * 1024];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int li = lane & 15, g = lane >> 4;
    const int64_t nblk = (n + Cfg::PTS - 1) / Cfg::PTS;
    if ((int64_t)blockIdx.x >= nblk) return;  // uniform over the workgroup
    const int64_t blocks = (nblk - 1 - blockIdx.x) / gridDim.x + 1;

    Ring3<Cfg::WAVES, Cfg::R, Cfg::SLOT, Cfg::CP> ring(lds, wave, lane);
    int64_t left = blocks * H * UNITS;  // units still to be copied
    int ih = 0, iu = 0;                 // the next one: head, unit of the head
    auto issue = [&]() {
        if (left > 0) {
            --left;
            if (iu < CK) ring.template issue<Cfg::N1>(w2x + ((size_t)ih * CK + iu) * Cfg::N1 * 512);
            else ring.template issue<Cfg::N2>(zx + ((size_t)ih * KM * CT / 4 + (iu - CK)) * Cfg::N2 * 512);
            if (++iu == UNITS) {
                iu = 0;
                if (++ih == H) ih = 0;
            }
        } else {  // past the end: keep the wait counts uniform with a copy that is not used
            ring.template issue<Cfg::N1>(w2x);
        }
    };
#pragma unroll 1
    for (int i = 0; i < Cfg::R - 1; ++i) issue();

    for (int64_t i = 0; i < blocks; ++i) {
        const int64_t p0 = ((int64_t)blockIdx.x + i * gridDim.x) * Cfg::PTS + wave * (16 * NT);
        Parts<3> xb[CK][NT];
        load_points<NT, CK>(x, n, C, p0, li, g, xb);
        f32x4 O[CT][NT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int t = 0; t < NT; ++t) O[ct][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        f32x4 bias[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) bias[mt] = *reinterpret_cast<const f32x4 *>(b2s + mt * 16 + g * 4);
#pragma unroll 1
        for (int h = 0; h < H; ++h) {
            f32x4 L[MT][NT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int t = 0; t < NT; ++t) L[mt][t] = bias[mt];
                // the next head's, a head ahead: a wait for them also covers the copies before them
                bias[mt] = *reinterpret_cast<const f32x4 *>(b2s + (h + 1 < H ? h + 1 : h) * M + mt * 16 + g * 4);
            }
#pragma unroll
            for (int kc = 0; kc < CK; ++kc) {
                const uint32_t at = ring.next();
                issue();
                constexpr int G = MT < 2 ? 1 : 2;
#pragma unroll
                for (int mt = 0; mt < MT; mt += G) mma_unit<G, NT>(&L[mt], lds + at + mt * 3072, lane, xb[kc]);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) softmax_col<MT, NT>(L, t, 1.f);
#pragma unroll
            for (int km = 0; km < KM; ++km) {
                Parts<3> wb[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) pack_parts<MT, NT>(L, t, km, wb[t]);
#pragma unroll
                for (int c4 = 0; c4 < CT; c4 += 4) {
                    const uint32_t at = ring.next();
                    issue();
#pragma unroll
                    for (int r = 0; r < 4; r += 2) mma_unit<2, NT>(&O[c4 + r], lds + at + r * 3072, lane, wb);
                }
            }
        }
        // lane (g, li) of tile ct: channels 16ct + 4g .. +3 of point li
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int64_t p = p0 + 16 * t + li;
            if (p >= n) continue;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                *reinterpret_cast<float4 *>(out + p * C + ct * 16 + g * 4) =
                    float4{O[ct][t][0], O[ct][t][1], O[ct][t][2], O[ct][t][3]};
        }
    }
    wait_vmcnt<0>();  // no copy may land after the workgroup's LDS is given to another
}

template <int C, int M> struct BwDx3Cfg {
    static constexpr int MT = M / 16, CT = C / 16, CK = C / 32, KM = M >= 32 ? M / 32 : 1;
    static constexpr int NT = 1, WAVES = 8, PTS = WAVES * 16 * NT;
    static constexpr int N1 = 2 * MT * 3, N2 = CT * 3;  // two K steps of slice tiles; one of channel tiles
    static constexpr int SLOT = N1 > N2 ? N1 : N2, R = 5;
    static constexpr int U1 = CK / 2;                   // units of one operand over channels
    static constexpr int UNITS = 3 * U1 + 2 * KM;       // per head
    static constexpr int CP = ((N1 < N2 ? N1 : N2) + WAVES - 1) / WAVES;
    static_assert(CK % 2 == 0, "channel K steps in pairs");
};

// dx for eight waves of 16 points (two per SIMD): per head
//   w   = softmax(W2' x + b2')                          2 C M products per point
//   dw  = Z g + ds_raw x + dd, dz = w (dw - sum w dw) / tau     4 C M
//   dx += W2 dz + ds_raw^T w                                    4 C M
// dz is also written to dzs [H][n][M] (the dW2 pass reads it there).  480 MFMAs per 16
// points and head at C = 128, M = 64, and each fragment read from LDS feeds six: the
// LDS reads take as long as the products.  Four waves of 32 points would halve the
// reads, but their operands do not fit beside two banks of 256 registers (279 spills,
// 6.7 ms per 1M points).  With float32 MFMAs and fragments read from L2 by
// every wave, 1M points took 7.08 ms.
template <int C, int M>
__global__ __launch_bounds__(512, 1) void k_bw_dx3(const float *__restrict__ x, const float *__restrict__ gout, int64_t n,
                                                   int32_t H, const bf16_t *__restrict__ w2x,
                                                   const float *__restrict__ b2s, BwOperands op,
                                                   const float *__restrict__ dd, float inv_tau,
                                                   float *__restrict__ dx, float *__restrict__ dzs) {
    using Cfg = BwDx3Cfg<C, M>;
    constexpr int MT = Cfg::MT, CT = Cfg::CT, CK = Cfg::CK, KM = Cfg::KM, NT = Cfg::NT, U1 = Cfg::U1;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[Cfg::R * Cfg::SLOT * 1024];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int li = lane & 15, g = lane >> 4;
    const int64_t p0 = (int64_t)blockIdx.x * Cfg::PTS + wave * (16 * NT);  // waves past n work on its last row

    Ring3<Cfg::WAVES, Cfg::R, Cfg::SLOT, Cfg::CP> ring(lds, wave, lane);
    int ih = 0, iu = 0;
    auto issue = [&]() {
        const int h = ih < H ? ih : 0;  // past the end: a copy that is not used
        const size_t c1 = (size_t)h * U1, c2 = (size_t)h * KM;
        // order: W2' | Z and ds_raw in turn | W2 and ds_raw^T in turn
        if (iu < U1) ring.template issue<Cfg::N1>(w2x + (c1 + iu) * Cfg::N1 * 512);
        else if (iu < 3 * U1) {
            const int v = iu - U1;
            ring.template issue<Cfg::N1>((v & 1 ? op.ds : op.zr) + (c1 + (v >> 1)) * Cfg::N1 * 512);
        } else {
            const int v = iu - 3 * U1;
            ring.template issue<Cfg::N2>((v & 1 ? op.dst : op.w2t) + (c2 + (v >> 1)) * Cfg::N2 * 512);
        }
        if (++iu == Cfg::UNITS) {
            iu = 0;
            ++ih;
        }
    };
#pragma unroll 1
    for (int i = 0; i < Cfg::R - 1; ++i) issue();

    Parts<3> xb[CK][NT], gb[CK][NT];
    load_points<NT, CK>(x, n, C, p0, li, g, xb);
    load_points<NT, CK>(gout, n, C, p0, li, g, gb);
    bool valid[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) valid[t] = p0 + 16 * t + li < n;
    f32x4 O[CT][NT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int t = 0; t < NT; ++t) O[ct][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int h = 0; h < H; ++h) {
        f32x4 E[MT][NT], Dz[MT][NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const float4 b = *reinterpret_cast<const float4 *>(b2s + h * M + mt * 16 + g * 4);
            const float4 d = *reinterpret_cast<const float4 *>(dd + h * M + mt * 16 + g * 4);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                E[mt][t] = f32x4{b.x, b.y, b.z, b.w};
                Dz[mt][t] = f32x4{d.x, d.y, d.z, d.w};
            }
        }
#pragma unroll
        for (int u = 0; u < U1; ++u) {
            const uint32_t at = ring.next();
            issue();
            mma_exact<MT, NT>(E, lds + at, lane, xb[2 * u]);
            mma_exact<MT, NT>(E, lds + at + MT * 3072, lane, xb[2 * u + 1]);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) softmax_col<MT, NT>(E, t, valid[t] ? 1.f : 0.f);
#pragma unroll
        for (int u = 0; u < U1; ++u) {
            uint32_t at = ring.next();
            issue();
            mma_exact<MT, NT>(Dz, lds + at, lane, gb[2 * u]);
            mma_exact<MT, NT>(Dz, lds + at + MT * 3072, lane, gb[2 * u + 1]);
            at = ring.next();
            issue();
            mma_exact<MT, NT>(Dz, lds + at, lane, xb[2 * u]);
            mma_exact<MT, NT>(Dz, lds + at + MT * 3072, lane, xb[2 * u + 1]);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            float s = 0.f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) s += E[mt][t][r] * Dz[mt][t][r];
            s = xrow_sum(s);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) Dz[mt][t][r] = inv_tau * E[mt][t][r] * (Dz[mt][t][r] - s);
            if (valid[t]) {
                // lane (g, li): slices 16mt + 4g .. +3 of point p0 + 16t + li
                float *row = dzs + ((size_t)h * n + p0 + 16 * t + li) * M + 4 * g;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    *reinterpret_cast<f32x4 *>(row + 16 * mt) = Dz[mt][t];
            }
        }
#pragma unroll
        for (int km = 0; km < KM; ++km) {
            Parts<3> b[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) pack_parts<MT, NT>(Dz, t, km, b[t]);
            uint32_t at = ring.next();
            issue();
#pragma unroll
            for (int ct = 0; ct < CT; ct += 2) mma_unit<2, NT>(&O[ct], lds + at + ct * 3072, lane, b);
#pragma unroll
            for (int t = 0; t < NT; ++t) pack_parts<MT, NT>(E, t, km, b[t]);
            at = ring.next();
            issue();
#pragma unroll
            for (int ct = 0; ct < CT; ct += 2) mma_unit<2, NT>(&O[ct], lds + at + ct * 3072, lane, b);
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int64_t p = p0 + 16 * t + li;
        if (!valid[t]) continue;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
            *reinterpret_cast<f32x4 *>(dx + p * C + ct * 16 + g * 4) = O[ct][t];
    }
    wait_vmcnt<0>();  // no copy may land after the workgroup's LDS is given to another
}

}  // namespace ts3
