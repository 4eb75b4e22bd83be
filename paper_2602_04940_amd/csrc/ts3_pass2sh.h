// Pass 2 in the slice-state form with a head per wave (16-bit storage, head width 16):
// the products, their order and the softmax of k_deslice_sf (ts3_pass2sf.h), so every
// point's result is the same to the bit, split another way.
//
// One workgroup of H waves walks blocks of 32 points:
//   wave h   logits of head h (A = its W2'^T fragments, in registers for the whole
//            launch, B = x^T), exp2, u_h = (s'_h^T e) / sum(e), as half a B fragment of
//            the last product to LDS (two slots, one barrier per block);
//   wave ct  after the barrier, output channel tile ct = h: O = b3 + W3^T u (its W3^T
//            fragments in registers too), 4 consecutive channels per lane.
// k_deslice_sf gives a wave 32 points and all heads and stages 128 KB of operands in LDS
// first: 256 points and 14 us are its least step.  Here a block is 32 points and nothing
// is staged, but a block is a chain across the barrier.  Launches in a row in a graph,
// k_deslice_sf and this, in us:
//   (C, M)     5,003 points   16,384        24,576         32,768         65,536 points
//   (128, 64)  13.5 and 6.7   13.9 and 9.2  14.2 and 11.5  14.6 and 13.7  17.4 and 22.6
//   (128, 32)  10.7 and 5.8   11.0 and 8.1  11.3 and 10.3  11.7 and 12.5  13.3 and 21.2
//   (64, 32)    5.4 and 3.0    5.5 and 3.8   5.7 and 4.5    5.9 and 5.2    6.5 and 8.0
// Three blocks per workgroup (24,576 points on 256 compute units) are the last count at
// which this is the faster one for every shape.  Called one by one, no call takes less
// than the host's 7.6 to 8.4 us.
//
// Blocks with an exp2 sum outside the window are noted in LDS by any of the waves and
// redone at the end, as there.
#pragma once
#include "ts3_pass2sf.h"

namespace ts3 {

constexpr int SH_MAX_ITERS = 3;  // blocks per workgroup, see above (at most the bits of `failed`)

// Operands as for k_deslice_sf.  Grid: at most ceil(n / 32) workgroups of 64 H threads,
// each with at most SH_MAX_ITERS blocks.
template <int C, int M>
__global__ __launch_bounds__(4 * C, 1) void k_deslice_sh(const bf16_t *__restrict__ x, int64_t n,
                                                         const bf16_t *__restrict__ w2p, const float *__restrict__ b2s,
                                                         const bf16_t *__restrict__ sf, const bf16_t *__restrict__ w3f,
                                                         const float *__restrict__ b3, bf16_t *__restrict__ out) {
    using Cfg = Pass2SFCfg<C, M>;
    using T = bf16_t;
    constexpr int CT = Cfg::CT, MT = Cfg::MT, CK = Cfg::CK, KM = Cfg::KM, PT = Cfg::PT, PTS = 16 * PT;
    static_assert(Cfg::H == CT, "a head and an output channel tile per wave");
    __shared__ __attribute__((aligned(1024))) unsigned char us[2][CK * PT * 1024];
    __shared__ uint32_t failed;  // bit i: block i left the fast path

    const int lane = threadIdx.x & 63;
    const int h = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int li = lane & 15, g = lane >> 4;
    const int64_t nblk = (n + PTS - 1) / PTS;
    if (n <= 0 || (int64_t)blockIdx.x >= nblk) return;                 // uniform over the workgroup
    const int iters = (int)((nblk - 1 - blockIdx.x) / gridDim.x + 1);  // <= SH_MAX_ITERS (host)
    const int64_t pw = (int64_t)blockIdx.x * PTS, bstride = (int64_t)gridDim.x * PTS;
    if (threadIdx.x == 0) failed = 0;

    // rows past the end repeat the last one, as do a block's loads past the last block
    auto load_x = [&](int64_t p0, Frag<T> (&xf)[PT][CK]) {
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) {
            const int64_t p = p0 + pt * 16 + li, pc = p < n ? p : n - 1;
#pragma unroll
            for (int kc = 0; kc < CK; ++kc) load8(xf[pt][kc], x + (size_t)pc * C + kc * 32 + g * 8);
        }
    };
    Frag<T> xb[PT][CK], w2[MT][CK], sa[KM], w3[CK];
    load_x(pw, xb);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int kc = 0; kc < CK; ++kc) load8(w2[mt][kc], w2p + ((((size_t)h * MT + mt) * CK + kc) * 64 + lane) * 8);
    f32x4 bias[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const float4 b = *reinterpret_cast<const float4 *>(b2s + h * M + mt * 16 + g * 4);
        bias[mt] = f32x4{b.x, b.y, b.z, b.w};
    }
#pragma unroll
    for (int km = 0; km < KM; ++km) load8(sa[km], sf + (((size_t)h * KM + km) * 64 + lane) * 8);
#pragma unroll
    for (int kk = 0; kk < CK; ++kk) load8(w3[kk], w3f + (((size_t)kk * CT + h) * 64 + lane) * 8);
    const int c0 = 32 * (h >> 1) + 8 * g + 4 * (h & 1);  // zchan(h, 4g): the lane's four output channels
    const float4 b3v = *reinterpret_cast<const float4 *>(b3 + c0);
    Frag<T> ones;
    ones8(ones);
    __syncthreads();  // `failed` is clear

    for (int i = 0; i < iters; ++i) {
        const int64_t p0 = pw + (int64_t)i * bstride;
        f32x4 L[MT][PT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) L[mt][pt] = bias[mt];
#pragma unroll
        for (int kc = 0; kc < CK; ++kc)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int pt = 0; pt < PT; ++pt) mma(L[mt][pt], w2[mt][kc], xb[pt][kc]);
        load_x(p0 + bstride, xb);
        bool ok = true;
        unsigned char *const slot = us[i & 1];
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) L[mt][pt][r] = fast_exp2(L[mt][pt][r]);
            Frag<T> wf[PT][KM];
            pack_weights<T, MT, PT, KM>(L, pt, 1.0f, wf);
            f32x4 U{0.f, 0.f, 0.f, 0.f}, S{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int km = 0; km < KM; ++km) {
                mma(U, sa[km], wf[pt][km]);
                mma(S, ones, wf[pt][km]);
            }
            ok = ok && softmax_sum_ok(S[0]);
            const float inv = fast_rcp(S[0]);
#pragma unroll
            for (int r = 0; r < 4; ++r) U[r] *= inv;
            Frag<T> u;
            u.set2(0, U[0], U[1]);
            u.set2(2, U[2], U[3]);
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
            *reinterpret_cast<bf16x4 *>(slot + ((h >> 1) * PT + pt) * 1024 + lane * 16 + (h & 1) * 8) =
                bf16x4{u.v[0], u.v[1], u.v[2], u.v[3]};
        }
        if (__any(!ok) && lane == 0) atomicOr(&failed, 1u << i);
        // The slot is written again two blocks on, past the next barrier, which no wave
        // passes before every wave has read it.
        __syncthreads();
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) {
            f32x4 O{b3v.x, b3v.y, b3v.z, b3v.w};
#pragma unroll
            for (int kk = 0; kk < CK; ++kk) {
                Frag<T> u;
                u.v = *reinterpret_cast<const bf16x8 *>(slot + (kk * PT + pt) * 1024 + lane * 16);
                mma(O, w3[kk], u);
            }
            const int64_t p = p0 + pt * 16 + li;
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
            *reinterpret_cast<bf16x4 *>(out + (size_t)(p < n ? p : n - 1) * C + c0) =
                bf16x4{(__bf16)O[0], (__bf16)O[1], (__bf16)O[2], (__bf16)O[3]};
        }
    }
    wait_vmcnt<0>();  // the rows of a failed block are written before they are written again
    __syncthreads();
    if (h < PT)
        for (uint32_t f = failed; f; f &= f - 1)
            deslice_tile_global_sf<C, M>(x, n, pw + (int64_t)__builtin_ctz(f) * bstride + 16 * h, w2p, b2s, sf, w3f, b3, out,
                                         lane);
}

}  // namespace ts3
