// Small kernels of the layer: operand preparation and the ordered fold of span
// partials.  These touch O(H*M*C) data and run in microseconds.
#pragma once
#include "ts3_device.h"

namespace ts3 {

__device__ __forceinline__ void store_elem(bf16_t *p, float v) {
    *reinterpret_cast<__bf16 *>(p) = (__bf16)v;
}

// W2' = W2 * scale in MFMA fragment order [H][MT][CK][64][8]: lane l, slot t
// holds W2'[32*kc + 8*(l>>4) + t][h*M + 16*mt + (l&15)].  b2s = b2 * scale.
// scale = log2(e) / tau, so the softmax can use exp2.  With w1p, also W1 in the
// projected pass 1's operand order (head width 16), as two bfloat16 parts whose
// sum is W1 to about 2^-17 relative: w1p[0][H][CK][64][8] the rounded values,
// w1p[1][...] the rounded remainders; lane l, slot t holds
// W1[32*kc + 8*(l>>4) + t][h*16 + (l&15)].
template <typename T>
__global__ void k_prep_w2(const float *__restrict__ W2, const float *__restrict__ b2, float scale,
                          int C, int H, int M, T *__restrict__ w2p, float *__restrict__ b2s,
                          const float *__restrict__ W1, bf16_t *__restrict__ w1p) {
    const int MT = M / 16, CK = C / 32, HM = H * M;
    const int64_t total = (int64_t)H * MT * CK * 64 * 8;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int t = (int)(i & 7), lane = (int)((i >> 3) & 63);
        int64_t r = i >> 9;
        const int kc = (int)(r % CK); r /= CK;
        const int mt = (int)(r % MT);
        const int h = (int)(r / MT);
        const int c = kc * 32 + (lane >> 4) * 8 + t;
        const int col = h * M + mt * 16 + (lane & 15);
        store_elem(w2p + i, W2[(int64_t)c * HM + col] * scale);
    }
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (tid < HM) b2s[tid] = (b2 ? b2[tid] : 0.f) * scale;
    const int64_t n1 = w1p ? (int64_t)H * CK * 512 : 0;
    for (int64_t i = tid; i < n1; i += (int64_t)gridDim.x * blockDim.x) {
        const int t = (int)(i & 7), lane = (int)((i >> 3) & 63);
        const int64_t r = i >> 9;
        const int kc = (int)(r % CK), h = (int)(r / CK);
        const float w = W1[(int64_t)(kc * 32 + (lane >> 4) * 8 + t) * C + h * 16 + (lane & 15)];
        const __bf16 hi = (__bf16)w;
        reinterpret_cast<__bf16 *>(w1p)[i] = hi;
        reinterpret_cast<__bf16 *>(w1p)[n1 + i] = (__bf16)(w - (float)hi);
    }
}

// Z in decoding-operand order [H][CT][KM][64][8]: lane l, slot t holds
// Z[h][32*km + 16*(t>>2) + 4*(l>>4) + (t&3)][zchan(ct, l&15)] + b3[c] / H (zero
// past M).  Each head's slice weights sum to one (Eq. (1)), so the H heads of
// the deslice add b3 exactly once per point and pass 2 needs no bias pass.
template <typename T>
__global__ void k_prep_z(const float *__restrict__ Z, const float *__restrict__ b3, int C, int H, int M,
                         T *__restrict__ zp) {
    const int CT = C / 16, KM = M >= 32 ? M / 32 : 1;
    const float bscale = 1.f / (float)H;
    const int64_t total = (int64_t)H * CT * KM * 64 * 8;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int t = (int)(i & 7), lane = (int)((i >> 3) & 63);
        int64_t r = i >> 9;
        const int km = (int)(r % KM); r /= KM;
        const int ct = (int)(r % CT);
        const int h = (int)(r / CT);
        const int m = km * 32 + (t >> 2) * 16 + (lane >> 4) * 4 + (t & 3);
        const int c = zchan(ct, lane & 15);
        store_elem(zp + i, m < M ? Z[((int64_t)h * M + m) * C + c] + b3[c] * bscale : 0.f);
    }
}

// Zero the partials of spans that no tile wrote, so the fold sees zeros there.
__global__ void k_zero(float *__restrict__ p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.f;
}

// Sum of n values at stride E, in order, added to `acc`.
template <typename TS, typename TA>
__device__ __forceinline__ TA ordered_sum(const TS *__restrict__ p, int64_t E, int64_t n, TA acc = 0) {
    int64_t i = 0;
    for (; i + 16 <= n; i += 16) {  // sixteen loads in flight
        TS v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = p[(i + k) * E];
#pragma unroll
        for (int k = 0; k < 16; ++k) acc += (TA)v[k];
    }
    for (; i < n; ++i) acc += (TA)p[i * E];
    return acc;
}

// Ordered fold of span partials (Eq. (4) sum over tiles): element e of
// [H][M][C+1] is summed over spans 0..nspan-1 in two fixed levels (runs of
// FOLD spans, then the runs in order), giving the same bits for any tiling.
constexpr int FOLD = 64;
// T is the fold's accumulator: float, or double (the partials are added in
// float64 and rounded once at the end); runs hold T.
template <typename T>
__global__ void k_fold_runs(const float *__restrict__ partials, int64_t E, int64_t nspan, T *__restrict__ runs) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t run = blockIdx.y;
    if (e >= E) return;
    const int64_t s0 = run * FOLD;
    const int64_t s1 = s0 + FOLD < nspan ? s0 + FOLD : nspan;
    runs[run * E + e] = ordered_sum<float, T>(partials + s0 * E + e, E, s1 - s0);
}

// The same fold taken one tile at a time: the tile's spans [g0, g0 + ns)
// (partials[0 .. ns) of this launch) are added to the runs they fall in.  A
// run starting inside the tile starts from zero, one begun by an earlier tile
// continues from its stored sum; each run is thus the same sequential sum,
// in span order, as k_fold_runs forms, and holds the same bits.
template <typename T>
__global__ void k_fold_runs_tile(const float *__restrict__ partials, int64_t E, int64_t g0, int64_t ns,
                                 T *__restrict__ runs) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t run = g0 / FOLD + blockIdx.y;
    if (e >= E) return;
    const int64_t r0 = run * FOLD;
    const int64_t s0 = r0 > g0 ? r0 : g0;
    const int64_t s1 = r0 + FOLD < g0 + ns ? r0 + FOLD : g0 + ns;
    const T from = s0 == r0 ? (T)0 : runs[run * E + e];
    runs[run * E + e] = ordered_sum<float, T>(partials + (s0 - g0) * E + e, E, s1 - s0, from);
}

template <typename T>
__global__ void k_fold_final(const T *__restrict__ runs, int64_t E, int64_t nrun, int C, float *__restrict__ s_raw,
                             float *__restrict__ dsum) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= E) return;
    const T acc = ordered_sum<T, T>(runs + e, E, nrun);
    const int64_t hm = e / (C + 1);
    const int c = (int)(e - hm * (C + 1));
    if (c < C)
        s_raw[hm * C + c] = (float)acc;
    else
        dsum[hm] = (float)acc;
}

}  // namespace ts3
