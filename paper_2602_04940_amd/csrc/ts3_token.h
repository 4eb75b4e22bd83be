// Slice-domain work of the layer, between the two passes: the last level of the
// ordered fold, Linear1 on the slice means, the attention among each head's M
// tokens and Linear3 (the work that the paper moves off the points, Eq. (3) and
// Table 2).  O(H*M*C) data; what bounds these kernels is latency: chains of
// dependent loads and sums, and the launches themselves.  Two kernels, split over
// the slice rows (which depend on each other only through k and v), with every
// weight element loaded once per workgroup for all its rows.  Before, five
// launches (fold, mean and Linear1 by one wave per token, attention by one
// workgroup per head, and the operand preparations) took 120 us at C = 256, M =
// 64, H = 8; see each kernel for its own time.
#pragma once
#include "ts3_device.h"
#include "ts3_pass2.h"  // zchan
#include "ts3_fp32.h"
#include "ts3_rt.h"
#include "ts3_small.h"

namespace ts3 {

// Element (h, m, c) of the decoding operand [H][CT][KM][64][8] (see k_prep_z).
__device__ __forceinline__ int64_t zp_index(int h, int m, int c, int CT, int KM) {
    const int cc = c & 31, ct = 2 * (c >> 5) + ((cc >> 2) & 1), i = (cc >> 3) * 4 + (cc & 3);
    const int mm = m & 31, t = (mm >> 4) * 4 + (mm & 3), g = (mm & 15) >> 2;
    return ((((int64_t)h * CT + ct) * KM + (m >> 5)) * 64 + g * 16 + i) * 8 + t;
}

constexpr int TOK_ROWS = 2;       // slice rows (h, m) per workgroup of k_slice_tokens
constexpr int TOK_THREADS = 512;
constexpr int TOK_MAX_C = 512;

// The fold's last level and the slice tokens, for TOK_ROWS rows per workgroup
// (grid H*M / TOK_ROWS, 512 threads; M is a multiple of 16, so a workgroup's rows
// are one head's):
//   s_raw, d = sum over `count` terms at stride E, in order (runs of part sums,
//              or the part sums themselves when they make up one run),
//   s[m][j]  = b1 + (s_raw / (d + eps))[m][:] . W1[:, h*dh + j]   (rowc = C), or
//   s[m][j]  = b1 + (t / (d + eps))[m][j]                         (projected).
// The mean is taken before Linear1 (the physical state of Appendix A.4); an empty
// slice (d + eps <= 0) has mean zero.  512 / dh groups of threads take every
// (512/dh)-th channel each and are added in order.  At C = 256, M = 64, H = 8:
// 30 us as one wave per token (a chain of 256 dependent loads and sums, one
// division each).
template <typename TS, typename TA>
__global__ __launch_bounds__(TOK_THREADS) void k_slice_tokens(const TS *__restrict__ src, int64_t E, int64_t count, int rowc,
                                                      bool projected, const float *__restrict__ W1,
                                                      const float *__restrict__ b1, int H, int M, int dh, float eps,
                                                      float *__restrict__ s_raw, float *__restrict__ dsum,
                                                      float *__restrict__ s) {
    __shared__ float raw[TOK_ROWS * (TOK_MAX_C + 1)];
    __shared__ float red[TOK_THREADS * TOK_ROWS];
    const int tid = threadIdx.x;
    const int hm0 = (int)blockIdx.x * TOK_ROWS, h = hm0 / M;
    const int ld = rowc + 1, HD = H * dh;
    for (int e = tid; e < TOK_ROWS * ld; e += TOK_THREADS) {
        const float v = (float)ordered_sum<TS, TA>(src + (int64_t)hm0 * ld + e, E, count);
        raw[e] = v;
        const int r = e / ld, c = e - r * ld;
        if (c < rowc) s_raw[(int64_t)(hm0 + r) * rowc + c] = v;
        else dsum[hm0 + r] = v;
    }
    __syncthreads();
    if (projected) {
        for (int i = tid; i < TOK_ROWS * dh; i += TOK_THREADS) {
            const int r = i / dh, j = i - r * dh;
            const float den = raw[r * ld + rowc] + eps;
            s[(int64_t)(hm0 + r) * dh + j] = (den > 0.f ? raw[r * ld + j] / den : 0.f) + (b1 ? b1[h * dh + j] : 0.f);
        }
        return;
    }
    for (int e = tid; e < TOK_ROWS * rowc; e += TOK_THREADS) {
        const int r = e / rowc, c = e - r * rowc;
        const float den = raw[r * ld + rowc] + eps;
        raw[r * ld + c] = den > 0.f ? raw[r * ld + c] / den : 0.f;
    }
    __syncthreads();
    const int groups = TOK_THREADS / dh, cg = tid / dh, j = tid - cg * dh;  // dh <= 256
    if (cg < groups) {
        float acc[TOK_ROWS];
#pragma unroll
        for (int r = 0; r < TOK_ROWS; ++r) acc[r] = 0.f;
#pragma unroll 8
        for (int c = cg; c < rowc; c += groups) {
            const float w = W1[(int64_t)c * HD + h * dh + j];
#pragma unroll
            for (int r = 0; r < TOK_ROWS; ++r) acc[r] = fmaf(raw[r * ld + c], w, acc[r]);
        }
#pragma unroll
        for (int r = 0; r < TOK_ROWS; ++r) red[(cg * TOK_ROWS + r) * dh + j] = acc[r];
    }
    __syncthreads();
    for (int i = tid; i < TOK_ROWS * dh; i += TOK_THREADS) {
        float acc = b1 ? b1[h * dh + i % dh] : 0.f;
        for (int q = 0; q < groups; ++q) acc += red[q * TOK_ROWS * dh + i];
        s[(int64_t)hm0 * dh + i] = acc;
    }
}

// Where the decoding operands go; what a layer does not use is NULL.
template <typename T> struct AttendOut {
    float *s1, *Z, *b3;
    T *zp;         // fragments [H][CT][KM][64][8], or parts: the runtime-shape layout (rt heads
                   // at a time), or for float32 that of k_deslice3
    int rt;        // 0, or GH of the runtime-shape layout
    bf16_t *sf;    // slice-state pass 2 (dh = 16, M a multiple of 32): s'^T fragments
    bf16_t *w3f;   // and W3^T fragments
};

constexpr int ATT_ROWS = 16;  // token rows per workgroup of k_attend
constexpr int ATT_KV = 8;     // rows of q, k and v that a thread forms at a time

__host__ __device__ __forceinline__ size_t attend_lds_bytes(int M, int dh) {
    const int dp = (dh + 3) & ~3;
    return (size_t)(2 * M * dp + M * (dp + 4) + ATT_ROWS * M + 2 * ATT_ROWS * dp) * 4;
}
__device__ __forceinline__ float dot4(float acc, const float4 &a, const float4 &b) {
    return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, fmaf(a.x, b.x, acc))));
}

// Rows rg, rg + groups, ... (count of them) of in [.][dp] times w [dh][dh], column
// j, for one or two matrices: out[row * ld + j].  Rows of `in` are zero past dh.
template <int NW>
__device__ __forceinline__ void token_rows(const float *in, int rows, int rg, int groups, int dh, int dp, int j,
                                           const float *const (&w)[NW], float *const (&out)[NW], const int (&ld)[NW]) {
    for (int rb = rg; rb < rows; rb += groups * ATT_KV) {
        float acc[NW][ATT_KV];
#pragma unroll
        for (int k = 0; k < NW; ++k)
#pragma unroll
            for (int i = 0; i < ATT_KV; ++i) acc[k][i] = 0.f;
#pragma unroll 4
        for (int u = 0; u < dp; u += 4) {
            float4 wv[NW];
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                const float *p = w[k] + u * dh + j;
                wv[k] = float4{p[0], u + 1 < dh ? p[dh] : 0.f, u + 2 < dh ? p[2 * dh] : 0.f, u + 3 < dh ? p[3 * dh] : 0.f};
            }
#pragma unroll
            for (int i = 0; i < ATT_KV; ++i) {
                const int r = rb + i * groups;
                const float4 x = *reinterpret_cast<const float4 *>(in + (r < rows ? r : 0) * dp + u);
#pragma unroll
                for (int k = 0; k < NW; ++k) acc[k][i] = dot4(acc[k][i], x, wv[k]);
            }
        }
#pragma unroll
        for (int i = 0; i < ATT_KV; ++i) {
            const int r = rb + i * groups;
            if (r < rows)
#pragma unroll
                for (int k = 0; k < NW; ++k) out[k][r * ld[k] + j] = acc[k][i];
        }
    }
}

// Attention among a head's M tokens, Linear3 and the decoding operands, for
// ATT_ROWS token rows per workgroup: q, k, v = s Wq[h], s Wk[h], s Wv[h];
// A = softmax(q k^T / sqrt(dh)); s1 = A v; Z[h][m][c] = s1[m][:] .
// W3[h*dh .. h*dh+dh-1][c], stored with b3 / H as the decoding operand (k_prep_z
// has its order).  Every workgroup of a head forms all of k and v again, which
// costs M/16 times 2*M*dh*dh products but no second launch.  Grid H * M / 16, then
// `extra` workgroups for W3^T fragments and b3; 256 threads.  Bound by LDS
// instructions: rows are padded to four floats and read as such (36 us at C = 256,
// M = 64, H = 8 with single floats; 110 us as one workgroup per head and 64
// channels, of which most was the softmax of a whole row by one thread).
template <typename T>
__global__ __launch_bounds__(256) void k_attend(const float *__restrict__ s, const float *__restrict__ Wq,
                                                const float *__restrict__ Wk, const float *__restrict__ Wv,
                                                const float *__restrict__ W3, const float *__restrict__ b3, int C,
                                                int H, int M, int dh, int extra, AttendOut<T> out) {
    extern __shared__ __attribute__((aligned(16))) float sm[];
    const int tid = threadIdx.x;
    const int tiles = M / ATT_ROWS, main = H * tiles;
    if ((int)blockIdx.x >= main) {
        const int part = (int)blockIdx.x - main;
        if (out.w3f) {
            const int CT = C / 16;
            const int total = C * C;  // C <= 512
            for (int i = part * 256 + tid; i < total; i += extra * 256) {
                const int t = i & 7, lane = (i >> 3) & 63, r = i >> 9;
                const int ct = r % CT, kk = r / CT;
                const int k = 16 * (2 * kk + (t >> 2)) + 4 * (lane >> 4) + (t & 3);
                store_elem(out.w3f + i, W3[(int64_t)k * C + zchan(ct, lane & 15)]);
            }
        }
        if (out.rt) rt_zero_pad((bf16_t *)out.zp, C, H, M, RtGroup(out.rt, M), RT_NP<T>, tid + part * 256, extra * 256);
        if (part == 0)
            for (int c = tid; c < C; c += 256) out.b3[c] = b3 ? b3[c] : 0.f;
        return;
    }
    const int h = (int)blockIdx.x / tiles, m0 = ((int)blockIdx.x - h * tiles) * ATT_ROWS;
    const int dp = (dh + 3) & ~3, kld = dp + 4;
    float *ss = sm;                // [M][dp]
    float *k = ss + M * dp;        // [M][dp + 4]: the rows' lanes fall on different banks
    float *v = k + M * kld;        // [M][dp]
    float *q = v + M * dp;         // [16][dp]
    float *A = q + ATT_ROWS * dp;  // [16][M]
    float *o = A + ATT_ROWS * M;   // [16][dp]
    for (int i = tid; i < M * dp; i += 256) {
        const int m = i / dp, u = i - m * dp;
        ss[i] = u < dh ? s[((int64_t)h * M + m) * dh + u] : 0.f;
    }
    if (dp != dh)  // columns past dh of q, k and v are read as part of four floats
        for (int i = tid; i < M * (dp - dh); i += 256) {
            const int m = i / (dp - dh), u = dh + i - m * (dp - dh);
            k[m * kld + u] = 0.f;
            v[m * dp + u] = 0.f;
            if (m < ATT_ROWS) q[m * dp + u] = o[m * dp + u] = 0.f;
        }
    __syncthreads();
    const int64_t wh = (int64_t)h * dh * dh;
    const int groups = 256 / dh, rg = tid / dh, j = tid - rg * dh;
    if (rg < groups) {
        token_rows<2>(ss, M, rg, groups, dh, dp, j, {Wk + wh, Wv + wh}, {k, v}, {kld, dp});
        token_rows<1>(ss + m0 * dp, ATT_ROWS, rg, groups, dh, dp, j, {Wq + wh}, {q}, {dp});
    }
    __syncthreads();
    // Row r's scores and softmax on the 16 lanes of one DPP row.
    const int r = tid >> 4, l = tid & 15;
    {
        const float scale = 1.0f / sqrtf((float)dh);
        float mx = -INFINITY;
        for (int b = l; b < M; b += 16) {
            float acc = 0.f;
#pragma unroll 4
            for (int u = 0; u < dp; u += 4)
                acc = dot4(acc, *reinterpret_cast<const float4 *>(q + r * dp + u),
                           *reinterpret_cast<const float4 *>(k + b * kld + u));
            acc *= scale;
            A[r * M + b] = acc;
            mx = fmaxf(mx, acc);
        }
        mx = row16_max(mx);
        float sum = 0.f;
        for (int b = l; b < M; b += 16) {
            const float e = expf(A[r * M + b] - mx);
            A[r * M + b] = e;
            sum += e;
        }
        sum = row16_sum(sum);
        for (int b = l; b < M; b += 16) A[r * M + b] /= sum;
    }
    __syncthreads();
    for (int j4 = 4 * l; j4 < dp; j4 += 64) {
        float4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int b = 0; b < M; b += 4) {
            const float4 a = *reinterpret_cast<const float4 *>(A + r * M + b);
            const float aw[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 x = *reinterpret_cast<const float4 *>(v + (b + i) * dp + j4);
                acc.x = fmaf(aw[i], x.x, acc.x);
                acc.y = fmaf(aw[i], x.y, acc.y);
                acc.z = fmaf(aw[i], x.z, acc.z);
                acc.w = fmaf(aw[i], x.w, acc.w);
            }
        }
        *reinterpret_cast<float4 *>(o + r * dp + j4) = acc;
        const float av[4] = {acc.x, acc.y, acc.z, acc.w};
        const int m = m0 + r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int jj = j4 + i;
            if (jj >= dh) break;
            out.s1[((int64_t)h * M + m) * dh + jj] = av[i];
            if (out.sf) {
                const int mm = m & 31, t = (mm >> 4) * 4 + (mm & 3), lane = ((mm & 15) >> 2) * 16 + jj;
                store_elem(out.sf + (((int64_t)h * (M / 32) + (m >> 5)) * 64 + lane) * 8 + t, av[i]);
            }
        }
    }
    __syncthreads();
    const int CT = C / 16, KM = M >= 32 ? M / 32 : 1;
    const float bscale = 1.f / (float)H;
    for (int c = tid; c < C; c += 256) {
        float acc[ATT_ROWS];
#pragma unroll
        for (int i = 0; i < ATT_ROWS; ++i) acc[i] = 0.f;
        const float *w3 = W3 + (int64_t)h * dh * C + c;
#pragma unroll 4
        for (int u = 0; u < dp; u += 4) {
            const float *p = w3 + (int64_t)u * C;
            const float4 w{p[0], u + 1 < dh ? p[C] : 0.f, u + 2 < dh ? p[2 * C] : 0.f, u + 3 < dh ? p[3 * C] : 0.f};
#pragma unroll
            for (int i = 0; i < ATT_ROWS; ++i) acc[i] = dot4(acc[i], *reinterpret_cast<const float4 *>(o + i * dp + u), w);
        }
        const float bb = b3 ? b3[c] * bscale : 0.f;
#pragma unroll
        for (int i = 0; i < ATT_ROWS; ++i) {
            const int m = m0 + i;
            out.Z[((int64_t)h * M + m) * C + c] = acc[i];
            if (out.rt) {
                store_parts((bf16_t *)out.zp, rt_z_index(h, m, c, CT, M, RtGroup(out.rt, M), RT_NP<T>), acc[i] + bb,
                            RT_NP<T>);
            } else if constexpr (sizeof(T) == 4) {
                const int64_t at = z3_index(h, m, c, CT, KM);
                store_parts((bf16_t *)out.zp, at, acc[i] + bb, 3);
                if (M == 16) store_parts((bf16_t *)out.zp, at + 4, 0.f, 3);  // slots 4..7: past M
            } else {
                const int64_t at = zp_index(h, m, c, CT, KM);
                store_elem(out.zp + at, acc[i] + bb);
                if (M == 16) store_elem(out.zp + at + 4, 0.f);  // slots 4..7: past M
            }
        }
    }
}

}  // namespace ts3
