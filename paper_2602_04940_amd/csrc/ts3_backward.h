// Backward of the Physics-Attention layer for float32 storage, with the slice
// weights recomputed tile by tile instead of stored: the paper trains with
// every tile's slice computation checkpointed (section 3.2, "Geometry slice
// tiling", and the Checkpoint steps of Algorithm 1).  Given the output
// gradient g = dL/dx_out:
//
//   k_sum3      per (part, head): recompute w; partial dZ[m][:] =
//               sum_p w[p][m] g_p (and sum_p w in column C)
//   k_bw_token  per head: back through Linear3, the attention among the
//               head's M tokens, Linear1 and the normalisation: ds_raw, dd
//               and the token-side weight gradients
//   k_bw_dx3    per block of points, over all heads: recompute
//               w; dw = g.Z + x.ds_raw + dd; dz = (1/tau) w (dw - sum_m w dw);
//               dx = sum_h dz W2_h^T + w ds_raw_h; dz is stored
//   k_sum3      per (part, head): partial dW2^T[m][:] = sum_p dz[p][m] x_p
//               and db2 = sum_p dz, from the stored dz
//
// Part sums are folded in index order by the forward's fold kernels, so
// every gradient is a fixed function of the inputs (any tiling, any run).
// This file holds the token side and the softmax that the float32 passes share.
#pragma once
#include "ts3_device.h"

namespace ts3 {

// Max-shifted softmax over a head's M slices of one 16-point tile, in place
// (E holds exp2-scaled logits), times `scale` (0 for a point past the end).
template <int MT>
__device__ __forceinline__ void softmax_tile(f32x4 (&E)[MT], float scale) {
    float mx = E[0][0];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, E[mt][r]);
    mx = xrow_max(mx);
    float sum = 0.f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float e = fast_exp2(E[mt][r] - mx);
            E[mt][r] = e;
            sum += e;
        }
    const float tot = xrow_sum(sum);  // every lane takes part in the cross-row swaps
    const float inv = scale / tot;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) E[mt][r] *= inv;
}

// Token side of the backward, one workgroup per head (1,024 threads; a row's softmax and
// sums on 16 lanes; 211 us at C = 128, M = 64 with 256 threads and a row per thread):
//   Z[h] = s1[h] W3_h            -> ds1, dW3_h
//   s1 = softmax(q k^T / sqrt(dh)) v, q,k,v = s Wq,Wk,Wv  -> ds, dWq, dWk, dWv
//   s = mean W1_h + b1_h          -> dmean, dW1_h, db1_h
//   mean = s_raw / (d + eps) (0 where d + eps <= 0) -> ds_raw, dd
// and db3 = sum_m dZ[0][m] (every head's weights sum to one per point).
// Dynamic LDS: floats mean, dZ [M][C] and s, s1, q, k, v, ds1, dq, dk, dv, ds
// [M][dh] and P, dP [M][M]; STAGED also W3_h and then W1_h^T [dh][C], with a float of
// padding per row of those, dZ, k and v.  Bound by LDS and by the lines that a load
// touches: where lanes run over the rows of W3_h or W1_h each load from memory takes one
// line per lane, and where they run over k's rows sixteen share a bank.  131 us at C =
// 128, M = 64 from memory and without padding, 49 us staged; the other form serves the
// shape whose LDS that would exceed (one head of width 128).
constexpr int BW_TOKEN_THREADS = 1024;
inline size_t bw_token_lds(int C, int M, int dh, bool staged) {
    return (size_t)(2 * M * C + 10 * M * dh + 2 * M * M + (staged ? dh * (C + 1) + 3 * M : 0)) * 4;
}
template <bool STAGED>
__global__ __launch_bounds__(BW_TOKEN_THREADS, 1) void k_bw_token(
    const float *__restrict__ s_raw, const float *__restrict__ dsum, const float *__restrict__ s,
    const float *__restrict__ s1, const float *__restrict__ dZ, const float *__restrict__ W1,
    const float *__restrict__ Wq, const float *__restrict__ Wk, const float *__restrict__ Wv,
    const float *__restrict__ W3, int C, int H, int M, int dh, float eps, float *__restrict__ dsr,
    float *__restrict__ dd, float *__restrict__ dW1, float *__restrict__ db1,
    float *__restrict__ dWq, float *__restrict__ dWk, float *__restrict__ dWv, float *__restrict__ dW3,
    float *__restrict__ db3) {
    extern __shared__ float sm[];
    const int h = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int HD = H * dh;
    const int gp = STAGED ? C + 1 : C, kp = STAGED ? dh + 1 : dh;  // row strides of gz (and wl), k and v
    float *mean = sm, *gz = mean + M * C;
    float *ss = gz + M * gp, *s1s = ss + M * dh, *q = s1s + M * dh, *k = q + M * dh, *v = k + M * kp;
    float *ds1 = v + M * kp, *dq = ds1 + M * dh, *dk = dq + M * dh, *dv = dk + M * dh, *ds = dv + M * dh;
    float *P = ds + M * dh, *dP = P + M * M, *wl = dP + M * M;
    const float scale = 1.f / sqrtf((float)dh);
    for (int i = tid; i < M * C; i += nt) {
        const int m = i / C;
        const float den = dsum[h * M + m] + eps;
        mean[i] = den > 0.f ? s_raw[(size_t)h * M * C + i] / den : 0.f;
        gz[m * gp + (i - m * C)] = dZ[(size_t)h * M * C + i];
    }
    for (int i = tid; i < M * dh; i += nt) {
        ss[i] = s[(size_t)h * M * dh + i];
        s1s[i] = s1[(size_t)h * M * dh + i];
    }
    if constexpr (STAGED)
        for (int i = tid; i < dh * C; i += nt) wl[i / C * gp + i % C] = W3[(size_t)h * dh * C + i];
    __syncthreads();
    // ds1 = dZ W3_h^T; dW3_h = s1^T dZ; q, k, v
    for (int i = tid; i < M * dh; i += nt) {
        const int m = i / dh, j = i % dh;
        float a = 0.f, aq = 0.f, ak = 0.f, av = 0.f;
#pragma unroll 8
        for (int c = 0; c < C; ++c) a += gz[m * gp + c] * (STAGED ? wl[j * gp + c] : W3[(size_t)(h * dh + j) * C + c]);
#pragma unroll 8
        for (int t = 0; t < dh; ++t) {
            const float sv = ss[m * dh + t];
            aq += sv * Wq[((size_t)h * dh + t) * dh + j];
            ak += sv * Wk[((size_t)h * dh + t) * dh + j];
            av += sv * Wv[((size_t)h * dh + t) * dh + j];
        }
        ds1[i] = a;
        q[i] = aq;
        k[m * kp + j] = ak;
        v[m * kp + j] = av;
    }
    for (int i = tid; i < dh * C; i += nt) {
        const int j = i / C, c = i % C;
        float a = 0.f;
#pragma unroll 8
        for (int m = 0; m < M; ++m) a += s1s[m * dh + j] * gz[m * gp + c];
        dW3[(size_t)(h * dh + j) * C + c] = a;
    }
    if (h == 0)
        for (int c = tid; c < C; c += nt) {
            float a = 0.f;
#pragma unroll 8
            for (int m = 0; m < M; ++m) a += gz[m * gp + c];
            db3[c] = a;
        }
    __syncthreads();
    if constexpr (STAGED)  // W3_h is no longer read
        for (int i = tid; i < dh * C; i += nt) wl[i % dh * gp + i / dh] = W1[(size_t)(i / dh) * HD + h * dh + i % dh];
    // P = softmax_rows(q k^T * scale); dP = ds1 v^T
    for (int i = tid; i < M * M; i += nt) {
        const int a_ = i / M, b_ = i % M;
        float dot = 0.f, dpv = 0.f;
#pragma unroll 8
        for (int j = 0; j < dh; ++j) {
            dot += q[a_ * dh + j] * k[b_ * kp + j];
            dpv += ds1[a_ * dh + j] * v[b_ * kp + j];
        }
        P[i] = dot * scale;
        dP[i] = dpv;
    }
    __syncthreads();
    // a row on the 16 lanes of one DPP row (M is a multiple of 16)
    for (int a_ = tid >> 4; a_ < M; a_ += nt >> 4) {
        const int l = tid & 15;
        float mx = -INFINITY;
        for (int b_ = l; b_ < M; b_ += 16) mx = fmaxf(mx, P[a_ * M + b_]);
        mx = row16_max(mx);
        float sum = 0.f;
        for (int b_ = l; b_ < M; b_ += 16) {
            const float e = expf(P[a_ * M + b_] - mx);
            P[a_ * M + b_] = e;
            sum += e;
        }
        const float inv = 1.f / row16_sum(sum);
        float dot = 0.f;
        for (int b_ = l; b_ < M; b_ += 16) {
            P[a_ * M + b_] *= inv;
            dot += dP[a_ * M + b_] * P[a_ * M + b_];
        }
        dot = row16_sum(dot);
        // dP becomes da = P (dP - rowsum(dP P))
        for (int b_ = l; b_ < M; b_ += 16) dP[a_ * M + b_] = P[a_ * M + b_] * (dP[a_ * M + b_] - dot);
    }
    __syncthreads();
    // dv = P^T ds1; dq = da k * scale; dk = da^T q * scale
    for (int i = tid; i < M * dh; i += nt) {
        const int m = i / dh, j = i % dh;
        float av = 0.f, aq = 0.f, ak = 0.f;
#pragma unroll 8
        for (int t = 0; t < M; ++t) {
            av += P[t * M + m] * ds1[t * dh + j];
            aq += dP[m * M + t] * k[t * kp + j];
            ak += dP[t * M + m] * q[t * dh + j];
        }
        dv[i] = av;
        dq[i] = aq * scale;
        dk[i] = ak * scale;
    }
    __syncthreads();
    // dWq/dWk/dWv = s^T (dq, dk, dv); ds = dq Wq^T + dk Wk^T + dv Wv^T
    for (int i = tid; i < dh * dh; i += nt) {
        const int t = i / dh, j = i % dh;
        float aq = 0.f, ak = 0.f, av = 0.f;
#pragma unroll 8
        for (int m = 0; m < M; ++m) {
            const float sv = ss[m * dh + t];
            aq += sv * dq[m * dh + j];
            ak += sv * dk[m * dh + j];
            av += sv * dv[m * dh + j];
        }
        dWq[(size_t)h * dh * dh + i] = aq;
        dWk[(size_t)h * dh * dh + i] = ak;
        dWv[(size_t)h * dh * dh + i] = av;
    }
    for (int i = tid; i < M * dh; i += nt) {
        const int m = i / dh, t = i % dh;
        float a = 0.f;
#pragma unroll 8
        for (int j = 0; j < dh; ++j)
            a += dq[m * dh + j] * Wq[((size_t)h * dh + t) * dh + j] + dk[m * dh + j] * Wk[((size_t)h * dh + t) * dh + j] +
                 dv[m * dh + j] * Wv[((size_t)h * dh + t) * dh + j];
        ds[i] = a;
    }
    __syncthreads();
    // dW1_h = mean^T ds; db1_h = sum_m ds
    for (int i = tid; i < C * dh; i += nt) {
        const int c = i / dh, j = i % dh;
        float a = 0.f;
#pragma unroll 8
        for (int m = 0; m < M; ++m) a += mean[m * C + c] * ds[m * dh + j];
        dW1[(size_t)c * HD + h * dh + j] = a;
    }
    for (int j = tid; j < dh; j += nt) {
        float a = 0.f;
#pragma unroll 8
        for (int m = 0; m < M; ++m) a += ds[m * dh + j];
        db1[h * dh + j] = a;
    }
    // dmean = ds W1_h^T (kept in gz); ds_raw = dmean / den; dd = -sum_c dmean mean / den
    for (int i = tid; i < M * C; i += nt) {
        const int m = i / C, c = i % C;
        float a = 0.f;
#pragma unroll 8
        for (int j = 0; j < dh; ++j) a += ds[m * dh + j] * (STAGED ? wl[j * gp + c] : W1[(size_t)c * HD + h * dh + j]);
        const float den = dsum[h * M + m] + eps;
        const float r = den > 0.f ? a / den : 0.f;
        gz[m * gp + c] = a;
        dsr[(size_t)h * M * C + i] = r;
    }
    __syncthreads();
    for (int m = tid >> 4; m < M; m += nt >> 4) {
        const float den = dsum[h * M + m] + eps;
        float a = 0.f;
        for (int c = tid & 15; c < C; c += 16) a += gz[m * gp + c] * mean[m * C + c];
        a = row16_sum(a);
        if ((tid & 15) == 0) dd[h * M + m] = den > 0.f ? -a / den : 0.f;
    }
}

// dW2[c][h*M + m] = dW2T[h][m][c].
__global__ void k_bw_transpose_w2(const float *__restrict__ dW2T, int C, int HM, float *__restrict__ dW2) {
    const int64_t total = (int64_t)C * HM;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = i / HM, hm = i % HM;
        dW2[i] = dW2T[hm * C + c];
    }
}

}  // namespace ts3
