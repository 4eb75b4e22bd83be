// Runtime-shape kernels: the layer for any C and M that are multiples of 16
// (C <= 512, M <= 256) without a tuned kernel.  The same computation as the tuned
// passes (paper Eq. (1), Eq. (4) and Eq. (5), Algorithm 1), with the same span
// partials and ordered fold, so results are tiling-independent in the same way.
//
// All products run on bf16 matrix cores with float32 accumulation.  What is held
// in float32 (x, W2', Z of float32 storage, and the slice weights of either
// storage) enters as three bfloat16 parts (Parts), so no operand is rounded.  As
// plain vector arithmetic these kernels took 12.8 + 2.2 ms for 30,000 float32
// points at (C, H, M) = (256, 8, 64), bound by one LDS read per product, the layer now
// 0.36 ms; 50,021 bf16 points at (192, 4, 48): 20.2 ms, now 0.15 ms.
//
// Operand layouts (16-bit parts, NP = 3 for float32 storage, 1 for bf16; written by
// k_prep_w2_rt, k_prep_z_rt and k_attend, zero past C and past the last slice):
//   w2r [H][MT][CK][NP][64][8]: lane l, slot t holds
//       W2[32*kc + 8*(l>>4) + t][h*M + 16*mt + (l&15)] * log2(e) / tau
//   zr  [ceil(H/GH)][CT][KG][NP][64][8], groups of GH heads whose slices follow one
//       another (k = (h % GH) * M + m, KG = ceil(GH*M / 32)): lane l, slot t holds
//       Z[h][m][16*ct + (l&15)] + b3 / H for k = 32*km + 8*(l>>4) + t
#pragma once
#include "ts3_pass1.h"  // lds_s16x4
#include "ts3_small.h"  // store_elem

namespace ts3 {

constexpr int RT_MAX_C = 512, RT_MAX_M = 256;
constexpr int RT_LDS_MAX = 160 * 1024;
template <typename T> constexpr int RT_NP = sizeof(T) == 4 ? 3 : 1;

__host__ __device__ __forceinline__ int rt_ck(int C) { return (C + 31) / 32; }

// How pass 2 covers a shape: blocks of 16 * PT points, GH heads at a time.
struct RtGroup {
    int GH, KG;
    __host__ __device__ __forceinline__ RtGroup(int gh, int M) : GH(gh), KG((gh * M + 31) / 32) {}
};
__device__ __forceinline__ int64_t rt_z_index(int h, int m, int c, int CT, int M, const RtGroup &gr, int NP) {
    const int k = (h % gr.GH) * M + m;
    return (((((int64_t)(h / gr.GH) * CT + (c >> 4)) * gr.KG + (k >> 5)) * NP) * 64 + ((k & 31) >> 3) * 16 + (c & 15)) * 8 +
           (k & 7);
}
// Element `at` of a one- or three-part operand (parts are 512 elements apart).
__device__ __forceinline__ void store_parts(bf16_t *p, int64_t at, float v, int NP) {
    __bf16 *q = reinterpret_cast<__bf16 *>(p) + at;
    const __bf16 h = (__bf16)v;
    q[0] = h;
    if (NP == 3) {
        const float r = v - (float)h;
        const __bf16 m = (__bf16)r;
        q[512] = m;
        q[1024] = (__bf16)(r - (float)m);
    }
}
// Element i of the padding of zr: every slot that holds no slice.
__device__ __forceinline__ int rt_z_pad(int H, int M, int group, const RtGroup &gr) {
    const int heads = H - group * gr.GH < gr.GH ? H - group * gr.GH : gr.GH;
    return gr.KG * 32 - heads * M;
}
__device__ __forceinline__ void rt_zero_pad(bf16_t *zr, int C, int H, int M, const RtGroup &gr, int NP, int64_t first,
                                            int64_t step) {
    const int CT = C / 16;
    for (int group = 0; group * gr.GH < H; ++group) {
        const int pad = rt_z_pad(H, M, group, gr);
        for (int64_t i = first; i < (int64_t)pad * C; i += step) {
            const int c = (int)(i % C), k = gr.KG * 32 - pad + (int)(i / C);
            const int64_t at = (((((int64_t)group * CT + (c >> 4)) * gr.KG + (k >> 5)) * NP) * 64 + ((k & 31) >> 3) * 16 +
                                (c & 15)) * 8 + (k & 7);
            store_parts(zr, at, 0.f, NP);
        }
    }
}

__global__ void k_prep_w2_rt(const float *__restrict__ W2, const float *__restrict__ b2, float scale, int C, int H,
                             int M, int NP, bf16_t *__restrict__ w2r, float *__restrict__ b2s) {
    const int HM = H * M, CK = rt_ck(C);
    const int64_t total = (int64_t)HM * CK * 32;
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t i = tid; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int t = (int)(i & 7), lane = (int)((i >> 3) & 63);
        const int64_t r = i >> 9;
        const int kc = (int)(r % CK), c = kc * 32 + (lane >> 4) * 8 + t;
        const int64_t hm = r / CK * 16 + (lane & 15);  // (h * MT + mt) * 16 + row
        store_parts(w2r, (r * NP * 64 + lane) * 8 + t, c < C ? W2[(int64_t)c * HM + hm] * scale : 0.f, NP);
    }
    if (tid < HM) b2s[tid] = (b2 ? b2[tid] : 0.f) * scale;
}

__global__ void k_prep_z_rt(const float *__restrict__ Z, const float *__restrict__ b3, int C, int H, int M, RtGroup gr,
                            int NP, bf16_t *__restrict__ zr) {
    const float bscale = 1.f / (float)H;
    const int64_t total = (int64_t)H * M * C, tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = tid; i < total; i += step) {
        const int c = (int)(i % C);
        const int64_t hm = i / C;
        store_parts(zr, rt_z_index((int)(hm / M), (int)(hm % M), c, C / 16, M, gr, NP), Z[i] + b3[c] * bscale, NP);
    }
    rt_zero_pad(zr, C, H, M, gr, NP, tid, step);
}

// acc[i] += A[i] . B over one K32 step for N row tiles that share B; the part
// products run outermost, so consecutive MFMAs are independent.
template <int N, int NA, int NB>
__device__ __forceinline__ void mma_parts(f32x4 *acc, const Parts<NA> (&a)[N], const Parts<NB> &b) {
    using PP = PartProducts<NA, NB>;
#pragma unroll
    for (int q = 0; q < PP::N; ++q)
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = mma_bf16(a[i].p[PP::I[q]], b.p[PP::J[q]], acc[i]);
}

// The same for a long sum over points: the step's products are summed from zero and
// then added to acc on the vector unit, or, where the step's A operand is negated,
// subtracted.  A bf16 MFMA drops the low bits of its terms that lie below its largest
// one, and it rounds down (measured: a sum that starts from the accumulator lost
// 2.6e-5 of the float32 weight gradients of 2M points, one that starts from zero
// 7.4e-6, against 1.1e-6 with float32 MFMAs): from zero fewer bits are dropped, and
// negating every other step's A turns the bias of those over.
template <int N, int NA, int NB>
__device__ __forceinline__ void mma_parts_add(f32x4 *acc, const Parts<NA> (&a)[N], const Parts<NB> &b, bool negated) {
    f32x4 t[N];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    mma_parts<N, NA, NB>(t, a, b);
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = negated ? acc[i] - t[i] : acc[i] + t[i];
}

// Eight storage elements of a point row as operand parts (zero past the row).
__device__ __forceinline__ void rt_load8(float (&v)[8], const float *p, bool ok) {
    const float4 a = ok ? reinterpret_cast<const float4 *>(p)[0] : float4{0.f, 0.f, 0.f, 0.f};
    const float4 b = ok ? reinterpret_cast<const float4 *>(p)[1] : float4{0.f, 0.f, 0.f, 0.f};
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <typename T> struct RtRow;
template <> struct RtRow<float> {
    float v[8];
    __device__ __forceinline__ void load(const float *p, bool ok) { rt_load8(v, p, ok); }
    __device__ __forceinline__ void parts(Parts<3> &f) const { split8(v, f); }
};
template <> struct RtRow<bf16_t> {
    bf16x8 v;
    __device__ __forceinline__ void load(const bf16_t *p, bool ok) {
        v = ok ? *reinterpret_cast<const bf16x8 *>(p) : bf16x8{};
    }
    __device__ __forceinline__ void parts(Parts<1> &f) const { f.p[0] = v; }
};

// Max-shifted softmax over a head's MT <= MTMAX slice tiles of 16 points (lane (g,
// li): slices 16mt + 4g + r of point li), then the weights' three parts, four
// slices (8 bytes) per tile and part, to ws + part * plane + 32 * mt, times `scale`
// (0 for a point past the end, -1 to negate).
template <int MTMAX>
__device__ __forceinline__ void rt_softmax_store(f32x4 (&L)[MTMAX], int MT, float scale, unsigned char *ws, int plane) {
    float mx = -INFINITY;
#pragma unroll
    for (int mt = 0; mt < MTMAX; ++mt)
        if (mt < MT)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, L[mt][r]);
    mx = xrow_max(mx);
    float sum = 0.f;
#pragma unroll
    for (int mt = 0; mt < MTMAX; ++mt)
        if (mt < MT)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float e = fast_exp2(L[mt][r] - mx);
                L[mt][r] = e;
                sum += e;
            }
    const float tot = xrow_sum(sum);  // every lane takes part in the cross-row swaps
    const float inv = scale / tot;
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
#pragma unroll
    for (int mt = 0; mt < MTMAX; ++mt)
        if (mt < MT) {
            u32x2 u[3];
#pragma unroll
            for (int r = 0; r < 4; r += 2) {
                const float a = L[mt][r] * inv, b = L[mt][r + 1] * inv;
                const uint32_t h = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
                const float a1 = a - __uint_as_float(h << 16), b1 = b - __uint_as_float(h & 0xffff0000u);
                const uint32_t m = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a1, (__bf16)b1});
                u[0][r >> 1] = h;
                u[1][r >> 1] = m;
                u[2][r >> 1] = __builtin_bit_cast(
                    uint32_t, bf16x2{(__bf16)(a1 - __uint_as_float(m << 16)), (__bf16)(b1 - __uint_as_float(m & 0xffff0000u))});
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2 *>(ws + k * plane + 32 * mt) = u[k];
        }
}

// Logits of the 16 points whose operand parts `row(kc, parts)` yields, against
// head h's W2' fragments from memory (the next K step's are loaded during the
// products).  Tiles past MT repeat the last one; their logits are not used.
template <int MTMAX, int NP, typename Raw, typename Load, typename Use>
__device__ __forceinline__ void rt_logits(f32x4 (&L)[MTMAX], const bf16_t *w2r, const float *b2s, int h, int MT, int CK,
                                          int lane, Load load, Use use) {
    // tiles that share a point operand (two where four would spill)
    constexpr int G = MTMAX < 4 ? MTMAX : NP == 3 && MTMAX > 4 ? 2 : 4;
    const int g = lane >> 4;
#pragma unroll
    for (int gb = 0; gb < MTMAX; gb += G) {
        if (gb >= MT) break;
        const bf16_t *wt[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int mt = gb + i < MT ? gb + i : MT - 1;
            wt[i] = w2r + (((int64_t)h * MT + mt) * CK * NP * 64 + lane) * 8;
            const float4 b = *reinterpret_cast<const float4 *>(b2s + (h * MT + mt) * 16 + g * 4);
            L[gb + i] = f32x4{b.x, b.y, b.z, b.w};
        }
        Parts<NP> a[G], an[G];
        Raw x, xn;
        auto fetch = [&](int kc, Parts<NP> (&dst)[G], Raw &xd) {
#pragma unroll
            for (int i = 0; i < G; ++i)
#pragma unroll
                for (int k = 0; k < NP; ++k)
                    dst[i].p[k] = *reinterpret_cast<const bf16x8 *>(wt[i] + (kc * NP + k) * 512);
            load(kc, xd);
        };
        fetch(0, a, x);
#pragma unroll 2
        for (int kc = 0; kc < CK; ++kc) {
            if (kc + 1 < CK) fetch(kc + 1, an, xn);
            Parts<NP> b;
            use(kc, gb == 0, x, b);
            mma_parts<G, NP, NP>(&L[gb], a, b);
#pragma unroll
            for (int i = 0; i < G; ++i) a[i] = an[i];
            x = xn;
        }
    }
}

// Row strides (bytes) of the LDS planes: 16 bytes of padding spread the rows over
// the banks for the transposing reads.
__host__ __device__ __forceinline__ int rt_stride(int elems) { return elems * 2 + 16; }

// A fragment whose K slots hold rows: slot (g, t) is row r0 + 8g + t, lane column
// col0 + (l & 15), of a plane of the given row stride.
__device__ __forceinline__ bf16x8 rt_tr(const unsigned char *plane, int stride, int r0, int col0, int lane) {
    const int j = lane & 15, g = lane >> 4;
    const unsigned char *lo = plane + (r0 + 8 * g + (j >> 2)) * stride + (col0 + 4 * (j & 3)) * 2;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)lo);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(lo + 4 * stride));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_bit_cast(bf16x8, v);
}

// Channel tiles per wave of pass 1 (NCT * MTMAX accumulators beside the logits'
// operands: more spill).
__host__ __device__ constexpr int rt_acc_tiles(int mtmax) { return mtmax <= 2 ? 4 : mtmax <= 8 ? 2 : 1; }

// Pass 1 for one (part, head, chunk of CC channels): blocks of PB points (64 or
// 128).  Wave v < PB/16 computes the slice weights of points 16v.. of the block and
// leaves its x rows' chunk in LDS as parts; then every wave contracts the block
// for its own 16-channel tiles (wave, wave + 8, ...) over all slices, and the
// waves share the column sums d.  Two barriers per block.  Channel chunks are as wide as LDS
// and the accumulators allow (the logits are formed again for each chunk).
// Grid: parts * H * nchunk workgroups of 512 threads.  partials: [part][H][M][C+1].
// Bound by the W2' fragments, which each wave reads from L2 for its 16 points.
template <typename T, int MTMAX>
__global__ __launch_bounds__(512, 1) void k_slice_accumulate_rt(const T *__restrict__ x, int64_t n_tile, int64_t span0,
                                                                SpanGeo geo, int32_t nspan, int32_t H, int C, int M,
                                                                int CC, int PB, const bf16_t *__restrict__ w2r,
                                                                const float *__restrict__ b2s,
                                                                float *__restrict__ partials) {
    constexpr int NP = RT_NP<T>, NCT = rt_acc_tiles(MTMAX), ND = (MTMAX + 7) / 8;
    extern __shared__ __attribute__((aligned(16))) unsigned char rt_lds[];
    const int nchunk = (C + CC - 1) / CC, MT = M / 16, CK = rt_ck(C);
    int bid = xcd_remap((int)blockIdx.x, nspan * H * nchunk);  // a part's workgroups share an XCD (and its L2)
    const int chunk = bid % nchunk;
    bid /= nchunk;
    const int h = bid % H, span_local = bid / H;
    const int c0 = chunk * CC, cw = C - c0 < CC ? C - c0 : CC, cct = cw / 16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const int xstride = rt_stride(CC), wstride = rt_stride(M);
    const int xplane = PB * xstride, wplane = PB * wstride;
    unsigned char *const xs = rt_lds, *const ws = rt_lds + NP * xplane;
    const int64_t p_begin = geo.begin(span_local);
    const int64_t p_end = geo.end(span_local, n_tile);

    f32x4 S[NCT][MTMAX], D[ND];
#pragma unroll
    for (int mt = 0; mt < MTMAX; ++mt)
#pragma unroll
        for (int i = 0; i < NCT; ++i) S[i][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < ND; ++i) D[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    Frag<bf16_t> ones;
    ones8(ones);

    for (int64_t pb = p_begin; pb < p_end; pb += PB) {
        __syncthreads();  // the previous block's planes are no longer read
        if (wave * 16 < PB) {
            const int64_t p = pb + wave * 16 + li;
            const bool valid = p < p_end;
            const T *row = x + (valid ? p : p_end - 1) * C;  // padding rows: finite data, zero weights
            unsigned char *xd = xs + (wave * 16 + li) * xstride;
            f32x4 L[MTMAX];
            rt_logits<MTMAX, NP, RtRow<T>>(
                L, w2r, b2s, h, MT, CK, lane,
                [&](int kc, RtRow<T> &r) { r.load(row + 32 * kc + 8 * g, 32 * kc + 8 * g < C); },
                [&](int kc, bool first, const RtRow<T> &r, Parts<NP> &f) {
                    r.parts(f);
                    const int c = 32 * kc + 8 * g - c0;
                    if (first && c >= 0 && c < cw)
#pragma unroll
                        for (int k = 0; k < NP; ++k) *reinterpret_cast<bf16x8 *>(xd + k * xplane + c * 2) = f.p[k];
                });
            rt_softmax_store<MTMAX>(L, MT, valid ? (wave & 2 ? -1.f : 1.f) : 0.f, ws + (wave * 16 + li) * wstride + 8 * g,
                                    wplane);
        }
        __syncthreads();
        for (int r0 = 0; r0 < PB; r0 += 32) {
            const float sign = r0 & 32 ? -1.f : 1.f;  // odd 32-point tiles hold negated weights
            Parts<NP> b[NCT];
#pragma unroll
            for (int i = 0; i < NCT; ++i) {
                const int ct = wave + 8 * i;
                if (ct < cct)
#pragma unroll
                    for (int k = 0; k < NP; ++k) b[i].p[k] = rt_tr(xs + k * xplane, xstride, r0, ct * 16, lane);
            }
#pragma unroll
            for (int mt = 0; mt < MTMAX; ++mt) {
                if (mt < MT) {
                    Parts<3> a;
#pragma unroll
                    for (int k = 0; k < 3; ++k) a.p[k] = rt_tr(ws + k * wplane, wstride, r0, mt * 16, lane);
                    // summed from zero and then added or subtracted: see mma_parts_add
                    using PP = PartProducts<3, NP>;
                    f32x4 t[NCT], d{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int i = 0; i < NCT; ++i) t[i] = d;
#pragma unroll
                    for (int q = 0; q < PP::N; ++q)
#pragma unroll
                        for (int i = 0; i < NCT; ++i)
                            if (wave + 8 * i < cct) t[i] = mma_bf16(a.p[PP::I[q]], b[i].p[PP::J[q]], t[i]);
#pragma unroll
                    for (int i = 0; i < NCT; ++i)
                        if (wave + 8 * i < cct) S[i][mt] += sign * t[i];
                    if (chunk == 0 && (mt & 7) == wave) {
#pragma unroll
                        for (int k = 2; k >= 0; --k) d = mma_bf16(a.p[k], ones.v, d);
                        D[mt >> 3] += sign * d;
                    }
                }
            }
        }
    }
    // lane (g, li) of tile (mt, ct): slice 16mt + 4g + r, channel c0 + 16ct + li
    float *dst = partials + ((size_t)(span0 + span_local) * H + h) * (size_t)M * (C + 1);
#pragma unroll
    for (int mt = 0; mt < MTMAX; ++mt)
        if (mt < MT)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float *row = dst + (size_t)(mt * 16 + g * 4 + r) * (C + 1);
#pragma unroll
                for (int i = 0; i < NCT; ++i)
                    if (wave + 8 * i < cct) row[c0 + (wave + 8 * i) * 16 + li] = S[i][mt][r];
                if (chunk == 0 && (mt & 7) == wave && li == 0) row[C] = D[mt >> 3][r];
            }
}

// Pass 2 for 16 * PT points per workgroup (512 threads): the block's x rows stay in LDS
// as parts; per group of GH heads, wave (head hh = v / PT, point tile v % PT)
// computes the slice weights into LDS, then every wave adds the group's share of
// its own channel tiles (v, v + 8, ...) for all the block's points, so each Z
// fragment is read from L2 once per block.
template <typename T, int MTMAX, int PT>
__global__ __launch_bounds__(512, 1) void k_deslice_rt(const T *__restrict__ x, int64_t n, int32_t H, int C, int M,
                                                       RtGroup gr, const bf16_t *__restrict__ w2r,
                                                       const float *__restrict__ b2s, const bf16_t *__restrict__ zr,
                                                       T *__restrict__ out) {
    constexpr int NP = RT_NP<T>, NCT = PT == 4 ? 2 : 4, P = 16 * PT;  // NCT * 8 tiles cover C (host)
    extern __shared__ __attribute__((aligned(16))) unsigned char rt_lds[];
    const int MT = M / 16, CK = rt_ck(C), CT = C / 16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const int xstride = rt_stride(CK * 32), wstride = rt_stride(gr.KG * 32);
    const int xplane = P * xstride, wplane = P * wstride;
    unsigned char *const xs = rt_lds, *const ws = rt_lds + NP * xplane;
    const int64_t p0 = (int64_t)blockIdx.x * P;

    for (int i = tid; i < P * CK * 4; i += 512) {
        const int r = i / (CK * 4), c = (i - r * (CK * 4)) * 8;
        const int64_t p = p0 + r < n ? p0 + r : n - 1;  // rows past the end: finite data, never stored
        RtRow<T> v;
        v.load(x + p * C + c, c < C);
        Parts<NP> f;
        v.parts(f);
#pragma unroll
        for (int k = 0; k < NP; ++k) *reinterpret_cast<bf16x8 *>(xs + k * xplane + r * xstride + c * 2) = f.p[k];
    }
    // slots past a group's last slice meet zeros of zr; they must hold numbers
    for (int i = tid; i < 3 * wplane / 16; i += 512) reinterpret_cast<uint4 *>(ws)[i] = uint4{0u, 0u, 0u, 0u};

    f32x4 O[NCT][PT];
#pragma unroll
    for (int i = 0; i < NCT; ++i)
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) O[i][pt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int ngroup = (H + gr.GH - 1) / gr.GH;
    __syncthreads();
    for (int group = 0; group < ngroup; ++group) {
        const int hh = wave / PT, pt0 = wave % PT, h = group * gr.GH + hh;
        if (hh < gr.GH && h < H) {
            const unsigned char *row = xs + (pt0 * 16 + li) * xstride + g * 16;
            f32x4 L[MTMAX];
            rt_logits<MTMAX, NP, Parts<NP>>(
                L, w2r, b2s, h, MT, CK, lane,
                [&](int kc, Parts<NP> &f) {
#pragma unroll
                    for (int k = 0; k < NP; ++k)
                        f.p[k] = *reinterpret_cast<const bf16x8 *>(row + k * xplane + kc * 64);
                },
                [&](int, bool, const Parts<NP> &r, Parts<NP> &f) { f = r; });
            rt_softmax_store<MTMAX>(L, MT, 1.f, ws + (pt0 * 16 + li) * wstride + hh * M * 2 + 8 * g, wplane);
        }
        __syncthreads();
        if (wave < CT) {
            const bf16_t *zt[NCT];
#pragma unroll
            for (int i = 0; i < NCT; ++i) {
                const int ct = wave + 8 * i < CT ? wave + 8 * i : wave;
                zt[i] = zr + (((int64_t)group * CT + ct) * gr.KG * NP * 64 + lane) * 8;
            }
            Parts<NP> a[NCT], an[NCT];
            auto fetch = [&](int km, Parts<NP> (&dst)[NCT]) {
#pragma unroll
                for (int i = 0; i < NCT; ++i)
                    if (wave + 8 * i < CT)
#pragma unroll
                        for (int k = 0; k < NP; ++k)
                            dst[i].p[k] = *reinterpret_cast<const bf16x8 *>(zt[i] + (km * NP + k) * 512);
            };
            fetch(0, a);
#pragma unroll 2
            for (int km = 0; km < gr.KG; ++km) {
                if (km + 1 < gr.KG) fetch(km + 1, an);
                Parts<3> b[PT];
#pragma unroll
                for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        b[pt].p[k] = *reinterpret_cast<const bf16x8 *>(ws + k * wplane + (pt * 16 + li) * wstride +
                                                                       km * 64 + g * 16);
                using PP = PartProducts<NP, 3>;
#pragma unroll
                for (int i = 0; i < NCT; ++i)
                    if (wave + 8 * i < CT)
#pragma unroll
                        for (int q = 0; q < PP::N; ++q)
#pragma unroll
                            for (int pt = 0; pt < PT; ++pt)
                                O[i][pt] = mma_bf16(a[i].p[PP::I[q]], b[pt].p[PP::J[q]], O[i][pt]);
#pragma unroll
                for (int i = 0; i < NCT; ++i) a[i] = an[i];
            }
        }
        __syncthreads();  // the weights are rewritten by the next group
    }
    // lane (g, li) of tile ct: channels 16ct + 4g .. +3 of point li
#pragma unroll
    for (int i = 0; i < NCT; ++i)
        if (wave + 8 * i < CT)
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) {
                const int64_t p = p0 + pt * 16 + li;
                if (p >= n) continue;
                T *dst = out + p * C + (wave + 8 * i) * 16 + 4 * g;
                const f32x4 &o = O[i][pt];
                if constexpr (sizeof(T) == 4) {
                    *reinterpret_cast<float4 *>(dst) = float4{o[0], o[1], o[2], o[3]};
                } else {
                    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
                    *reinterpret_cast<bf16x4 *>(dst) =
                        bf16x4{(__bf16)o[0], (__bf16)o[1], (__bf16)o[2], (__bf16)o[3]};
                }
            }
}

// The point blocks of pass 1 for a shape: channels per chunk and points per block.
struct RtPass1 {
    int CC, PB, lds;
};
inline int rt_pass1_lds(int NP, int PB, int CC, int M) { return PB * (NP * rt_stride(CC) + 3 * rt_stride(M)); }
// The widest chunk that LDS and the accumulators (NCT tiles for each of eight waves)
// hold with 64-point blocks, then blocks of 128 points (eight waves of logits
// instead of four) if they fit at that width.
inline RtPass1 rt_pass1(int NP, int C, int M) {
    const int most = 128 * rt_acc_tiles((M + 15) / 16);
    int chunks = 1, CC = C;
    while (CC > most || rt_pass1_lds(NP, 64, CC, M) > RT_LDS_MAX) {
        ++chunks;
        CC = ((C + chunks - 1) / chunks + 15) / 16 * 16;
    }
    const int PB = rt_pass1_lds(NP, 128, CC, M) <= RT_LDS_MAX ? 128 : 64;
    return RtPass1{CC, PB, rt_pass1_lds(NP, PB, CC, M)};
}

// Points and heads per step of pass 2 for a shape: 64 points and two heads keep
// eight waves busy; fewer heads, then fewer points, where LDS asks for it (32
// points always for C > 256, whose channel tiles take four accumulators per wave).
// The Z layout depends on GH, so it follows from the shape alone.
struct RtPass2 {
    int PT, GH;
};
inline int rt_pass2_lds(int NP, int PT, int GH, int C, int M) {
    return 16 * PT * (NP * rt_stride(rt_ck(C) * 32) + 3 * rt_stride((GH * M + 31) / 32 * 32));
}
inline RtPass2 rt_pass2(int NP, int C, int M) {
    for (int PT = C <= 256 ? 4 : 2; PT >= 2; PT /= 2)
        for (int GH = 8 / PT; GH >= 1; GH /= 2)
            if (rt_pass2_lds(NP, PT, GH, C, M) <= RT_LDS_MAX) return RtPass2{PT, GH};
    return RtPass2{2, 1};  // C = 512, M = 256 takes 150 KB: every shape fits above
}

}  // namespace ts3
