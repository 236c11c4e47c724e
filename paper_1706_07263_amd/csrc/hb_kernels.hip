// HIP kernels of the haemoglobin-estimation path for gfx950 (MI355X).
//
//   K0  k_tikhonov_fp64     plan time, FP64: E, (E'E + gamma I)^-1 E'   (Method, Eq. 5)
//   K1  k_log_haar_reg<n>   log-attenuation, n-level 2D Haar, Tikhonov on the
//                           directional coefficients and the inverse Haar of
//                           that detail part, one block per thread (n <= 2);
//                           with the linear low-pass estimator also the maps
//       k_log_haar          the same in LDS-staged strips (unaligned frames of
//                           n <= 2 levels)
//       k_log_haar_df       log-attenuation, block means and detail part in
//                           double-float: three levels and more, and operators
//                           with a large norm at any n    (Eq. 1-2, 4, 5)
//   K2a k_reference         best probe over the whole grid (split grids only)
//   K2  k_posterior         posterior mean over the THb x SO2 grid on the
//                           low-pass band (MFMA logits); with one split and
//                           n <= 3 it also writes the maps         (Fig. 1)
//       k_posterior_direct  the same with VALU logits (coarse grids, small sigma;
//                           double-float logits for the coarsest)
//   K3  k_recompose         split merge plus detail part to the THb/SO2 maps
//                           (split grids, four levels and more, the linear
//                           low-pass of unaligned frames)
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "hb_df.h"
#include "hb_internal.h"

namespace hb {

namespace {

// ---------------------------------------------------------------------------
// K0: Jacobian of the forward model at the reference point and the Tikhonov
// operator, in double precision.  in = [n, L, ref_hb, ref_hbo2, lambda,
// eps_hb[n], eps_hbo2[n], response[3][n] (rows normalised to unit sum)];
// out = [E(6), M(6), gamma, ok]; mf[0..5] = M rounded to float32 and
// mf[8..13] the low parts (M - mf[0..5], rounded), so that mf[i] + mf[8 + i]
// carries M to double-float precision (mf[6, 7] and mf[14, 15] are the
// host's low-pass offset).
// ---------------------------------------------------------------------------
__global__ void k_tikhonov_fp64(const double *__restrict__ in, double *__restrict__ out,
                                float *__restrict__ mf) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const int n = (int)in[0];
    const double L = in[1], chb = in[2], chbo2 = in[3], lam = in[4];
    const double *ehb = in + 5, *eox = in + 5 + n, *resp = in + 5 + 2 * n;
    double E[6];
    for (int k = 0; k < 3; ++k) {
        double den = 0.0, nh = 0.0, no = 0.0;
        for (int j = 0; j < n; ++j) {
            double w = resp[k * n + j] * exp(-L * (ehb[j] * chb + eox[j] * chbo2));
            den += w;
            nh += w * ehb[j];
            no += w * eox[j];
        }
        E[2 * k] = L * nh / den;
        E[2 * k + 1] = L * no / den;
    }
    double a00 = 0, a01 = 0, a11 = 0;
    for (int k = 0; k < 3; ++k) {
        a00 += E[2 * k] * E[2 * k];
        a01 += E[2 * k] * E[2 * k + 1];
        a11 += E[2 * k + 1] * E[2 * k + 1];
    }
    const double gamma = lam * 0.5 * (a00 + a11);
    const double b00 = a00 + gamma, b11 = a11 + gamma;
    const double det = b00 * b11 - a01 * a01;
    const bool ok = fabs(det) > 1e-14 * (fabs(b00 * b11) + a01 * a01);
    const double i00 = b11 / det, i01 = -a01 / det, i11 = b00 / det;
    for (int k = 0; k < 3; ++k) {
        double m0 = i00 * E[2 * k] + i01 * E[2 * k + 1];
        double m1 = i01 * E[2 * k] + i11 * E[2 * k + 1];
        out[6 + k] = m0;
        out[9 + k] = m1;
        mf[k] = (float)m0;
        mf[3 + k] = (float)m1;
        mf[8 + k] = (float)(m0 - (double)(float)m0);   // low parts
        mf[11 + k] = (float)(m1 - (double)(float)m1);
    }
    for (int i = 0; i < 6; ++i) out[i] = E[i];
    out[12] = gamma;
    out[13] = ok ? 1.0 : 0.0;
}

// Clang vector types (the non-temporal builtins and the MFMA builtins take these).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x3 __attribute__((ext_vector_type(3)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// Word 3 of a raw buffer resource on gfx9-family GPUs (32-bit data format).
constexpr int kBufferWord3 = 0x00020000;

// ---------------------------------------------------------------------------
// Storage-type loads.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float load_px(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_px(const __half *p, size_t i) { return __half2float(p[i]); }
__device__ __forceinline__ float load_px(const uint16_t *p, size_t i) {
    return __uint_as_float((uint32_t)p[i] << 16);  // bfloat16 -> float32 is exact
}

__device__ __forceinline__ void load4(const float *p, float v[4]) {
    const float4 x = *reinterpret_cast<const float4 *>(p);
    v[0] = x.x;
    v[1] = x.y;
    v[2] = x.z;
    v[3] = x.w;
}
__device__ __forceinline__ void load4(const __half *p, float v[4]) {
    const uint2 x = *reinterpret_cast<const uint2 *>(p);
    v[0] = __half2float(__ushort_as_half((unsigned short)(x.x & 0xffffu)));
    v[1] = __half2float(__ushort_as_half((unsigned short)(x.x >> 16)));
    v[2] = __half2float(__ushort_as_half((unsigned short)(x.y & 0xffffu)));
    v[3] = __half2float(__ushort_as_half((unsigned short)(x.y >> 16)));
}
__device__ __forceinline__ void load4(const uint16_t *p, float v[4]) {
    const uint2 x = *reinterpret_cast<const uint2 *>(p);
    v[0] = __uint_as_float(x.x << 16);
    v[1] = __uint_as_float(x.x & 0xffff0000u);
    v[2] = __uint_as_float(x.y << 16);
    v[3] = __uint_as_float(x.y & 0xffff0000u);
}

// z less its mean over the channels, as double-floats.
__device__ __forceinline__ void remove_channel_mean(float zh[3], float zl[3]) {
    float sh = zh[0], sl = zl[0];
    df_add2(sh, sl, zh[1], zl[1]);
    df_add2(sh, sl, zh[2], zl[2]);
    // (sh + sl) / 3: the remainder of the leading quotient is exact by FMA
    const float mh = sh * (1.0f / 3.0f);
    const float ml = (fmaf(-3.0f, mh, sh) + sl) * (1.0f / 3.0f);
#pragma unroll
    for (int k = 0; k < 3; ++k) df_add2(zh[k], zl[k], -mh, -ml);
}

struct StripPos {
    int f, br, blk0, nb, ncols, Wt, row0, col0, B;
};

__device__ __forceinline__ StripPos strip_pos(const Dims &d) {
    StripPos s;
    int idx = blockIdx.x;
    const int sc = idx % d.strips_per_row;
    idx /= d.strips_per_row;
    s.br = idx % d.hl;
    s.f = idx / d.hl;
    s.blk0 = sc * d.bps;
    s.nb = min(d.bps, d.wl - s.blk0);
    s.B = 1 << d.levels;
    s.ncols = s.nb << d.levels;
    s.Wt = d.bps << d.levels;
    s.row0 = s.br << d.levels;
    s.col0 = s.blk0 << d.levels;
    return s;
}

// -ln(I / R) for a pixel relative to its block mean R, rinv = 1 / R: with
// x = (I - R) rinv (one rounded product), ln(1 + x) for |x| <= 1/16 is the
// series x + x^2 (-1/2 + x/3 - x^2/4 + x^3/5 - x^4/6 + x^5/7) (truncation
// below 2^-28 relative; 0.55 ulp worst measured against a double log1p over
// 5e7 samples), and log1pf beyond.  Both K1 variants use this, so they agree
// bit for bit.
__device__ __forceinline__ float neg_log_ratio(float I, float R, float rinv) {
    const float x = (I - R) * rinv;
    if (fabsf(x) <= 0.0625f) {
        float q = fmaf(x, 1.0f / 7.0f, -1.0f / 6.0f);
        q = fmaf(q, x, 0.2f);
        q = fmaf(q, x, -0.25f);
        q = fmaf(q, x, 1.0f / 3.0f);
        q = fmaf(q, x, -0.5f);
        return -fmaf(x * x, q, x);
    }
    return -log1pf(x);
}

// ---------------------------------------------------------------------------
// K1: one workgroup per strip of 2^n pixel rows x (bps * 2^n) columns.
//
// Numerics: each block's log-attenuation is carried relative to the block's
// mean intensity R, u(q) = -ln(I(q)/R) = -log1p((I(q) - R)/R), so directional
// coefficients are computed from small, accurately rounded numbers.  Details of
// u equal those of y = -ln I (they differ by a per-block constant); the block
// mean of y is recovered as -ln(R/I_ref) + mean(u) relative to the plan's
// reference intensity I_ref.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlockThreads) void k_log_haar(const T *__restrict__ frames, HaarArgs a) {
    __shared__ float s_i[3][kStripPixels];
    __shared__ float s_u[3][kStripPixels];
    __shared__ float s_r[3][kStripPixels / 4];
    const Dims &d = a.d;
    const StripPos s = strip_pos(d);
    const int n = d.levels, B = s.B, Wt = s.Wt, ncols = s.ncols;
    const int tid = threadIdx.x;

    // 1. Coalesced load of the strip, clamp.  Each row of the strip is one
    //    contiguous HWC run of ncols * 3 values; with 4-value alignment the
    //    loads are 16-byte (FP32) or 8-byte (FP16/BF16) vectors, all issued
    //    before any is used.
    const size_t frame_off = (size_t)s.f * d.H * d.W * 3;
    const int run = ncols * 3;
    const T *__restrict__ base = frames + frame_off + ((size_t)s.row0 * d.W + s.col0) * 3;
    const size_t row_stride = (size_t)d.W * 3;
    auto put = [&](int r, int p, float v) {
        const int c = p / 3, k = p - 3 * c;
        v = (v < a.floor) ? a.floor : v;  // NaN stays NaN
        s_i[k][r * Wt + c] = v;
        s_u[k][r * Wt + c] = v;
    };
    if (a.vec4 && (d.W & 3) == 0 && (run & 3) == 0) {
        const int r4 = run >> 2, total = B * r4;
        constexpr int kMaxVec = kStripPixels * 3 / 4 / kBlockThreads;   // 6
        float v[kMaxVec][4];
        int rr[kMaxVec], jj[kMaxVec];
#pragma unroll
        for (int t = 0; t < kMaxVec; ++t) {
            const int idx = tid + t * kBlockThreads;
            rr[t] = idx < total ? idx / r4 : 0;
            jj[t] = idx < total ? idx - rr[t] * r4 : -1;
            if (jj[t] >= 0) load4(base + rr[t] * row_stride + 4 * jj[t], v[t]);
        }
#pragma unroll
        for (int t = 0; t < kMaxVec; ++t)
            if (jj[t] >= 0)
#pragma unroll
                for (int e = 0; e < 4; ++e) put(rr[t], 4 * jj[t] + e, v[t][e]);
    } else {
        for (int r = 0; r < B; ++r)
            for (int p = tid; p < run; p += kBlockThreads) put(r, p, load_px(base, r * row_stride + p));
    }
    __syncthreads();

    // 2. Block sums of intensity by a 2x2 cascade, then the block mean R.
    for (int l = 1; l <= n; ++l) {
        const int h = 1 << (l - 1), g2 = 2 * h, gc = ncols >> l;
        for (int r = 0; r < B; r += g2)
            for (int q = tid; q < gc * 3; q += kBlockThreads) {
                const int cg = q / 3, k = q - 3 * cg, c = cg * g2;
                float *u = s_u[k];
                u[r * Wt + c] = (u[r * Wt + c] + u[r * Wt + c + h]) + (u[(r + h) * Wt + c] + u[(r + h) * Wt + c + h]);
            }
        __syncthreads();
    }
    if (n > 0) {
        const float inv = 1.0f / (float)(1 << (2 * n));
        for (int q = tid; q < s.nb * 3; q += kBlockThreads) {
            const int j = q / 3, k = q - 3 * j;
            s_r[k][j] = s_u[k][j << n] * inv;
        }
    }
    __syncthreads();

    // 3. Log-ratio to the block reference.
    for (int r = 0; r < B; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k)
            for (int c = tid; c < ncols; c += kBlockThreads) {
                const float I = s_i[k][r * Wt + c];
                const float R = (n > 0) ? s_r[k][c >> n] : I;
                s_u[k][r * Wt + c] = neg_log_ratio(I, R, 1.0f / R);
            }
    __syncthreads();

    // 4. n-level Haar in place.  Window (a, b, c, d) = (r,c), (r,c+h), (r+h,c),
    //    (r+h,c+h); coefficients = window * H (Eq. 1-2): LL -> (r,c),
    //    row difference -> (r+h,c), diagonal -> (r+h,c+h), column difference -> (r,c+h).
    for (int l = 1; l <= n; ++l) {
        const int h = 1 << (l - 1), g2 = 2 * h, gc = ncols >> l;
        for (int r = 0; r < B; r += g2)
            for (int q = tid; q < gc * 3; q += kBlockThreads) {
                const int cg = q / 3, k = q - 3 * cg, c = cg * g2;
                float *u = s_u[k];
                const int i0 = r * Wt + c, i1 = i0 + h, i2 = (r + h) * Wt + c, i3 = i2 + h;
                const float w0 = u[i0], w1 = u[i1];
                const float w2 = u[i2], w3 = u[i3];
                u[i0] = 0.5f * ((w0 + w1) + (w2 + w3));
                u[i2] = 0.5f * ((w0 + w1) - (w2 + w3));
                u[i3] = 0.5f * ((w0 - w1) - (w2 - w3));
                u[i1] = 0.5f * ((w0 - w1) + (w2 - w3));
            }
        __syncthreads();
    }

    // 5. Centred low-pass observation z = ybar - mu_ref per block, as a
    //    double-float: ybar - mu_ref = ln(I_ref / R) + mean(u).  With the
    //    illumination term z loses its mean over the channels (the component
    //    along (1,1,1) that a common log offset can absorb).
    const float invB = 1.0f / (float)B;
    if (!a.project) {
        for (int q = tid; q < s.nb * 3; q += kBlockThreads) {
            const int j = q / 3, k = q - 3 * j;
            const float R = (n > 0) ? s_r[k][j] : s_i[k][j];
            float zh, zl;
            ln_ratio_df(a.iref[k], R, zh, zl);
            df_add(zh, zl, s_u[k][j << n] * invB);
            const size_t o = (size_t)s.br * d.wl + s.blk0 + j;
            a.z[((size_t)s.f * 6 + k) * d.LL + o] = zh;
            a.z[((size_t)s.f * 6 + 3 + k) * d.LL + o] = zl;
        }
    } else {
        for (int j = tid; j < s.nb; j += kBlockThreads) {
            float zh[3], zl[3];
            for (int k = 0; k < 3; ++k) {
                const float R = (n > 0) ? s_r[k][j] : s_i[k][j];
                ln_ratio_df(a.iref[k], R, zh[k], zl[k]);
                df_add(zh[k], zl[k], s_u[k][j << n] * invB);
            }
            remove_channel_mean(zh, zl);
            const size_t o = (size_t)s.br * d.wl + s.blk0 + j;
            for (int k = 0; k < 3; ++k) {
                a.z[((size_t)s.f * 6 + k) * d.LL + o] = zh[k];
                a.z[((size_t)s.f * 6 + 3 + k) * d.LL + o] = zl[k];
            }
        }
    }

    // 6. Tikhonov on every directional coefficient: (Hb, HbO2) = M * (R, G, B),
    //    the low-pass slot set to 0 (s_i, read by step 5 when n = 0, then
    //    holds the result).
    __syncthreads();
    const float m0 = a.M[0], m1 = a.M[1], m2 = a.M[2], m3 = a.M[3], m4 = a.M[4], m5 = a.M[5];
    for (int r = 0; r < B; ++r)
        for (int c = tid; c < ncols; c += kBlockThreads) {
            float ox = 0.0f, oy = 0.0f;
            if (((r | c) & (B - 1)) != 0) {
                const float d0 = s_u[0][r * Wt + c], d1 = s_u[1][r * Wt + c], d2 = s_u[2][r * Wt + c];
                ox = fmaf(m0, d0, fmaf(m1, d1, m2 * d2));
                oy = fmaf(m3, d0, fmaf(m4, d1, m5 * d2));
            }
            s_i[0][r * Wt + c] = ox;
            s_i[1][r * Wt + c] = oy;
        }
    __syncthreads();

    // 7. Inverse Haar of the detail part (Eq. 4: window = coefficients * H,
    //    levels n..1): the maps are this plus the block's low-pass estimate.
    for (int l = n; l >= 1; --l) {
        const int h = 1 << (l - 1), g2 = 2 * h, gc = ncols >> l;
        for (int r = 0; r < B; r += g2)
            for (int q = tid; q < gc * 2; q += kBlockThreads) {
                const int k = q & 1, c = (q >> 1) * g2;
                float *u = s_i[k];
                const float ll = u[r * Wt + c], d1 = u[(r + h) * Wt + c];
                const float d2 = u[(r + h) * Wt + c + h], d3 = u[r * Wt + c + h];
                u[r * Wt + c] = 0.5f * ((ll + d1) + (d2 + d3));
                u[r * Wt + c + h] = 0.5f * ((ll + d1) - (d2 + d3));
                u[(r + h) * Wt + c] = 0.5f * ((ll - d1) - (d2 - d3));
                u[(r + h) * Wt + c + h] = 0.5f * ((ll - d1) + (d2 - d3));
            }
        __syncthreads();
    }
    for (int r = 0; r < B; ++r)
        for (int c = tid; c < ncols; c += kBlockThreads)
            a.det[((size_t)s.f * d.H + s.row0 + r) * d.W + s.col0 + c] =
                make_float2(s_i[0][r * Wt + c], s_i[1][r * Wt + c]);
}

// Maps of V consecutive pixels (offset o) from their detail part and the
// block's low-pass estimate e; vector stores when V > 1 (the host checks the
// alignment of the map pointers).  Null maps are skipped.
template <int V>
__device__ __forceinline__ void write_maps(float *mhb, float *mox, float *mth, float *mso, float thb_eps, size_t o,
                                           float2 e, const float2 *dp) {
    float hb[V], ox[V], th[V], so[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        hb[i] = e.x + dp[i].x;
        ox[i] = e.y + dp[i].y;
        th[i] = hb[i] + ox[i];
        so[i] = (th[i] > thb_eps) ? ox[i] / th[i] : __builtin_nanf("");
    }
    // streaming stores (non-temporal): the maps are not read again here
    auto put = [&](float *m, const float *v) {
        if (!m) return;
        if constexpr (V == 4) {
            __builtin_nontemporal_store(f32x4{v[0], v[1], v[2], v[3]}, reinterpret_cast<f32x4 *>(m + o));
        } else if constexpr (V == 2) {
            __builtin_nontemporal_store(f32x2{v[0], v[1]}, reinterpret_cast<f32x2 *>(m + o));
        } else {
            __builtin_nontemporal_store(v[0], m + o);
        }
    };
    put(mhb, hb);
    put(mox, ox);
    put(mth, th);
    put(mso, so);
}

// Linear low-pass estimate offset + M z with M, the offset and z as
// double-floats: the terms are about |M| |z| (~1e3 uM) while the estimate is
// tens of uM.
__device__ __forceinline__ float2 linear_estimate(const float *M, const float zh[3], const float zl[3]) {
    float hh = M[6], hl = M[14], oh = M[7], ol = M[15];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        df_mul_add(hh, hl, M[k], M[8 + k], zh[k], zl[k]);
        df_mul_add(oh, ol, M[3 + k], M[11 + k], zh[k], zl[k]);
    }
    return make_float2(hh + hl, oh + ol);
}

// ---------------------------------------------------------------------------
// K1, register variant for n <= 2: one thread per 2^n x 2^n block, the block
// held in registers (no LDS, no barriers), the strip kernel's arithmetic in
// the same order (so both give the same bits).  Each block row is a run of
// 3 * 2^n stored values starting at a multiple of 2^n values: three vector
// loads of 2^n values when the frames pointer is aligned to 2^n values.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ float half_bits(unsigned b);
template <>
__device__ __forceinline__ float half_bits<__half>(unsigned b) {
    return __half2float(__ushort_as_half((unsigned short)b));
}
template <>
__device__ __forceinline__ float half_bits<uint16_t>(unsigned b) {
    return __uint_as_float(b << 16);  // bfloat16 -> float32 is exact
}

template <typename T, int BW>
__device__ __forceinline__ void load_run(const T *p, float *v) {
    if constexpr (std::is_same<T, float>::value) {
        if constexpr (BW == 4) {
            const float4 x = *reinterpret_cast<const float4 *>(p);
            v[0] = x.x;
            v[1] = x.y;
            v[2] = x.z;
            v[3] = x.w;
        } else if constexpr (BW == 2) {
            const float2 x = *reinterpret_cast<const float2 *>(p);
            v[0] = x.x;
            v[1] = x.y;
        } else {
            v[0] = p[0];
        }
    } else {
        if constexpr (BW == 4) {
            const uint2 x = *reinterpret_cast<const uint2 *>(p);
            v[0] = half_bits<T>(x.x & 0xffffu);
            v[1] = half_bits<T>(x.x >> 16);
            v[2] = half_bits<T>(x.y & 0xffffu);
            v[3] = half_bits<T>(x.y >> 16);
        } else if constexpr (BW == 2) {
            const unsigned x = *reinterpret_cast<const unsigned *>(p);
            v[0] = half_bits<T>(x & 0xffffu);
            v[1] = half_bits<T>(x >> 16);
        } else {
            v[0] = half_bits<T>(*reinterpret_cast<const unsigned short *>(p));
        }
    }
}

// Detail-part rows are streamed out (non-temporal): they are read again
// only by the posterior's epilogue or the recomposition kernel.
template <int BW>
__device__ __forceinline__ void store_row(float2 *p, const float2 *o) {
    if constexpr (BW == 4) {
        __builtin_nontemporal_store(f32x4{o[0].x, o[0].y, o[1].x, o[1].y}, reinterpret_cast<f32x4 *>(p));
        __builtin_nontemporal_store(f32x4{o[2].x, o[2].y, o[3].x, o[3].y}, reinterpret_cast<f32x4 *>(p) + 1);
    } else if constexpr (BW == 2) {
        __builtin_nontemporal_store(f32x4{o[0].x, o[0].y, o[1].x, o[1].y}, reinterpret_cast<f32x4 *>(p));
    } else {
        __builtin_nontemporal_store(f32x2{o[0].x, o[0].y}, reinterpret_cast<f32x2 *>(p));
    }
}

// BW pixels of a block row at offset o: the detail part, and with the linear
// low-pass estimator (MAPS) the four maps from it and the block's estimate e,
// in stores of a.vec pixels.
template <int BW, bool MAPS>
__device__ __forceinline__ void put_row(const HaarArgs &a, size_t o, const float2 *row, float2 e) {
    if (!MAPS || a.det) store_row<BW>(a.det + o, row);
    if constexpr (MAPS) {
        if (BW == 4 && a.vec == 4) {
            write_maps<4>(a.hb, a.hbo2, a.thb, a.so2, a.thb_eps, o, e, row);
        } else if (BW >= 2 && a.vec >= 2) {
#pragma unroll
            for (int c = 0; c + 2 <= BW; c += 2) write_maps<2>(a.hb, a.hbo2, a.thb, a.so2, a.thb_eps, o + c, e, row + c);
        } else {
#pragma unroll
            for (int c = 0; c < BW; ++c) write_maps<1>(a.hb, a.hbo2, a.thb, a.so2, a.thb_eps, o + c, e, row + c);
        }
    }
}

// MAPS (linear low-pass estimator, no posterior): the estimate and the maps
// too, so that neither the detail part nor the observation is read again.
// Bound by HBM: sixteen 1920x1080 FP32 frames 254 us at 38 bytes a pixel, 5.0
// TB/s (a plain copy reaches 5.1); K1 and the maps kernel took 287 for 47.
template <typename T, int N, bool MAPS>
__global__ __launch_bounds__(kBlockThreads) void k_log_haar_reg(const T *__restrict__ frames, HaarArgs a) {
    constexpr int BW = 1 << N, NP = BW * BW;
    const Dims &d = a.d;
    const unsigned q = blockIdx.x * kBlockThreads + threadIdx.x, f = blockIdx.y;   // block of frame f
    if (q >= (unsigned)d.LL) return;
    const int br = (int)(q / (unsigned)d.wl), bc = (int)(q - (unsigned)br * (unsigned)d.wl);
    const int row0 = br << N, col0 = bc << N;
    const T *__restrict__ base = frames + ((size_t)f * d.H * d.W + (size_t)row0 * d.W + col0) * 3;

    // 1. Loads (all issued first), clamp.  I[k][r * BW + c].
    float v[BW][3 * BW];
#pragma unroll
    for (int r = 0; r < BW; ++r)
#pragma unroll
        for (int t = 0; t < 3; ++t) load_run<T, BW>(base + (size_t)r * d.W * 3 + t * BW, &v[r][t * BW]);
    float I[3][NP], u[3][NP];
#pragma unroll
    for (int r = 0; r < BW; ++r)
#pragma unroll
        for (int e = 0; e < 3 * BW; ++e) {
            const float x = v[r][e];
            I[e % 3][r * BW + e / 3] = (x < a.floor) ? a.floor : x;  // NaN stays NaN
        }

    // 2. Block sum by the 2x2 cascade, block mean R.
    float R[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int i = 0; i < NP; ++i) u[k][i] = I[k][i];
#pragma unroll
        for (int l = 1; l <= N; ++l) {
            const int h = 1 << (l - 1), g2 = 2 * h;
#pragma unroll
            for (int r = 0; r < BW; r += g2)
#pragma unroll
                for (int c = 0; c < BW; c += g2)
                    u[k][r * BW + c] = (u[k][r * BW + c] + u[k][r * BW + c + h]) +
                                       (u[k][(r + h) * BW + c] + u[k][(r + h) * BW + c + h]);
        }
        R[k] = (N > 0) ? u[k][0] * (1.0f / (float)(1 << (2 * N))) : I[k][0];
    }

    // 3. Log-ratio to the block mean; 4. Haar in place (window * H, Eq. 1-2).
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float rinv = 1.0f / R[k];
#pragma unroll
        for (int i = 0; i < NP; ++i) u[k][i] = neg_log_ratio(I[k][i], R[k], rinv);
#pragma unroll
        for (int l = 1; l <= N; ++l) {
            const int h = 1 << (l - 1), g2 = 2 * h;
#pragma unroll
            for (int r = 0; r < BW; r += g2)
#pragma unroll
                for (int c = 0; c < BW; c += g2) {
                    const int i0 = r * BW + c, i1 = i0 + h, i2 = (r + h) * BW + c, i3 = i2 + h;
                    const float w0 = u[k][i0], w1 = u[k][i1];
                    const float w2 = u[k][i2], w3 = u[k][i3];
                    u[k][i0] = 0.5f * ((w0 + w1) + (w2 + w3));
                    u[k][i2] = 0.5f * ((w0 + w1) - (w2 + w3));
                    u[k][i3] = 0.5f * ((w0 - w1) - (w2 - w3));
                    u[k][i1] = 0.5f * ((w0 - w1) + (w2 - w3));
                }
        }
    }

    // 5. Centred low-pass observation (double-float), optionally projected.
    const float invB = 1.0f / (float)BW;
    float zh[3], zl[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        ln_ratio_df(a.iref[k], R[k], zh[k], zl[k]);
        df_add(zh[k], zl[k], u[k][0] * invB);
    }
    if (a.project) remove_channel_mean(zh, zl);
    if (!MAPS || a.z)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            a.z[((size_t)f * 6 + k) * d.LL + q] = zh[k];
            a.z[((size_t)f * 6 + 3 + k) * d.LL + q] = zl[k];
        }
    float2 e = make_float2(0.0f, 0.0f);
    if constexpr (MAPS) {
        e = linear_estimate(a.M, zh, zl);
        if (a.est) a.est[(size_t)f * d.LL + q] = e;
    }

    // 6. Tikhonov on the directional coefficients (low-pass slot 0); 7. the
    //    inverse Haar of this detail part; block rows as vector stores.
    const float m0 = a.M[0], m1 = a.M[1], m2 = a.M[2], m3 = a.M[3], m4 = a.M[4], m5 = a.M[5];
    float o[2][NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        o[0][i] = o[1][i] = 0.0f;
        if (i != 0) {
            const float d0 = u[0][i], d1 = u[1][i], d2 = u[2][i];
            o[0][i] = fmaf(m0, d0, fmaf(m1, d1, m2 * d2));
            o[1][i] = fmaf(m3, d0, fmaf(m4, d1, m5 * d2));
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int l = N; l >= 1; --l) {
            const int h = 1 << (l - 1), g2 = 2 * h;
#pragma unroll
            for (int r = 0; r < BW; r += g2)
#pragma unroll
                for (int c = 0; c < BW; c += g2) {
                    const float ll = o[k][r * BW + c], d1 = o[k][(r + h) * BW + c];
                    const float d2 = o[k][(r + h) * BW + c + h], d3 = o[k][r * BW + c + h];
                    o[k][r * BW + c] = 0.5f * ((ll + d1) + (d2 + d3));
                    o[k][r * BW + c + h] = 0.5f * ((ll + d1) - (d2 + d3));
                    o[k][(r + h) * BW + c] = 0.5f * ((ll - d1) - (d2 - d3));
                    o[k][(r + h) * BW + c + h] = 0.5f * ((ll - d1) + (d2 - d3));
                }
        }
#pragma unroll
    for (int r = 0; r < BW; ++r) {
        float2 row[BW];
#pragma unroll
        for (int c = 0; c < BW; ++c) row[c] = make_float2(o[0][r * BW + c], o[1][r * BW + c]);
        put_row<BW, MAPS>(a, ((size_t)f * d.H + row0 + r) * d.W + col0, row, e);
    }
}

// ---------------------------------------------------------------------------
// K1, double-float variant (three or more levels, or |M| above
// kK1PrecisionBudget).  With float32 log-ratios their rounding, which grows
// with the block, reaches the maps through |M| (1e3 to 2e3 uM per unit) at up
// to 1.3e-4 uM for three levels; here the log-attenuations, their block mean
// and the Tikhonov apply are double-floats and each detail value is rounded
// once.  The Haar transform is orthonormal, so what the Tikhonov operator M
// makes of the directional coefficients recomposes to M (y - block mean of y):
// neither the transform nor its inverse has to be formed.
//
// One thread takes a 4 x 4 sub-block (the block itself up to two levels); the
// 4^(N - 2) threads of a block are neighbouring lanes in Z order and sum their
// means by lane exchanges (every lane gets the same bits).  VEC: the frames
// pointer is aligned to BW stored values.  Bound by VALU issue (about 180
// operations per pixel; 135 registers, three waves per SIMD): four 1920x1080
// frames at three levels 64 us; the strips in LDS with a double-float Haar
// cascade that this replaces took 212.
// ---------------------------------------------------------------------------
template <typename T, int N, bool VEC, bool MAPS>
__global__ __launch_bounds__(kBlockThreads) void k_log_haar_df(const T *__restrict__ frames, HaarArgs a) {
    constexpr int SB = N < 2 ? N : 2, BW = 1 << SB, UP = N - SB;
    const Dims &d = a.d;
    const unsigned idx = blockIdx.x * kBlockThreads + threadIdx.x, f = blockIdx.y;
    const unsigned q = idx >> (2 * UP);            // block of frame f
    if (q >= (unsigned)d.LL) return;               // all lanes of a block or none
    const int sub = (int)(idx & ((1 << (2 * UP)) - 1));
    int sr = 0, sc = 0;   // Z order: even bits column, odd bits row
#pragma unroll
    for (int l = 0; l < UP; ++l) {
        sc |= (sub >> (2 * l) & 1) << l;
        sr |= (sub >> (2 * l + 1) & 1) << l;
    }
    const int br = (int)(q / (unsigned)d.wl), bc = (int)(q - (unsigned)br * (unsigned)d.wl);
    const int row0 = (br << N) + (sr << SB), col0 = (bc << N) + (sc << SB);
    const T *__restrict__ base = frames + ((size_t)f * d.H * d.W + (size_t)row0 * d.W + col0) * 3;

    // Loads (all issued first), clamp, ln I.  h[r][3 c + k] + l[r][3 c + k].
    float h[BW][3 * BW], l[BW][3 * BW];
#pragma unroll
    for (int r = 0; r < BW; ++r)
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const T *p = base + (size_t)r * d.W * 3 + t * BW;
            if constexpr (VEC)
                load_run<T, BW>(p, &h[r][t * BW]);
            else
#pragma unroll
                for (int e = 0; e < BW; ++e) h[r][t * BW + e] = load_px(p, e);
        }
    // Block mean of ln I: sums with the rounding errors carried.
    float mh[3], ml[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        mh[k] = ml[k] = 0.0f;
#pragma unroll
        for (int r = 0; r < BW; ++r)
#pragma unroll
            for (int c = 0; c < BW; ++c) {
                const float x = h[r][3 * c + k];
                ln_df((x < a.floor) ? a.floor : x, h[r][3 * c + k], l[r][3 * c + k]);   // NaN stays NaN
                carry_add(mh[k], ml[k], h[r][3 * c + k], l[r][3 * c + k]);
            }
#pragma unroll
        for (int o = 1; o < 1 << (2 * UP); o <<= 1) {
            const float xh = __shfl_xor(mh[k], o), xl = __shfl_xor(ml[k], o);
            float s, e;
            two_sum(mh[k], xh, s, e);
            mh[k] = s;
            ml[k] = (ml[k] + xl) + e;
        }
        const float inv = 1.0f / (float)(1 << (2 * N));   // exact
        fast_two_sum(mh[k] * inv, ml[k] * inv, mh[k], ml[k]);
    }

    // Centred low-pass observation z = ln I_ref - mean ln I, optionally
    // without its mean over the channels (illumination term).
    float2 e = make_float2(0.0f, 0.0f);
    if (MAPS || sub == 0) {
        float zh[3], zl[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            zh[k] = a.ln_iref[k];
            zl[k] = a.ln_iref[3 + k];
            df_add2(zh[k], zl[k], -mh[k], -ml[k]);
        }
        if (a.project) remove_channel_mean(zh, zl);
        if (sub == 0 && (!MAPS || a.z))
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                a.z[((size_t)f * 6 + k) * d.LL + q] = zh[k];
                a.z[((size_t)f * 6 + 3 + k) * d.LL + q] = zl[k];
            }
        if constexpr (MAPS) {
            e = linear_estimate(a.M, zh, zl);
            if (sub == 0 && a.est) a.est[(size_t)f * d.LL + q] = e;
        }
    }

    // Detail part M (y - mean y) = M (mean ln I - ln I), each value a
    // compensated dot product.
#pragma unroll
    for (int r = 0; r < BW; ++r) {
        float2 row[BW];
#pragma unroll
        for (int c = 0; c < BW; ++c) {
            float dh[3], dl[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                two_sum(mh[k], -h[r][3 * c + k], dh[k], dl[k]);
                dl[k] += ml[k] - l[r][3 * c + k];
            }
            row[c] = make_float2(dot_df(a.M, a.M + 8, dh, dl), dot_df(a.M + 3, a.M + 11, dh, dl));
        }
        put_row<BW, MAPS>(a, ((size_t)f * d.H + row0 + r) * d.W + col0, row, e);
    }
}

// V consecutive detail-part values from offset o (streaming loads).
template <int V>
__device__ __forceinline__ void load_detail(const float2 *det, size_t o, float2 *dp) {
    if constexpr (V == 4) {
        const f32x4 x = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(det + o));
        const f32x4 y = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(det + o + 2));
        dp[0] = make_float2(x.x, x.y);
        dp[1] = make_float2(x.z, x.w);
        dp[2] = make_float2(y.x, y.y);
        dp[3] = make_float2(y.z, y.w);
    } else if constexpr (V == 2) {
        const f32x4 x = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(det + o));
        dp[0] = make_float2(x.x, x.y);
        dp[1] = make_float2(x.z, x.w);
    } else {
        const f32x2 x = __builtin_nontemporal_load(reinterpret_cast<const f32x2 *>(det + o));
        dp[0] = make_float2(x.x, x.y);
    }
}

// ---------------------------------------------------------------------------
// K2: posterior mean over the grid on the low-pass band.
//
// Likelihood in base 2 with scaled coordinates: t_g = -|s z - s mu'_g|^2 with
// s = sqrt(log2(e) / (2 sigma^2)) and mu' centred on mu_ref.  Inside a
// super-tile both the observation r = s z - centre (formed from the
// double-float observation) and the node coordinates v_g are small.
//
// The weights are taken relative to a per-pixel reference m fixed before the
// main loop: m_lo = best logit of one probe node per 8 x 8 patch (a node's
// logit up to rounding, so the top weight is about 1 or more and the sum cannot
// underflow), m_up = best upper bound over the super-tiles' boxes.  If
// m_up - m_lo <= kFarGap for the whole tile, m = m_lo and every weight lies in
// [0, 2^kFarGap]; otherwise the tile first takes the exact maximum over its
// nodes.  Moments are accumulated relative to the super-tile's centre inside a
// super-tile and merged with compensation relative to an anchor: the pixel's
// best probe node (direct kernel), or the centre of the tile's best-bounded
// super-tile (MFMA kernel).  The partial sums of the lanes are combined with
// compensated pairwise steps and the grid splits with Kahan compensation
// (recomposition kernel).
//
// Two kernels share this: k_posterior (MFMA logits, used when every
// super-tile is compact in scaled units) and k_posterior_direct (VALU
// difference form, for grids too coarse for the expanded logit's precision).
// ---------------------------------------------------------------------------
constexpr float kFarGap = 64.0f;

__device__ __forceinline__ void kahan_add(float &s, float &c, float x) {
    const float y = x - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

// s - c += from x L0 + L1, the product's and the sum's rounding errors kept in
// c: moments of a super-tile (L0, L1 about its centre) about an anchor that may
// lie the width of the grid away.
__device__ __forceinline__ void merge_far_moment(float &s, float &c, float from, float L0, float L1) {
#pragma clang fp contract(off)
    const float x = fmaf(from, L0, L1);
    const float xe = fmaf(from, L0, -x) + L1;
    float t, e;
    two_sum(s, x, t, e);
    s = t;
    c -= e + xe;
}

// Lane exchanges on the VALU (no LDS round trip): a DPP move, and the row
// swaps of gfx950.  swap_rows16 exchanges the odd 16-lane rows of a with the
// even rows of b, swap_rows32 the upper half of a with the lower half of b.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ void swap_rows16(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_rows32(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

template <bool MAX>
__device__ __forceinline__ float pick(float a, float b) {
    return MAX ? fmaxf(a, b) : fminf(a, b);
}
// Minimum / maximum over the 16 lanes of a row, every lane gets it.
template <bool MAX>
__device__ __forceinline__ float row_reduce(float x) {
    x = pick<MAX>(x, dpp<0xB1>(x));    // lane ^ 1
    x = pick<MAX>(x, dpp<0x4E>(x));    // lane ^ 2
    x = pick<MAX>(x, dpp<0x141>(x));   // the other quad of eight lanes
    return pick<MAX>(x, dpp<0x140>(x));   // the other eight of the row
}
// Maximum over the four lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ __forceinline__ float max_rows(float x) {
    float y = x;
    swap_rows16(x, y);
    x = y = fmaxf(x, y);
    swap_rows32(x, y);
    return fmaxf(x, y);
}
// Minimum / maximum over the wave (uniform).
__device__ __forceinline__ float lane_value(float x, int lane);
template <bool MAX>
__device__ __forceinline__ float wave_reduce(float x) {
    x = row_reduce<MAX>(x);
    return pick<MAX>(pick<MAX>(lane_value(x, 0), lane_value(x, 16)), pick<MAX>(lane_value(x, 32), lane_value(x, 48)));
}
__device__ __forceinline__ float lane_value(float x, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

__device__ __forceinline__ f32x4 mfma_16x16x32_bf16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Nearest bf16 (ties to even) of lo and hi, packed (lo in the low half).
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// Pixel (B) operand of the split bf16 MFMA.  Lane groups 0..2 carry the
// exact three-part split of u (twice the pixel's coordinate) in the order
// that pairs with the node parts of the split operand table; group 3 carries
// ones that pick up the node's squared-norm parts and the three parts of the
// pixel's constant c = -(|r|^2 + m), paired with node ones.  The parts are
// x1 = bf16(x), x2 = bf16(x - x1), x3 = bf16(x - x1 - x2), each difference
// exact in float32.
__device__ __forceinline__ bf16x8 split_pixel_operand(float u, float c, bool coord) {
    const float x = coord ? u : c;
    const unsigned p11 = pack_bf16(x, x);                        // (x1, x1)
    const float r1 = x - __uint_as_float(p11 << 16);             // x - x1, exact
    const float r2 = r1 - __uint_as_float(pack_bf16(r1, r1) << 16);   // r1 - x2, exact
    const unsigned p23 = pack_bf16(r1, r2);                      // (x2, x3)
    u32x4 b;
    b[0] = coord ? p11 : 0x3f803f80u;                            // (x1, x1) or (1, 1)
    b[1] = pack_bf16(coord ? r1 : 1.0f, x);                      // (x2, x1) or (1, x1)
    b[2] = p23;                                                  // (x2, x3)
    b[3] = coord ? p23 : 0u;                                     // (x2, x3) or (0, 0)
    return __builtin_bit_cast(bf16x8, b);
}


constexpr int kXcds = 8;   // accelerator complex dies of an MI355X, each with its own L2
// Waves resident at once: 256 CUs x 4 SIMDs x 6 waves.
constexpr int kResidentWaves = 256 * 4 * 6;

// Lowest set bit (-1: none) and the mask without bit c, one scalar
// instruction each.
__device__ __forceinline__ int lowest_bit(unsigned long long m) {
    int c;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(c) : "s"(m));
    return c;
}
__device__ __forceinline__ unsigned long long clear_bit(unsigned long long m, int c) {
    asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(c));
    return m;
}

struct WaveWork {
    int f, split, s0, s1;
    int r0, c0;  // origin of the wave's tile (of the workgroup's region) in LL pixels
};

// (p, pe) = r^2 exactly (product and its FMA residual) if sq, else (m, 0).
__device__ __forceinline__ void square_or(float r, float m, bool sq, float &p, float &pe) {
#pragma clang fp contract(off)
    const float rr = r * r;
    p = sq ? rr : m;
    pe = sq ? fmaf(r, r, -rr) : 0.0f;
}

// Renumbered workgroup.  Workgroups are dealt to the 8 XCDs in turn; each XCD
// takes runs of 2^run_log2 neighbouring blocks in turn (run_log2 = 0: one
// contiguous eighth of the launch), since neighbouring pixels keep overlapping
// chunks, which then stay in that XCD's L2.  Workgroups past the last whole
// round of runs keep their numbers.  A launch whose workgroups are all resident
// at once keeps the plain numbering: interleaved blocks spread the frame's
// costly regions over all eight.
__device__ __forceinline__ int xcd_order(int bid, int n, int resident, int run_log2) {
    if (n <= resident) return bid;
    if (run_log2 == 0) {
        const int per_xcd = n / kXcds;
        return bid < per_xcd * kXcds ? (bid % kXcds) * per_xcd + bid / kXcds : bid;
    }
    if (bid >= n / kXcds >> run_log2 << run_log2 << 3) return bid;
    const int j = bid / kXcds, run = j >> run_log2;
    return ((run * kXcds + bid % kXcds) << run_log2) + (j - (run << run_log2));
}

// Block number idx of BW x BH LL pixels (and its grid split).  Blocks go in
// squares of kOrderSquare x kOrderSquare (bands of that many block rows,
// squares left to right, row-major inside a square): the workgroups an XCD runs
// at once then cover a compact part of the frame.  Divisions by the launch's
// numbers are products: as divisions they took some 500 scalar instructions at
// the start of every wave, where it has no load in flight yet.
template <int BW, int BH>
__device__ __forceinline__ WaveWork block_work(const PosteriorArgs &a, int idx) {
    WaveWork w;
    const BlockOrder &o = a.order;
    int chunk = idx;
    w.split = 0;
    if (a.split > 1) {
        chunk = o.split.divide(idx);
        w.split = idx - chunk * a.split;
    }
    w.f = o.frame.divide(chunk);
    const int t = chunk - w.f * o.frame.d;
    const int band = o.band.divide(t), in_band = t - band * o.band.d;
    const bool low = band == o.low_band;            // the last band, with fewer rows
    const int square = kOrderSquare * (low ? o.low_rows : kOrderSquare);
    int br, bc;
    if (in_band < o.full * square) {
        const int sq = low ? o.low_square.divide(in_band) : in_band / (kOrderSquare * kOrderSquare);
        const int in = in_band - sq * square;
        br = in / kOrderSquare;
        bc = sq * kOrderSquare + in % kOrderSquare;
    } else {
        const int in = in_band - o.full * square;
        br = o.rest.divide(in);
        bc = o.full * kOrderSquare + in - br * o.rest.d;
    }
    w.r0 = (band * kOrderSquare + br) * BH;
    w.c0 = bc * BW;
    w.s0 = 0;
    w.s1 = a.n_supers;
    if (a.split > 1) {
        w.s0 = (int)((long long)a.n_supers * w.split / a.split);
        w.s1 = (int)((long long)a.n_supers * (w.split + 1) / a.split);
    }
    return w;
}

// LL index of pixel i of the workgroup's region, RW pixels wide.
template <int RW>
__device__ __forceinline__ long long region_pixel(const PosteriorArgs &a, const WaveWork &w, int i) {
    return (long long)(w.r0 + i / RW) * a.wl + w.c0 + i % RW;
}

// Scaled double-float observation of LL pixel p, channel k.
__device__ __forceinline__ void load_obs(const float *zf, long long LL, long long p, int k, float sc,
                                         float &h, float &l) {
    const float zh = zf[k * LL + p], zl = zf[(3 + k) * LL + p];
    h = sc * zh;
    l = fmaf(sc, zh, -h) + sc * zl;
}

// A table that no kernel writes, in the constant address space: reads at a
// wave-uniform index are scalar loads wherever they stand (behind a fence or
// a store the compiler would make vector loads of them).
typedef const __attribute__((address_space(4))) float ConstFloat;
__device__ __forceinline__ ConstFloat *constant(const float *p) { return (ConstFloat *)(uintptr_t)p; }

template <typename Table>
__device__ __forceinline__ void recentre(Table T, const float ph[3], const float pl[3], float r[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) r[k] = (ph[k] - T[k]) + (pl[k] - T[3 + k]);
}

// Upper bound of the logit over an axis-aligned box [lo, hi] (6 floats).
__device__ __forceinline__ float box_bound(const float *box, const float r[3]) {
    const float e0 = fmaxf(fmaxf(box[0] - r[0], r[0] - box[3]), 0.0f);
    const float e1 = fmaxf(fmaxf(box[1] - r[1], r[1] - box[4]), 0.0f);
    const float e2 = fmaxf(fmaxf(box[2] - r[2], r[2] - box[5]), 0.0f);
    return -fmaf(e0, e0, fmaf(e1, e1, e2 * e2));
}

// Upper bound of the logit between two boxes (6 floats each: lo[3], hi[3]).
__device__ __forceinline__ float box_box_bound(const float *box, const float r[6]) {
    const float e0 = fmaxf(fmaxf(box[0] - r[3], r[0] - box[3]), 0.0f);
    const float e1 = fmaxf(fmaxf(box[1] - r[4], r[1] - box[4]), 0.0f);
    const float e2 = fmaxf(fmaxf(box[2] - r[5], r[2] - box[5]), 0.0f);
    return -fmaf(e0, e0, fmaf(e1, e1, e2 * e2));
}

// Skipped weight of a chunk whose logits lie at most v above the wave's
// reference, rounded up, in units of 2^-mass_log2.  What is skipped lies below
// the first depth: at most 2^(kMassDepthLog2 + kChunkNodesLog2) + 1 units.
__device__ __forceinline__ unsigned mass_units(float v, float mass_log2) {
    constexpr float kMost = kMassDepthLog2 + kChunkNodesLog2;
    return (unsigned)__builtin_amdgcn_exp2f(fminf(v + (mass_log2 + kChunkNodesLog2), kMost)) + 1u;
}
// Whether the skipped weight `mass` (relative to mmin) is too large for a pixel
// whose sums hold 2^held; a count that has saturated is no bound.
__device__ __forceinline__ bool certificate_fails(const PosteriorArgs &a, unsigned mass, float held, float mmin) {
    return mass == ~0u || __log2f((float)mass) - a.mass_log2 > a.cert_log2 + (held - mmin);
}

// Widening of the wave's observation box for rounding (scaled units).
constexpr float kBoxSlack = 1.0e-3f;

// Coordinate of an observation along one of the boxes' axes.
__device__ __forceinline__ float axis_coordinate(const float axis[3], float x0, float x1, float x2) {
    return fmaf(axis[0], x0, fmaf(axis[1], x1, axis[2] * x2));
}

// Widens an observation box for rounding (of the rotation too, at the scale
// of the observation: far2 its squared distance from the origin).
__device__ __forceinline__ void widen_box(float zbox[6], float far2) {
    const float slack = kBoxSlack + sqrtf(far2) * 0x1p-20f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        zbox[k] -= slack;
        zbox[3 + k] += slack;
    }
}

// Best probe of super-tile T for observation r (recentred on T): updates the
// running best logit and its anchor node.
template <typename Table>
__device__ __forceinline__ void probe_supertile(Table T, const float r[3], float &mlo, float &ahb, float &aox) {
    const int np = __float_as_int(T[14]);
    for (int i = 0; i < np; ++i) {
        const auto P = T + kSupHdr + i * kProbeFloats;
        const float d0 = r[0] - P[0], d1 = r[1] - P[1], d2 = r[2] - P[2];
        const float tp = -fmaf(d0, d0, fmaf(d1, d1, d2 * d2));
        if (tp > mlo) {
            mlo = tp;
            ahb = P[3];
            aox = P[4];
        }
    }
}

// Global reference for split grids: one lane per LL pixel, the best probe
// logit over all super-tiles (the same search as above without the split).
// Each split then skips against max(own reference, global reference), so a
// split far from the pixel's posterior skips against the posterior's peak.
__global__ __launch_bounds__(kBlockThreads) void k_reference(PosteriorArgs a) {
    const long long i = (long long)blockIdx.x * kBlockThreads + threadIdx.x;
    if (i >= (long long)a.n_frames * a.LL) return;
    const long long f = i / a.LL, p = i - f * a.LL;
    const float *zf = a.z + (size_t)f * 6 * a.LL;
    float ph[3], pl[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) load_obs(zf, a.LL, p, k, a.scale, ph[k], pl[k]);
    float mlo = -INFINITY, mup = -INFINITY, ahb = 0.0f, aox = 0.0f;
    int best = 0;
    for (int si = 0; si < a.n_supers; ++si) {
        const float *__restrict__ T = a.supers + (size_t)si * a.super_stride;
        float r[3];
        recentre(T, ph, pl, r);
        const float ub = box_bound(T + 8, r);
        if (ub > mup) {
            mup = ub;
            best = si;
        }
    }
    {
        const float *__restrict__ T = a.supers + (size_t)best * a.super_stride;
        float r[3];
        recentre(T, ph, pl, r);
        probe_supertile(T, r, mlo, ahb, aox);
    }
    for (int si = 0; si < a.n_supers; ++si) {
        const float *__restrict__ T = a.supers + (size_t)si * a.super_stride;
        float r[3];
        recentre(T, ph, pl, r);
        if (si != best && box_bound(T + 8, r) > mlo) probe_supertile(T, r, mlo, ahb, aox);
    }
    a.gref[i] = mlo;
}

// Exact maximum logit over the nodes of the chunks a wave may keep, difference
// form; each pixel's LPP lanes split every chunk's nodes.  super_test(si) and
// chunk_test(si, c) are the bounds of the main loop's own tests (one
// super-tile or chunk per lane): a chunk that the loop evaluates but this scan
// leaves out could hold weights that overflow relative to the result.
// The NW waves of a tile take the super-tiles in turn.  Returns the maximum of
// cur and of the wave's share.
template <int PW, int LPP, int NW, typename SuperTest, typename ChunkTest>
__device__ float far_gap_max(const PosteriorArgs &a, const WaveWork &w, const float ph[3], const float pl[3],
                             int part, int wave, SuperTest super_test, ChunkTest chunk_test, float mmin, float cur) {
    const int lane = threadIdx.x & 63;
    const float nskip = -a.skip_log2;
    float mx = cur;
    int turn = 0;
    for (int g = w.s0; g < w.s1; g += 64) {
        const int sl = g + lane;
        unsigned long long smask = __ballot(sl < w.s1 && super_test(sl) - mmin > nskip);
        while (smask) {
            const int si = g + __builtin_ctzll(smask);
            smask &= smask - 1;
            if (NW > 1 && turn++ % NW != wave) continue;
            const float *__restrict__ T = a.supers + (size_t)si * a.super_stride;
            float r[3];
            recentre(T, ph, pl, r);
            const float *__restrict__ C0 = T + kSupHdr + kMaxProbes * kProbeFloats;
            for (int cg = 0; cg < a.chunks_per_super; cg += 64) {
                const int ct = min(cg + lane, a.chunks_per_super - 1);
                unsigned long long mask =
                    __ballot(cg + lane < a.chunks_per_super && chunk_test(si, ct) - mmin > nskip);
                while (mask) {
                    const float *__restrict__ C = C0 + (size_t)(cg + __builtin_ctzll(mask)) * kChunkFloats;
                    mask &= mask - 1;
                    for (int j = part; j < kChunkNodes; j += LPP) {
                        const float d0 = r[0] - C[j], d1 = r[1] - C[16 + j], d2 = r[2] - C[32 + j];
                        mx = fmaxf(mx, -fmaf(d0, d0, fmaf(d1, d1, d2 * d2)));
                    }
                }
            }
        }
    }
#pragma unroll
    for (int o = PW; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    return mx;
}

// Fused recomposition for one split and n <= 3, in units of V pixels along a
// row, from the estimates of the region's pixels: the maps of the whole region
// of RW x RH LL pixels, or (LIST) those of `count` listed ones, by thread `thread`
// of `threads`.
template <int RW, int RH, bool LIST, int V>
__device__ __forceinline__ void fused_maps(const PosteriorArgs &a, const WaveWork &w, const float2 *est, int thread,
                                           int threads, const int *list, int count) {
    constexpr int kLogV = V == 4 ? 2 : (V == 2 ? 1 : 0);
    const int n = a.levels, B = 1 << n;
    const int n_units = ((LIST ? count : RW * RH) << 2 * n) >> kLogV;
    for (int u = thread; u < n_units; u += threads) {
        int i, y, x;   // pixel of the region, offset in its block
        if constexpr (LIST) {
            const int o = u & ((1 << (2 * n - kLogV)) - 1);
            i = list[u >> (2 * n - kLogV)];
            y = o >> (n - kLogV);
            x = (o << kLogV) & (B - 1);
        } else {
            const int row_shift = 4 + n - kLogV;   // log2 of the units of a region row
            static_assert(RW == 16, "row_shift");
            const int Y = u >> row_shift, X = (u << kLogV) & ((RW << n) - 1);
            i = (Y >> n) * RW + (X >> n);
            y = Y & (B - 1);
            x = X & (B - 1);
        }
        const int gr = w.r0 + i / RW, gc = w.c0 + i % RW;
        if (gr >= a.hl || gc >= a.wl) continue;
        const size_t o = ((size_t)w.f * a.H + ((size_t)gr << n) + y) * a.W + ((size_t)gc << n) + x;
        float2 dp[V];
        load_detail<V>(a.det, o, dp);
        write_maps<V>(a.hb, a.hbo2, a.thb, a.so2, a.thb_eps, o, est[i], dp);
    }
}
template <int RW, int RH, bool LIST>
__device__ __forceinline__ void fused_maps(const PosteriorArgs &a, const WaveWork &w, const float2 *est, int thread,
                                           int threads, const int *list = nullptr, int count = 0) {
    switch (a.vec) {
        case 4: fused_maps<RW, RH, LIST, 4>(a, w, est, thread, threads, list, count); break;
        case 2: fused_maps<RW, RH, LIST, 2>(a, w, est, thread, threads, list, count); break;
        default: fused_maps<RW, RH, LIST, 1>(a, w, est, thread, threads, list, count); break;
    }
}

// Logit minus the reference, nm - |r - v_j|^2 (nm = -m), with r and node j's
// coordinates v_j = C + LO held as double-floats: the differences, their
// squares and the sum carry their rounding errors, and the result is
// returned as a double-float (high part returned, low part in tl), so the
// weight exp2(t) (1 + tl ln 2) is free of the logit's float32 rounding too
// (a float32 difference form rounds at the scale of |r| and |v_j| instead,
// which coarse grids make large; on grids with very few nodes even the
// rounding of the logit itself, at a scale of tens of units, moves a
// posterior mean between two distant nodes by up to 1e-4 uM).
__device__ __forceinline__ float df_logit_v(const float rh[3], const float rl[3], const float vh[3],
                                            const float vl[3], float nm, float &tl) {
#pragma clang fp contract(off)
    float sh = 0.0f, sl = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        float dh, e;
        two_sum(rh[k], -vh[k], dh, e);
        const float dl = e + (rl[k] - vl[k]);
        const float q = dh * dh;
        const float qe = fmaf(2.0f * dh, dl, fmaf(dh, dh, -q));
        float s, es;
        two_sum(sh, q, s, es);
        sh = s;
        sl += es + qe;
    }
    float th, e;
    two_sum(nm, -sh, th, e);
    tl = e - sl;
    return th;
}

template <typename Table>
__device__ __forceinline__ float df_logit(const float rh[3], const float rl[3], Table C, Table LO, int j, float nm,
                                          float &tl) {
    const float vh[3] = {C[j], C[16 + j], C[32 + j]}, vl[3] = {LO[j], LO[16 + j], LO[32 + j]};
    return df_logit_v(rh, rl, vh, vl, nm, tl);
}

// The same pointer, hidden from the optimiser: loads through it are issued
// where they are written instead of being merged with earlier ones.
template <typename P>
__device__ __forceinline__ P *opaque(P *p) {
    asm volatile("" : "+s"(p));
    return p;
}

// The kernel's argument as it lies in the argument segment (address space 4).
using KernArgs = const __attribute__((address_space(4))) PosteriorArgs;

// The fields the far-pixel pass reads, loaded from the argument segment.
__device__ __forceinline__ PosteriorArgs far_args(KernArgs *k) {
    PosteriorArgs f{};
    f.LL = k->LL;
    f.hl = k->hl;
    f.wl = k->wl;
    f.z = k->z;
    f.scale = k->scale;
    f.gref = k->gref;
    f.far_rho2 = k->far_rho2;
    f.skip_log2 = k->skip_log2;
    f.supers = k->supers;
    f.super_stride = k->super_stride;
    f.chunks_per_super = k->chunks_per_super;
    f.lo = k->lo;
    f.headers = k->headers;
    f.boxes = k->boxes;
    for (int i = 0; i < 9; ++i) f.axes[i] = k->axes[i];
    for (int i = 0; i < 3; ++i) f.origin[i] = k->origin[i];
    return f;
}

// A lane value the optimiser cannot trace back (it is formed again where used).
__device__ __forceinline__ int opaque_v(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Posterior sums of one pixel over the wave's split with double-float logits
// (as the precise direct kernel forms them), for observations too far from the
// grid's surface for the MFMA kernel's expanded logit.  The whole wave works
// on the pixel: super-tiles one after another, lane l on node l % 16 of
// chunks l / 16, l / 16 + 4, ...  Skipping is the hard rule against the
// pixel's own reference m_skip (no budget band); nm = -m is the logit
// reference of the sums.  Returns the sums S0, S1, S2 about the anchors and
// their low parts E on every lane.
__device__ __forceinline__ void far_pixel_sums(const PosteriorArgs &a, const WaveWork &w, const float qh[3],
                                               const float ql[3], float m_skip, float nm, float anc_hb,
                                               float anc_ox, float S[3], float E[3]) {
    const int lane = threadIdx.x & 63;
    const int j = lane & 15;
    const float nskip = -a.skip_log2;
    // The boxes and slack of the main loop's tests: what is evaluated here is
    // then among the chunks that the pixel's reference was refined over.
    float zbox[6], far2 = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        zbox[k] = zbox[3 + k] = axis_coordinate(a.axes + 3 * k, (qh[0] - a.origin[0]) + ql[0],
                                                (qh[1] - a.origin[1]) + ql[1], (qh[2] - a.origin[2]) + ql[2]);
        far2 = fmaf(zbox[k], zbox[k], far2);
    }
    widen_box(zbox, far2);
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
    for (int si = w.s0; si < w.s1; ++si) {
        if (!(box_box_bound(a.headers + (size_t)si * kHdrFloats, zbox) - m_skip > nskip)) continue;
        const float *__restrict__ T = a.supers + (size_t)si * a.super_stride;
        float rh[3], rl[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            float sk, e;
            two_sum(qh[k], -T[k], sk, e);
            fast_two_sum(sk, e + (ql[k] - T[3 + k]), rh[k], rl[k]);
        }
        const float *__restrict__ C0 = T + kSupHdr + kMaxProbes * kProbeFloats;
        const float *__restrict__ LO0 = a.lo + (size_t)si * a.chunks_per_super * kLoFloats;
        float L0 = 0.f, L1 = 0.f, L2 = 0.f;
        for (int ci = lane >> 4; ci < a.chunks_per_super; ci += 4) {
            const float *__restrict__ C = C0 + (size_t)ci * kChunkFloats;
            if (box_box_bound(a.boxes + ((size_t)si * a.chunks_per_super + ci) * kBoxFloats, zbox) - m_skip > nskip) {
                float tl;
                const float th = df_logit(rh, rl, C, LO0 + (size_t)ci * kLoFloats, j, nm, tl);
                const float e = __builtin_amdgcn_exp2f(th);
                const float wt = fmaf(e, tl * 0.6931471805599453f, e);
                L0 += wt;
                L1 = fmaf(wt, C[64 + j], L1);
                L2 = fmaf(wt, C[80 + j], L2);
            }
        }
        kahan_add(s0, c0, L0);
        merge_far_moment(s1, c1, T[6] - anc_hb, L0, L1);
        merge_far_moment(s2, c2, T[7] - anc_ox, L0, L2);
    }
    // Sum over the 64 lanes, each pairwise step carrying its rounding error.
    float x[3] = {s0, s1, s2}, e[3] = {-c0, -c1, -c2};
#pragma unroll
    for (int o = 1; o <= 32; o <<= 1)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float y = __shfl_xor(x[k], o), ye = __shfl_xor(e[k], o);
            float t, err;
            two_sum(x[k], y, t, err);
            x[k] = t;
            e[k] = (e[k] + ye) + err;
        }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        S[k] = x[k];
        E[k] = e[k];
    }
}

// MFMA kernel: NW waves take a tile of 32 LL pixels, two blocks of 16; a
// workgroup takes RT tiles of a region of 128 pixels (all four, or one).  Per
// super-tile, 16-node chunk and pixel block one v_mfma_f32_16x16x32_bf16 forms
// the 16 x 16 logits
//   t - m = [v_g, -|v_g|^2, 1] . [2 r, 1, -(|r|^2 + m)]
// (nodes as rows, pixels as columns) from exact three-part bf16 splits of the
// FP32 operands: every product except the smallest (u3 v3), in half the
// cycles of the FP32 16x16x4 MFMA.  The node operand (1 KB per chunk) is
// loaded once for both blocks.  Each lane then holds 1 pixel x the 4
// nodes of one chunk row (lane l: pixel l % 16, THb row l / 16, SO2 offsets
// 0..3) and runs the exponentials and the moments on the VALU.
//
// The tile's reference, its chunk tests and its kept chunks are shared out
// between its waves; what is kept, the segments and their sums are the same
// for any NW and RT.  DFC: the pixel operand's constant |r|^2 + m summed as a
// double-float (plans near the precision budget).
//
// Bound by VALU issue: 94 to 99% busy on sixteen 1080p frames (256 x 256 grid),
// 14 instructions (one MFMA and four exponentials among them) per 256 pairs and
// about 3000 per tile around them (12850 in all).  Six waves per SIMD (80
// VGPRs; ten registers are spilled, outside the chunk loop, which every wave
// writes once: a quarter of the kernel's HBM writes).  Times a call with tiles of 8 x 4
// neighbours and boxes along the channels -> tiles of like observations and
// boxes along the nodes' axes: sixteen 1080p frames 2274 -> 1976 us, 1280x1024
// pair on a 512 x 512 grid 2794 -> 2470, 1280x1024 frame at level 0 with the
// illumination term 1198 -> 1049, sixteen 320x240 frames 205 -> 165, one
// 640x480 frame 85 -> 72.  What a wave does before its first chunk is a chain
// of latencies: the bounds of the first 64 super-tiles are formed once and kept
// in LDS, the next probe operand is fetched while one is evaluated and the
// block's place takes no division: a 64x64 frame 25.0 -> 24.3 us a call, one
// 1080p frame 180 -> 178, a 3840x2160 frame 223 -> 221.

// Order between the lanes of a tile: of its only wave, or of the workgroup.
template <int NW>
__device__ __forceinline__ void tile_sync() {
    if constexpr (NW == 1) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

struct KeptSuper {
    unsigned lo, hi;   // kept chunks of the super-tile, one bit each
    int si, segment;
};

// Lists up to 64 super-tiles from g on whose bound (relative to mmin) exceeds
// svlo, and the chunks of each whose bound v has vlo < v <= vhi; what lies
// below counts into `mass`.  The NW waves of a tile share the chunk tests:
// 64 / chunks_per_super super-tiles at once, lane sub * cps + ci chunk ci of
// the sub-th.  `bound` holds the bounds of the split's first 64 super-tiles.
// Returns the length of the list.  The caller orders the waves before the list
// is read.
struct ChunkTest {
    float vlo, vhi, svlo, mmin;
    bool last;   // nothing below counts
};
template <int NW>
__device__ __forceinline__ int list_chunks(const PosteriorArgs &a, const WaveWork &w, KeptSuper *kept,
                                           const float *bound, int wave, const float (&zbox)[6], const ChunkTest &t,
                                           int &g, unsigned &mass) {
    const int lane = threadIdx.x & 63;
    const int cps = a.chunks_per_super, per_test = a.supers_per_test;
    const int sub = (int)((unsigned)lane * (unsigned)a.inv_chunks >> 16), ci = lane - sub * cps;   // lane / cps
    const unsigned long long chunk_bits = cps >= 64 ? ~0ull : (1ull << cps) - 1;
    // Super-tiles, one per lane; the kept ones are listed.
    int K = 0;
    while (g < w.s1) {
        const int sl = g + lane;
        float sv = -INFINITY;
        if (g == w.s0)
            sv = bound[lane];
        else if (sl < w.s1)
            sv = box_box_bound(a.headers + (size_t)sl * kHdrFloats, zbox);
        sv -= t.mmin;
        const unsigned long long smask = __builtin_amdgcn_ballot_w64(sv > t.svlo);
        const int n = __popcll(smask);
        // the list holds 64; exact and no skipping take the same windows
        if (K + n > 64 || (K > 0 && !a.list_across)) break;
        if (!t.last && (NW == 1 || wave == 0) && sl < w.s1 && !(sv > t.svlo))
            mass = __builtin_elementwise_add_sat(mass, mass_units(sv, a.mass_log2) * (unsigned)cps);
        const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(smask >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((unsigned)smask, 0));
        if (sv > t.svlo) {   // every wave writes the same values
            kept[K + rank].si = sl;
            kept[K + rank].segment = __float_as_int(a.headers[(size_t)sl * kHdrFloats + 14]);
        }
        K += n;
        g += 64;
    }
    if (K == 0) return 0;
    tile_sync<1>();   // between the lanes of each wave, which has listed them itself
    for (int k0 = wave * per_test; k0 < K; k0 += NW * per_test) {
        const int k = k0 + sub;
        const bool real = sub < per_test && k < K;
        const int si = kept[real ? k : 0].si;
        const float v = box_box_bound(a.boxes + ((size_t)si * cps + ci) * kBoxFloats, zbox) - t.mmin;
        const unsigned long long in = __builtin_amdgcn_ballot_w64(real && v > t.vlo && v <= t.vhi);
        if (!t.last) mass = __builtin_elementwise_add_sat(mass, real && !(v > t.vlo) ? mass_units(v, a.mass_log2) : 0u);
        if (real && ci == 0) {
            const unsigned long long bits = in >> (sub * cps) & chunk_bits;
            kept[k].lo = (unsigned)bits;
            kept[k].hi = (unsigned)(bits >> 32);
        }
    }
    return K;
}

template <int NW>
struct TileShared {
    KeptSuper kept[64];
    float bound[64];               // of the split's first 64 super-tiles
    float total[6][kTilePixels];   // S0, S1, S2 and their compensation, per pixel
    // several waves: sums of the segments, best probes, skipped weights
    float part[NW > 1 ? kSegments : 1][6][NW > 1 ? kTilePixels : 1];
    float best[NW][NW > 1 ? kTilePixels : 1];
    float top[NW][NW > 1 ? kTilePixels : 1];   // each wave's share of far_gap_max
    unsigned mass[NW];
};

template <int NW, int RT>
struct RegionShared {
    TileShared<NW> tile[RT];
    float obs[6][kRegionPixels];        // scaled observation, high and low parts
    float rot[3][kRegionPixels];        // the same along the boxes' axes
    unsigned key[kRegionPixels];
    int rank[kRegionPixels];
    int slot[kRegionPixels];            // pixel of the region at each rank
    float2 est[kRegionPixels];
    int more[3];
};

// base + n / d with n = nh + nl and d = dh + dl, rounded once.
__device__ __forceinline__ float plus_quotient(float base, float nh, float nl, float dh, float dl) {
    const float q = nh / dh;
    float s, e;
    two_sum(base, q, s, e);
    return s + (e + (fmaf(-q, dh, nh) + fmaf(-q, dl, nl)) / dh);
}

template <int NW, int RT, bool DFC>
__global__ __launch_bounds__(64 * NW * RT) __attribute__((amdgpu_waves_per_eu(6))) void k_posterior(PosteriorArgs a) {
    constexpr int PB = kTilePixels / 16;
    __shared__ RegionShared<NW, RT> rsh;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wave = wid % NW;   // of its tile
    const int lp = lane & 15, lk = lane >> 4;
    const int bid = xcd_order(blockIdx.x, gridDim.x, kResidentWaves / (NW * RT), a.run_log2);
    const int tile = RT == 1 ? bid % kRegionTiles : wid / NW;   // of its region
    const WaveWork w = block_work<kRegionW, kRegionH>(a, RT == 1 ? bid / kRegionTiles : bid);
    TileShared<NW> &sh = rsh.tile[RT == 1 ? 0 : tile];
    // Pixels of the region ranked by their observation's coordinate along the
    // direction in which the nodes spread most; a tile takes 32 consecutive
    // ranks.  Its observations then lie closer together than those of 8 x 4
    // neighbours, whose noise spreads them, and their common box keeps fewer
    // chunks (sixteen 1080p frames: 8.3% of the pairs, with the boxes' axes,
    // instead of 9.8%).  Regions of 256 pixels would keep 3% fewer still, but
    // four waves a tile would not fit in one workgroup.  Ranks are counted: the
    // threads share the comparisons.
    const int rows = min(kRegionH, a.hl - w.r0), cols = min(kRegionW, a.wl - w.c0);
    const int n_valid = rows * cols;
    // A region of one tile (small low-pass bands) has nothing to rank: its pixels
    // in order, by the tile's own waves.  Waves that end here or below are not
    // counted by the workgroup's later barriers.  While they stayed, three
    // quarters of the waves of 4096 frames of 8 x 4 pixels idled: 163 us a call.
    const bool single = n_valid <= kTilePixels;
    if (single && tile > 0 && (RT == 1 || NW == 1)) return;
    {
        int i = threadIdx.x % kRegionPixels;
        const int part = threadIdx.x / kRegionPixels;
        constexpr int kParts = 64 * NW * RT / kRegionPixels, kKeys = kRegionPixels / kParts;
        if (single) i = i / cols * kRegionW + i % cols;
        if (single ? (int)threadIdx.x < n_valid : part == 0) {
            const int r = i / kRegionW, c = i % kRegionW;
            const bool inside = r < rows && c < cols;
            const long long p = (long long)(w.r0 + min(r, rows - 1)) * a.wl + w.c0 + min(c, cols - 1);
            const float *zf = a.z + (size_t)w.f * 6 * a.LL;
            float x[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                float h, l;
                load_obs(zf, a.LL, p, k, a.scale, h, l);
                rsh.obs[k][i] = h;
                rsh.obs[3 + k][i] = l;
                x[k] = (h - a.origin[k]) + l;
            }
            float q = 0.0f;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                q = axis_coordinate(a.axes + 3 * k, x[0], x[1], x[2]);
                rsh.rot[k][i] = q;
            }
            // ordered bits, the low seven replaced by the pixel's number; pixels
            // outside the frame last
            const unsigned u = __float_as_uint(q == q ? q : INFINITY);
            const unsigned ordered = u & 0x80000000u ? ~u : u | 0x80000000u;
            rsh.key[i] = (inside ? ordered & ~127u : 0xffffff80u) | (unsigned)i;
            rsh.rank[i] = 0;
            if (single) rsh.slot[threadIdx.x] = i;
        }
        for (int t = 64 * wave + lane; t < 6 * kTilePixels; t += 64 * NW) (&sh.total[0][0])[t] = 0.0f;
        if (threadIdx.x < 3) rsh.more[threadIdx.x] = 0;
        __syncthreads();
        if (!single) {
            const unsigned own = rsh.key[i];
            int rank = 0;
#pragma unroll 4
            for (int t = 0; t < kKeys; ++t) rank += rsh.key[part * kKeys + t] < own ? 1 : 0;
            atomicAdd(&rsh.rank[i], rank);
            __syncthreads();
            if (part == 0) rsh.slot[rsh.rank[i]] = i;
            __syncthreads();
        }
    }
    // A tile past the frame's pixels has nothing to do; a partial one repeats
    // its first pixel.
    const int base = tile * kTilePixels;
    bool active = base < n_valid;
    if ((RT == 1 || NW == 1) && !active) return;
    int ib[PB];   // region pixel b*16 + lp of the tile
    float ah[PB], al[PB];   // lane (lp, lk) holds its coordinate lk (lk == 3 repeats coordinate 0)
#pragma unroll
    for (int b = 0; b < PB; ++b) {
        const int q = base + b * 16 + lp;
        ib[b] = rsh.slot[q < n_valid ? q : (active ? base : 0)];
        ah[b] = rsh.obs[lk < 3 ? lk : 0][ib[b]];
        al[b] = rsh.obs[3 + (lk < 3 ? lk : 0)][ib[b]];
    }
    // Observation box of the tile along the boxes' axes, widened for rounding.
    float zbox[6], far2 = 0.0f;
    {
        const float x0 = rsh.rot[lk < 3 ? lk : 0][ib[0]], x1 = rsh.rot[lk < 3 ? lk : 0][ib[1]];
        const float lo = row_reduce<false>(fminf(x0, x1)), hi = row_reduce<true>(fmaxf(x0, x1));
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            zbox[k] = lane_value(lo, 16 * k);
            zbox[3 + k] = lane_value(hi, 16 * k);
            const float e = fmaxf(-zbox[k], zbox[3 + k]);
            far2 = fmaf(e, e, far2);
        }
        widen_box(zbox, far2);
    }
    auto super_bound = [&](int si) {   // -inf past the split's range
        return si < w.s1 ? box_box_bound(a.headers + (size_t)si * kHdrFloats, zbox) : -INFINITY;
    };
    // Pixel operands (the MFMA B operands) of both blocks from their
    // coordinates r (lane groups lk < 3) and m: c = -(|r|^2 + m), formed over
    // the pixel's four lanes, is wanted by its lane of group 3 only.
    auto pixel_operands = [&](const float (&r)[PB], const float (&m)[PB], auto dfc, bf16x8 (&av)[PB]) {
        float c0, c1;
        if constexpr (decltype(dfc)::value) {
            // as a double-float (plans near the precision budget)
            float p, pe, q, qe;
            square_or(r[0], m[0], lk < 3, p, pe);
            square_or(r[1], m[1], lk < 3, q, qe);
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                if (o == 0) {
                    swap_rows16(p, q);
                    swap_rows16(pe, qe);
                } else {
                    swap_rows32(p, q);
                    swap_rows32(pe, qe);
                }
                float t, e;
                two_sum(p, q, t, e);
                p = q = t;
                pe = qe = (pe + qe) + e;
            }
            c0 = c1 = -(p + pe);
        } else {
            float p = lk < 3 ? r[0] * r[0] : m[0], q = lk < 3 ? r[1] * r[1] : m[1];
            swap_rows16(p, q);   // rows: block 0 of rows 0 + 1, block 1 of rows 0 + 1, then of rows 2 + 3
            p = q = p + q;
            swap_rows32(p, q);
            c0 = c1 = -(p + q);   // rows: block 0, 1, 0, 1
        }
        swap_rows16(c0, c1);      // block 0 on every row, block 1 on every row
        av[0] = split_pixel_operand(2.0f * r[0], c0, lk < 3);
        av[1] = split_pixel_operand(2.0f * r[1], c1, lk < 3);
    };
    const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};

    // Reference: each pixel's best probe (one node per 8 x 8 patch) over the
    // split's super-tiles.  The super-tile with the highest bound is probed
    // first, then those bounded above the tile's lowest best probe: the
    // result equals a scan of every probe.  The probes' logits come from MFMAs
    // on split operands, 16 probes at once, in coordinates about the grid's
    // middle: they round at the scale of 2^-22 of the squared distance from it,
    // which the reference may (every weight is formed relative to the same m, and
    // the skip tests allow for far2 2^-20).
    float mup = -INFINITY;   // upper bound of every logit of the split
    int best = w.s0;
    for (int g = w.s0; g < w.s1; g += 64) {
        const float b = super_bound(g + lane);
        if (g == w.s0) sh.bound[lane] = b;   // every wave writes the same values
        const float r = row_reduce<true>(b);
        const float top = fmaxf(fmaxf(lane_value(r, 0), lane_value(r, 16)), fmaxf(lane_value(r, 32), lane_value(r, 48)));
        if (top > mup) {
            mup = top;
            best = g + __builtin_ctzll(__builtin_amdgcn_ballot_w64(b == top) | (1ull << 63));
        }
    }
    best = __builtin_amdgcn_readfirstlane(best);
    tile_sync<1>();   // each wave reads what it has written itself
    auto super_bound_of = [&](int g) { return g == w.s0 ? sh.bound[lane] : super_bound(g + lane); };
    float am[PB] = {-INFINITY, -INFINITY};   // reference of pixel b*16 + lp
    {
        bf16x8 pv[PB];
        const float o = lk == 1 ? a.origin[1] : (lk == 2 ? a.origin[2] : a.origin[0]);
        const float x[PB] = {(ah[0] - o) + al[0], (ah[1] - o) + al[1]}, none[PB] = {0.0f, 0.0f};
        pixel_operands(x, none, std::false_type{}, pv);
        const int shift = 4 - a.probe_shift;   // log2 of the super-tiles of one probe operand
        auto operand = [&](int blk) { return reinterpret_cast<const bf16x8 *>(a.probes)[(size_t)blk * 64 + lane]; };
        auto probe = [&](int blk, const bf16x8 &v) {
#pragma unroll
            for (int b = 0; b < PB; ++b) {
                f32x4 d = mfma_16x16x32_bf16(v, pv[b], zero4);
                if (a.split > 1) {
                    // the operand may hold super-tiles of other splits
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int si = (blk << shift) + ((4 * lk + e) >> a.probe_shift);
                        if (si < w.s0 || si >= w.s1) d[e] = -INFINITY;
                    }
                }
                am[b] = fmaxf(fmaxf(am[b], fmaxf(d[0], d[1])), fmaxf(d[2], d[3]));
            }
        };
        const int first = best >> shift;
        probe(first, operand(first));   // every wave
#pragma unroll
        for (int b = 0; b < PB; ++b) am[b] = max_rows(am[b]);
        float lowest = INFINITY;
#pragma unroll
        for (int b = 0; b < PB; ++b) lowest = fminf(lowest, am[b] > -INFINITY ? am[b] : INFINITY);
        lowest = lane_value(row_reduce<false>(lowest), 0);
        // The next operand is in flight while one is evaluated.
        int done = first, turn = 0;
        int held = -1;
        bf16x8 ahead = {};
        for (int g = w.s0; g < w.s1; g += 64) {
            unsigned long long cand = __builtin_amdgcn_ballot_w64(super_bound_of(g) > lowest);
            while (cand) {
                const int blk = (g + __builtin_ctzll(cand)) >> shift;
                cand &= cand - 1;
                if (blk == first || blk == done) continue;
                done = blk;
                if (NW > 1 && turn++ % NW != wave) continue;
                const bf16x8 v = ahead;
                ahead = operand(blk);
                if (held >= 0) probe(held, v);
                held = blk;
            }
        }
        if (held >= 0) probe(held, ahead);
        // over the pixel's lanes and the waves
#pragma unroll
        for (int b = 0; b < PB; ++b) am[b] = max_rows(am[b]);
        if constexpr (NW > 1) {
            if (lane < 32) sh.best[wave][lane] = lane < 16 ? am[0] : am[1];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NW; ++q)
#pragma unroll
                for (int b = 0; b < PB; ++b) am[b] = fmaxf(am[b], sh.best[q][16 * b + lp]);
        }
    }

    // Skipping.  A chunk (or super-tile) whose logit upper bound lies more
    // than skip_log2 below every pixel's reference has every weight below
    // 2^-skip_log2 (exactly 0 in float32 at kExactSkipLog2, so then leaving
    // it out changes no bit).  The bound is taken between the chunk's box and
    // the box of the tile's observations (min reference over the tile), one
    // chunk per lane.  With a posterior tolerance the first pass keeps only
    // the chunks bounded less than depth0 below the reference; the bounds of
    // those it leaves out add up to a bound on the skipped weight, which is
    // then held against the weight each pixel's sums really contain
    // (cert_log2), and while a pixel's certificate fails a further pass adds
    // the chunks of the next kDepthStep units, down to skip_log2.  (On tiles of
    // 8 x 4 neighbours this kept 9.8% of the pairs of sixteen 1080p frames
    // instead of 12.1%: 2.82 to 2.50 ms a call.)
    const int px = lane & 31;
    float mmin = INFINITY;
#pragma unroll
    for (int b = 0; b < PB; ++b) {
        float m = am[b];
        if (a.gref) m = fmaxf(m, a.gref[(size_t)w.f * a.LL + region_pixel<kRegionW>(a, w, ib[b])]);
        // A pixel without a finite logit (a NaN observation) gets NaN maps
        // whatever is kept; it must not switch skipping off for its tile.
        mmin = fminf(mmin, m > -INFINITY ? m : INFINITY);
    }
    mmin = lane_value(row_reduce<false>(mmin), 0) - far2 * 0x1p-20f;
    // If some weight could exceed 2^kFarGap relative to the best probe, take
    // the exact maximum over the nodes of the chunks that will be kept (the
    // only weights evaluated); a split far from the posterior usually keeps
    // none, and then the reference needs no refinement.  Several waves share
    // the scan and put their maxima together behind the first barrier below: a
    // 1920x1080 frame of random intensities, whose tiles spread over the whole
    // grid, took 11.9 ms while both waves of a tile scanned it all, 7.7 this way.
    bool refine = active && __any(!(mup - am[0] <= kFarGap) || !(mup - am[1] <= kFarGap));
    if (refine) {
        const int i = px < 16 ? ib[0] : ib[1];
        float ph[3], pl[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            ph[k] = rsh.obs[k][i];
            pl[k] = rsh.obs[3 + k][i];
        }
        auto chunk_test = [&](int si, int c) {
            return box_box_bound(a.boxes + ((size_t)si * a.chunks_per_super + c) * kBoxFloats, zbox);
        };
        const float m = far_gap_max<kTilePixels, 2, NW>(a, w, ph, pl, lane >> 5, wave, super_bound, chunk_test, mmin,
                                                        px < 16 ? am[0] : am[1]);
        if constexpr (NW > 1) {
            if (lane < 32) sh.top[wave][lane] = m;
        } else {
#pragma unroll
            for (int b = 0; b < PB; ++b) am[b] = __shfl(m, b * 16 + lp);
        }
    }
    // Anchor of the moments, for the whole tile: the centre of the super-tile
    // with the highest bound.
    const float anc_hb = constant(a.headers)[(size_t)best * kHdrFloats + 6];
    const float anc_ox = constant(a.headers)[(size_t)best * kHdrFloats + 7];
    // Observations that spread over much of the grid have estimates far from the
    // tile's one anchor: rounding at the scale of that distance would show (rms
    // error of random tissue on a 128 x 128 grid 2.5e-6 uM instead of 2.3e-6, of
    // random intensities 3.6e-6 instead of 2.0e-6), so their sums keep the rounding
    // errors of the moments' merges (eleven instead of five operations each: a
    // 64x64 frame, of whose tiles three fifths are wide, 23.5 -> 23.9 us a call;
    // 1080p frames, of whose tiles at most 0.2% are, as before).
    const bool wide = !(fmaf(a.spread[1], zbox[5] - zbox[2], a.spread[0] * (zbox[4] - zbox[1])) <= 1.0f);

    unsigned executed = 0;   // chunks evaluated by this wave
    // Chunk records through a buffer resource: the lane offset stays in a
    // register and the record's offset is scalar; loads past the table return 0.
    const __amdgpu_buffer_rsrc_t ops = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(a.split_ops), (short)0, a.n_supers * a.chunks_per_super * kChunkRecordBytes, kBufferWord3);
    const int cps = a.chunks_per_super;
    // Several waves per tile: the tiles of the workgroup go through the same
    // barriers, so they learn of each other whether one has more to do.
    int round = 0;
    auto any_tile = [&](bool mine) {
        if (mine) rsh.more[round] = 1;
        const int after = round == 2 ? 0 : round + 1;
        if (threadIdx.x == 0) rsh.more[after] = 0;   // read last two rounds ago
        __syncthreads();
        const bool any = rsh.more[round] != 0;
        round = after;
        return any;
    };

    // Passes: the chunks whose bound v (relative to mmin) has vlo < v <= vhi
    // are evaluated; a pass that reaches skip_log2 is the last.
    const float nskip = -a.skip_log2;
    float vhi = INFINITY, vlo = -a.depth0;
    for (;;) {
        const bool last = !(vlo > nskip);
        const float svlo = fmaxf(nskip, vlo - kSuperMargin);
        unsigned mass = 0;   // this lane's share of the skipped weight (saturating), in units of 2^-mass_log2
        int g = w.s0;
        for (bool more = true; more;) {
            const ChunkTest test{vlo, vhi, svlo, mmin, last};
            const int K = active ? list_chunks<NW>(a, w, sh.kept, sh.bound, wave, zbox, test, g, mass) : 0;
            if (NW == 1 && K == 0) break;
            tile_sync<NW>();
            if constexpr (NW > 1) {
                if (refine) {
#pragma unroll
                    for (int q = 0; q < NW; ++q)
#pragma unroll
                        for (int b = 0; b < PB; ++b) am[b] = fmaxf(am[b], sh.top[q][16 * b + lp]);
                    refine = false;
                }
            }
            // Segments in turn (which wave sums a segment changes no bit).
            const KeptSuper own = sh.kept[lane];
            for (int seg = wave; seg < kSegments; seg += NW) {
                unsigned long long list =
                    __builtin_amdgcn_ballot_w64(lane < K && own.segment == seg && (own.lo | own.hi) != 0);
                if (NW == 1 && list == 0) continue;
                // Result layout: lane (lp, lk) holds pixel b*16 + lp and the
                // four nodes of chunk row lk; its sums run over those nodes
                // of every chunk of the segment, with Kahan compensation
                // terms K0..K2 across super-tiles.
                float R0[PB], R1[PB], R2[PB], K0[PB], K1[PB], K2[PB];
#pragma unroll
                for (int b = 0; b < PB; ++b) R0[b] = R1[b] = R2[b] = K0[b] = K1[b] = K2[b] = 0.0f;
                for (; list; list &= list - 1) {
                    const int k = __builtin_ctzll(list);
                    unsigned long long walk = (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)own.hi, k) << 32 |
                                              (unsigned)__builtin_amdgcn_readlane((int)own.lo, k);
                    const int si = __builtin_amdgcn_readlane(own.si, k);
                    executed += __popcll(walk);
                    const int s_first = si * cps * kChunkRecordBytes;   // records of the super-tile
                    ConstFloat *H = constant(a.headers) + (size_t)si * kHdrFloats;
                    const float ch = lk == 0 ? H[8] : (lk == 1 ? H[9] : H[10]);
                    const float cl = lk == 0 ? H[11] : (lk == 1 ? H[12] : H[13]);
                    // Walk the kept chunks with two operand buffers: the next chunk's
                    // operands are in flight while the current one is evaluated.  The
                    // loads are issued unconditionally (past the last chunk they fetch
                    // the super-tile's first), so the wait counts match on every path
                    // and a wait for the current chunk never waits for the next one.
                    int left = __popcll(walk);
                    auto take = [&](bf16x8 &bv, f32x3 &qm) {
                        const int c = max(lowest_bit(walk), 0);
                        walk = clear_bit(walk, c);
                        const int at = s_first + c * kChunkRecordBytes;
                        bv = __builtin_bit_cast(
                            bf16x8, __builtin_amdgcn_raw_buffer_load_b128(ops, lane * kSplitLaneBytes, at, 0));
                        qm = __builtin_bit_cast(
                            f32x3, __builtin_amdgcn_raw_buffer_load_b96(ops, kSplitChunkBytes + lk * 16, at, 0));
                        // keep these loads ahead of the evaluation that follows
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    bf16x8 bA, bB;
                    f32x3 qA, qB;
                    take(bA, qA);
                    take(bB, qB);
                    bf16x8 av[PB];
                    const float r[PB] = {(ah[0] - ch) + (al[0] - cl), (ah[1] - ch) + (al[1] - cl)};
                    pixel_operands(r, am, std::integral_constant<bool, DFC>{}, av);
                    float L0[PB], L1[PB], L2[PB];
                    // Weights of the row's four nodes (SO2 offsets s = 0..3): their sum
                    // W0 and first moment W1 = sum s w_s give the row's Hb moment
                    // through the affine row coefficients, and W0 its THb moment (THb
                    // is constant along the row); HbO2 = THb - Hb after the super-tile.
                    // The first chunk of the super-tile starts the sums.
                    auto eval = [&](const bf16x8 &bv, const f32x3 &qm, auto first_chunk) {
#pragma unroll
                        for (int b = 0; b < PB; ++b) {
                            const f32x4 d = mfma_16x16x32_bf16(bv, av[b], zero4);
                            const float w0 = __builtin_amdgcn_exp2f(d[0]), w1 = __builtin_amdgcn_exp2f(d[1]);
                            const float w2 = __builtin_amdgcn_exp2f(d[2]), w3 = __builtin_amdgcn_exp2f(d[3]);
                            const float W0 = (w0 + w1) + (w2 + w3);
                            const float W1 = fmaf(3.0f, w3, fmaf(2.0f, w2, w1));
                            if constexpr (decltype(first_chunk)::value) {
                                L0[b] = W0;
                                L1[b] = fmaf(qm.x, W0, qm.y * W1);
                                L2[b] = qm.z * W0;
                            } else {
                                L0[b] += W0;
                                L1[b] = fmaf(qm.x, W0, fmaf(qm.y, W1, L1[b]));
                                L2[b] = fmaf(qm.z, W0, L2[b]);
                            }
                        }
                    };
                    using First = std::true_type;
                    using Next = std::false_type;
                    eval(bA, qA, First{});
                    while (--left) {
                        take(bA, qA);
                        eval(bB, qB, Next{});
                        if (--left == 0) break;
                        take(bB, qB);
                        eval(bA, qA, Next{});
                    }
                    const float from_hb = H[6] - anc_hb, from_ox = H[7] - anc_ox;
#pragma unroll
                    for (int b = 0; b < PB; ++b) {
                        kahan_add(R0[b], K0[b], L0[b]);
                        L2[b] -= L1[b];   // HbO2 = THb - Hb
                        if (wide) {
                            merge_far_moment(R1[b], K1[b], from_hb, L0[b], L1[b]);
                            merge_far_moment(R2[b], K2[b], from_ox, L0[b], L2[b]);
                        } else {
                            kahan_add(R1[b], K1[b], fmaf(from_hb, L0[b], L1[b]));
                            kahan_add(R2[b], K2[b], fmaf(from_ox, L0[b], L2[b]));
                        }
                    }
                }
                // Sum over the four chunk-row lanes with compensated (two-sum)
                // steps, both blocks at once: lane l < 32 ends up with pixel l.
                auto close = [&](float x, float y, float cx, float cy, int q) {
                    float t, e, f;
                    swap_rows16(x, y);
                    two_sum(x, y, t, e);
                    x = y = t;
                    if (wide) {
                        swap_rows16(cx, cy);
                        e -= cx + cy;
                    }
                    f = e;
                    swap_rows32(x, y);
                    swap_rows32(e, f);
                    float u, v;
                    two_sum(x, y, u, v);
                    const float err = (e + f) + v;
                    if (lane < 32) {
                        if constexpr (NW == 1) {
                            float hi = sh.total[q][lane], lo = sh.total[3 + q][lane];
                            carry_add(hi, lo, u, err);
                            sh.total[q][lane] = hi;
                            sh.total[3 + q][lane] = lo;
                        } else {
                            sh.part[seg][q][lane] = u;
                            sh.part[seg][3 + q][lane] = err;
                        }
                    }
                };
                close(R0[0], R0[1], K0[0], K0[1], 0);
                close(R1[0], R1[1], K1[0], K1[1], 1);
                close(R2[0], R2[1], K2[0], K2[1], 2);
            }
            tile_sync<NW>();   // the window's list is free again, its segments are summed
            more = active && g < w.s1;
            if constexpr (NW > 1) {
                const int q = (64 * wave + lane) / kTilePixels, i = lane % kTilePixels;
                if (K > 0 && q < 3) {
                    float hi = sh.total[q][i], lo = sh.total[3 + q][i];
#pragma unroll
                    for (int t = 0; t < kSegments; ++t) carry_add(hi, lo, sh.part[t][q][i], sh.part[t][3 + q][i]);
                    sh.total[q][i] = hi;
                    sh.total[3 + q][i] = lo;
                }
                more = any_tile(more);
            }
        }
        bool fails = false;
        if (active && !last) {
            // Certificate: the skipped weight, which is at most `mass` relative to mmin for
            // every pixel of the tile, against the pixel's sum.  A NaN sum certifies
            // itself: its maps are NaN whatever is kept.
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1)
                mass = __builtin_elementwise_add_sat(mass, (unsigned)__shfl_xor((int)mass, o));
        }
        if constexpr (NW > 1) {
            if (lane == 0) sh.mass[wave] = mass;
            __syncthreads();
            mass = sh.mass[0];
#pragma unroll
            for (int q = 1; q < NW; ++q) mass = __builtin_elementwise_add_sat(mass, sh.mass[q]);
        }
        if (active && !last) {
            const float held = (px < 16 ? am[0] : am[1]) + __log2f(sh.total[0][px] + sh.total[3][px]);
            fails = __any(certificate_fails(a, mass, held, mmin));
        }
        active = fails;
        if constexpr (NW > 1) {
            if (!any_tile(fails)) break;
        } else {
            if (!fails) break;
        }
        vhi = vlo;
        vlo = fmaxf(nskip, vlo - kDepthStep);
    }
    tile_sync<1>();   // several waves: the passes end with a barrier behind the last sums
    float S0 = sh.total[0][px] + sh.total[3][px];
    const float m = (px < 16 ? am[0] : am[1]);

    // Pixels whose observation lies farther than sqrt(far_rho2) (scaled
    // units) from the grid's nodes: the expanded logit's terms grow with that
    // distance, so their sums are formed again with double-float logits (the
    // plan sets far_rho2 from the precision budget).  The distance is the
    // soft minimum over the split's nodes, rho^2 = -log2 sum_j 2^-|r - v_j|^2
    // = -(m + log2 S0), at most the nearest node's; with a split grid, also
    // that of the best probe of the whole grid (-gref): a split whose nodes
    // all lie far from an observation that lies close to others carries a
    // negligible part of the posterior.  A pixel without a finite logit (a NaN
    // or infinite observation) gets NaN maps from its sums as they are: where a
    // tile holds nothing else they are all zero, which is no distance.  The
    // tile's waves take the pixels in turn.
    unsigned far_pixels = 0;
    // Lane indices for what follows, formed here again rather than kept
    // across the main loop.
    const int lane_e = opaque_v((int)threadIdx.x) & 63, px_e = lane_e & 31;
    const bool valid = base + px_e < n_valid;
    const int pixel = rsh.slot[valid ? base + px_e : 0];
    unsigned long long far =
        __builtin_amdgcn_ballot_w64(lane_e < 32 && valid && m > -INFINITY && m + __log2f(S0) < -a.far_rho2);
    // Every wave of the tile has formed its mask from the passes' sums before
    // one of them replaces a pixel's: the waves then deal the same pixels.
    tile_sync<NW>();
    if (__builtin_expect(far != 0, 0)) {
        // The pass reads the kernel's arguments again from the argument segment
        // (PosteriorArgs is the kernel's only argument): keeping the values it
        // needs live across the main loop would cost that loop registers.
        KernArgs *ka = (KernArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        for (int turn = 0; far != 0; ++turn) {
            const int q = __builtin_ctzll(far);
            far &= far - 1;
            if (NW > 1 && turn % NW != wave) continue;
            const PosteriorArgs fa = far_args(opaque(ka));
            const int i = __builtin_amdgcn_readlane(pixel, q);
            float qh[3], qlo[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                qh[k] = rsh.obs[k][i];
                qlo[k] = rsh.obs[3 + k][i];
            }
            const float mq = __shfl(m, q);
            float m_skip = mq;
            if (fa.gref) {
                const float g = fa.gref[(size_t)w.f * fa.LL + region_pixel<kRegionW>(fa, w, i)];
                if (!(g < -fa.far_rho2)) continue;
                m_skip = fmaxf(m_skip, g);
            }
            ++far_pixels;
            float S[3], E[3];
            far_pixel_sums(fa, w, qh, qlo, m_skip, -mq, anc_hb, anc_ox, S, E);
            const float hi = lane_e == 0 ? S[0] : (lane_e == 1 ? S[1] : S[2]);
            const float lo = lane_e == 0 ? E[0] : (lane_e == 1 ? E[1] : E[2]);
            if (lane_e < 3) {   // these replace the pixel's sums
                sh.total[lane_e][q] = hi;
                sh.total[3 + lane_e][q] = lo;
            }
        }
    }
    tile_sync<NW>();
    S0 = sh.total[0][px_e] + sh.total[3][px_e];
    if (a.work && lane_e == 0) {
        atomicAdd(a.work, (unsigned long long)executed * kTilePixels * kChunkNodes);
        if (far_pixels) atomicAdd(a.work + 1, (unsigned long long)far_pixels);
    }
    const bool writer = wave == 0 && lane_e < 32 && valid;
    const long long pe = region_pixel<kRegionW>(a, w, pixel);
    if (a.fuse) {
        // one split: the estimate is anchor + S1 / S0
        if (writer) {
            const float dh = sh.total[0][px_e], dl = sh.total[3][px_e];
            rsh.est[pixel] = make_float2(plus_quotient(anc_hb, sh.total[1][px_e], sh.total[4][px_e], dh, dl),
                                         plus_quotient(anc_ox, sh.total[2][px_e], sh.total[5][px_e], dh, dl));
            a.est[(size_t)w.f * a.LL + pe] = rsh.est[pixel];
        }
        __syncthreads();
        const int live = NW == 1 ? 64 * min(RT, (n_valid + kTilePixels - 1) / kTilePixels) : 64 * NW * RT;
        fused_maps<kRegionW, kRegionH, RT == 1>(a, w, rsh.est, threadIdx.x, live, rsh.slot + base,
                                                min(kTilePixels, n_valid - base));
        return;
    }
    if (writer) {
        // the moments about the split's own mean, which leaves them small
        const float dh = sh.total[0][px_e], dl = sh.total[3][px_e];
        float at[2], moment[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float nh = sh.total[1 + k][px_e], nl = sh.total[4 + k][px_e], anchor = k ? anc_ox : anc_hb;
            at[k] = S0 > 0.0f ? plus_quotient(anchor, nh, nl, dh, dl) : anchor;
            float from, e;
            two_sum(at[k], -anchor, from, e);
            moment[k] = fmaf(-from, dh, nh) + (nl - fmaf(from, dl, e * dh));
        }
        float *out = a.part + ((size_t)w.f * a.split + w.split) * kPartFields * a.LL;
        out[pe] = m;
        out[a.LL + pe] = S0;
        out[2 * a.LL + pe] = moment[0];
        out[3 * a.LL + pe] = moment[1];
        out[4 * a.LL + pe] = at[0];
        out[5 * a.LL + pe] = at[1];
    }
}


// Direct kernel: one LL pixel per lane, logits in the difference form
// t - m = -(r - v_g)^2 - m on the VALU with wave-uniform (scalar) node loads;
// PRECISE: from double-float differences (df_logit), for grids whose nodes
// are too far apart for float32 logits.  A wave takes a compact tile of 8 x 8
// pixels (its observations then lie close together, which the skip tests rely
// on), a workgroup 2 x 2 of them, whose maps it writes.  The reference search,
// skipping with its certificate, the exact maximum over kept chunks and
// (float32 logits) the double-float pass for far observations are as in the
// MFMA kernel.  Bound by VALU issue, about 8 operations and one exponential
// per (pixel, node).  Three 1006x758 frames at one level on a 24 x 20 grid: 89
// us a call with sums over single nodes, the a-priori skip threshold and a
// kernel of its own for the maps, 67 with the rows' affine moments, the
// certificate and the maps written here, 65 with the super-tiles' bounds kept in
// LDS and the block's place found without divisions.
constexpr int kDirectSide = 16;   // LL pixels of a workgroup's region along each axis
template <bool PRECISE>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(5))) void k_posterior_direct(PosteriorArgs a) {
    __shared__ KeptSuper s_kept[kBlockThreads / 64][64];
    __shared__ float s_bound[kBlockThreads / 64][64];
    __shared__ float2 s_est[kDirectSide * kDirectSide];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const WaveWork w =
        block_work<kDirectSide, kDirectSide>(a, xcd_order(blockIdx.x, gridDim.x, kResidentWaves / 4, a.run_log2));
    const int tr = (wave >> 1) * 8 + (lane >> 3), tc = (wave & 1) * 8 + (lane & 7);   // pixel of the region
    const bool valid = w.r0 + tr < a.hl && w.c0 + tc < a.wl;
    const long long p = (long long)min(w.r0 + tr, a.hl - 1) * a.wl + min(w.c0 + tc, a.wl - 1);
    // The wave of a tile outside the frame has nothing to do (see the MFMA kernel).
    const int wave_rows = w.r0 + 8 < a.hl ? 2 : 1, wave_cols = w.c0 + 8 < a.wl ? 2 : 1;
    if ((wave >> 1) >= wave_rows || (wave & 1) >= wave_cols) return;
    {
        const float *zf = a.z + (size_t)w.f * 6 * a.LL;
        float ph[3], pl[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) load_obs(zf, a.LL, p, k, a.scale, ph[k], pl[k]);
        // Observation box of the tile along the boxes' axes (see the MFMA kernel).
        float zbox[6], far2 = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float q = axis_coordinate(a.axes + 3 * k, (ph[0] - a.origin[0]) + pl[0],
                                            (ph[1] - a.origin[1]) + pl[1], (ph[2] - a.origin[2]) + pl[2]);
            zbox[k] = wave_reduce<false>(q);
            zbox[3 + k] = wave_reduce<true>(q);
            const float e = fmaxf(-zbox[k], zbox[3 + k]);
            far2 = fmaf(e, e, far2);
        }
        widen_box(zbox, far2);
        auto super_bound = [&](int si) {   // -inf past the split's range
            return si < w.s1 ? box_box_bound(a.headers + (size_t)si * kHdrFloats, zbox) : -INFINITY;
        };
        auto chunk_bound = [&](int si, int c) {
            return box_box_bound(a.boxes + ((size_t)si * a.chunks_per_super + c) * kBoxFloats, zbox);
        };

        // Reference logit and anchor: the best probe of the split's super-tiles,
        // the one with the highest bound first, then those bounded above the
        // tile's lowest best probe.
        float mup = -INFINITY, m = -INFINITY, anc_hb = 0.0f, anc_ox = 0.0f;
        int best = w.s0;
        for (int g = w.s0; g < w.s1; g += 64) {
            const float b = super_bound(g + lane), top = wave_reduce<true>(b);
            if (g == w.s0) s_bound[wave][lane] = b;
            if (top > mup) {
                mup = top;
                best = g + __builtin_ctzll(__builtin_amdgcn_ballot_w64(b == top) | (1ull << 63));
            }
        }
        best = __builtin_amdgcn_readfirstlane(best);
        auto probe = [&](int si) {
            ConstFloat *T = constant(a.supers) + (size_t)si * a.super_stride;
            float r[3];
            recentre(T, ph, pl, r);
            probe_supertile(T, r, m, anc_hb, anc_ox);
        };
        probe(best);
        const float lowest = wave_reduce<false>(m > -INFINITY ? m : INFINITY);
        for (int g = w.s0; g < w.s1; g += 64) {
            const int sl = g + lane;
            const float b = g == w.s0 ? s_bound[wave][lane] : super_bound(sl);
            unsigned long long cand = __builtin_amdgcn_ballot_w64(sl != best && b > lowest);
            while (cand) {
                probe(g + __builtin_ctzll(cand));
                cand &= cand - 1;
            }
        }
        float mmin = m;
        if (a.gref) mmin = fmaxf(mmin, a.gref[(size_t)w.f * a.LL + p]);
        mmin = wave_reduce<false>(mmin > -INFINITY ? mmin : INFINITY);   // NaN observation: see the MFMA kernel
        if (__any(!(mup - m <= kFarGap))) m = far_gap_max<64, 1, 1>(a, w, ph, pl, 0, 0, super_bound, chunk_bound, mmin, m);
        const float nm = -m;

        float R0 = 0.f, R1 = 0.f, R2 = 0.f, K0 = 0.f, K1 = 0.f, K2 = 0.f;
        unsigned executed = 0;
        KeptSuper *kept = s_kept[wave];
        const float nskip = -a.skip_log2;
        float vhi = INFINITY, vlo = -a.depth0;
        for (;;) {
            const bool last = !(vlo > nskip);
            unsigned mass = 0;
            const ChunkTest test{vlo, vhi, fmaxf(nskip, vlo - kSuperMargin), mmin, last};
            for (int g = w.s0;;) {
                const int K = list_chunks<1>(a, w, kept, s_bound[wave], 0, zbox, test, g, mass);
                if (K == 0) break;
                tile_sync<1>();
                const KeptSuper own = kept[lane];
                unsigned long long list = __builtin_amdgcn_ballot_w64(lane < K && (own.lo | own.hi) != 0);
                for (; list; list &= list - 1) {
                    const int k = __builtin_ctzll(list);
                    unsigned long long mask = (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)own.hi, k) << 32 |
                                              (unsigned)__builtin_amdgcn_readlane((int)own.lo, k);
                    const int si = __builtin_amdgcn_readlane(own.si, k);
                    executed += __popcll(mask);
                    ConstFloat *T = constant(a.supers) + (size_t)si * a.super_stride;
                    float r[3], rh[3], rl[3];
                    if (PRECISE) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            float sk, e;
                            two_sum(ph[c], -T[c], sk, e);
                            fast_two_sum(sk, e + (pl[c] - T[3 + c]), rh[c], rl[c]);
                        }
                    } else {
                        recentre(T, ph, pl, r);
                    }
                    float L0 = 0.f, L1 = 0.f, L2 = 0.f;
                    ConstFloat *C0 = T + kSupHdr + kMaxProbes * kProbeFloats;
                    for (; mask; mask &= mask - 1) {
                        const int ci = __builtin_ctzll(mask);
                        ConstFloat *C = C0 + (size_t)ci * kChunkFloats;
                        ConstFloat *LO =
                            PRECISE ? constant(a.lo) + ((size_t)si * a.chunks_per_super + ci) * kLoFloats : nullptr;
#pragma unroll
                        for (int row = 0; row < 4; ++row) {
                            float x[4];   // weights of the row's nodes
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                const int j = 4 * row + c;
                                if (PRECISE) {
                                    float tl;
                                    const float th = df_logit(rh, rl, C, LO, j, nm, tl);
                                    const float e = __builtin_amdgcn_exp2f(th);
                                    x[c] = fmaf(e, tl * 0.6931471805599453f, e);
                                    L0 += x[c];
                                    L1 = fmaf(x[c], C[64 + j], L1);
                                    L2 = fmaf(x[c], C[80 + j], L2);
                                } else {
                                    const float d0 = r[0] - C[j], d1 = r[1] - C[16 + j], d2 = r[2] - C[32 + j];
                                    float t = fmaf(-d0, d0, nm);
                                    t = fmaf(-d1, d1, t);
                                    t = fmaf(-d2, d2, t);
                                    x[c] = __builtin_amdgcn_exp2f(t);
                                }
                            }
                            if (!PRECISE) {
                                // the row's affine moments, as in the MFMA kernel; L2 the THb moment
                                const float W0 = (x[0] + x[1]) + (x[2] + x[3]);
                                const float W1 = fmaf(3.0f, x[3], fmaf(2.0f, x[2], x[1]));
                                L0 += W0;
                                L1 = fmaf(C[104 + 4 * row], W0, fmaf(C[105 + 4 * row], W1, L1));
                                L2 = fmaf(C[106 + 4 * row], W0, L2);
                            }
                        }
                    }
                    if (!PRECISE) L2 -= L1;   // HbO2 = THb - Hb
                    kahan_add(R0, K0, L0);
                    kahan_add(R1, K1, fmaf(T[6] - anc_hb, L0, L1));
                    kahan_add(R2, K2, fmaf(T[7] - anc_ox, L0, L2));
                }
                tile_sync<1>();   // the list is free again
                if (g >= w.s1) break;
            }
            if (last) break;
            // certificate, as in the MFMA kernel
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1)
                mass = __builtin_elementwise_add_sat(mass, (unsigned)__shfl_xor((int)mass, o));
            if (!__any(certificate_fails(a, mass, m + __log2f(R0), mmin))) break;
            vhi = vlo;
            vlo = fmaxf(nskip, vlo - kDepthStep);
        }
        if (a.work && lane == 0) atomicAdd(a.work, (unsigned long long)executed * 64 * kChunkNodes);
        if constexpr (!PRECISE) {
            // Pixels whose observation lies far from the grid's nodes: the float32
            // differences round at the scale of that distance, so their sums are
            // formed again with double-float logits, as in the MFMA kernel (the
            // plan sets far_rho2 from this kernel's precision budget).
            unsigned long long far = __ballot(valid && m > -INFINITY && m + __log2f(R0) < -a.far_rho2);
            unsigned far_pixels = 0;
            while (__builtin_expect(far != 0, 0)) {
                const int q = __builtin_ctzll(far);   // the pixel of lane q
                far &= far - 1;
                float qh[3], ql[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    qh[k] = __shfl(ph[k], q);
                    ql[k] = __shfl(pl[k], q);
                }
                const float mq = __shfl(m, q);
                float m_skip = mq;
                if (a.gref) {
                    const float g = a.gref[(size_t)w.f * a.LL + __shfl(p, q)];
                    if (!(g < -a.far_rho2)) continue;
                    m_skip = fmaxf(m_skip, g);
                }
                ++far_pixels;
                float S[3], E[3];
                far_pixel_sums(a, w, qh, ql, m_skip, -mq, __shfl(anc_hb, q), __shfl(anc_ox, q), S, E);
                if (lane == q) {
                    R0 = S[0];
                    R1 = S[1];
                    R2 = S[2];
                    K0 = -E[0];
                    K1 = -E[1];
                    K2 = -E[2];
                }
            }
            if (a.work && lane == 0 && far_pixels) atomicAdd(a.work + 1, (unsigned long long)far_pixels);
        }
        if (a.fuse) {
            // one split: the estimate is anchor + S1 / S0 (the Kahan terms hold
            // minus what the sums lack)
            const float2 e = make_float2(plus_quotient(anc_hb, R1, -K1, R0, -K0), plus_quotient(anc_ox, R2, -K2, R0, -K0));
            s_est[tr * kDirectSide + tc] = e;
            if (valid) a.est[(size_t)w.f * a.LL + p] = e;
        } else if (valid) {
            float *out = a.part + ((size_t)w.f * a.split + w.split) * kPartFields * a.LL;
            out[p] = m;
            out[a.LL + p] = R0;
            out[2 * a.LL + p] = R1;
            out[3 * a.LL + p] = R2;
            out[4 * a.LL + p] = anc_hb;
            out[5 * a.LL + p] = anc_ox;
        }
    }
    if (a.fuse) {
        __syncthreads();
        const int thread = 64 * ((wave >> 1) * wave_cols + (wave & 1)) + lane;
        fused_maps<kDirectSide, kDirectSide, false>(a, w, s_est, thread, 64 * wave_rows * wave_cols);
    }
}

// ---------------------------------------------------------------------------
// K3: merge the grid splits per LL pixel, inverse Haar of the Tikhonov
// details with the low-pass estimate added once at the end (the inverse of a
// low-pass-only block is that constant on every pixel), and the output maps.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float2 lowpass_estimate(const RecomposeArgs &a, int f, long long q) {
    if (a.lowpass == HB_LOWPASS_TIKHONOV) {
        const long long LL = a.d.LL;
        const float *zf = a.z + (size_t)f * 6 * LL + q;
        const float zh[3] = {zf[0], zf[LL], zf[2 * LL]}, zl[3] = {zf[3 * LL], zf[4 * LL], zf[5 * LL]};
        return linear_estimate(a.M, zh, zl);
    }
    const long long LL = a.d.LL;
    const float *P = a.part + (size_t)f * a.split * kPartFields * LL + q;
    float m = -INFINITY;
    for (int i = 0; i < a.split; ++i) m = fmaxf(m, P[(size_t)i * kPartFields * LL]);
    const float a_hb = P[4 * LL], a_ox = P[5 * LL];
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
    for (int i = 0; i < a.split; ++i) {
        const float *Pi = P + (size_t)i * kPartFields * LL;
        const float fct = exp2f(Pi[0] - m);
        const float S0 = Pi[LL];
        kahan_add(s0, c0, S0 * fct);
        kahan_add(s1, c1, fmaf(Pi[4 * LL] - a_hb, S0, Pi[2 * LL]) * fct);
        kahan_add(s2, c2, fmaf(Pi[5 * LL] - a_ox, S0, Pi[3 * LL]) * fct);
    }
    return make_float2(a_hb + s1 / s0, a_ox + s2 / s0);
}

// K3: one thread per (frame, block, block row): the block's low-pass
// estimate (split merge, or the Tikhonov low-pass), plus the row's detail
// part, to the four maps, V pixels per vector access.
template <int V>
__global__ __launch_bounds__(kBlockThreads) void k_recompose(RecomposeArgs a) {
    const Dims &d = a.d;
    const int n = d.levels, B = 1 << n;
    const unsigned idx = blockIdx.x * kBlockThreads + threadIdx.x, f = blockIdx.y;
    const unsigned q = idx >> n;   // block of frame f
    if (q >= (unsigned)d.LL) return;
    const int r = (int)(idx & (B - 1));
    const int br = (int)(q / (unsigned)d.wl), bc = (int)(q - (unsigned)br * (unsigned)d.wl);
    const float2 e = lowpass_estimate(a, f, q);
    if (r == 0) a.est[(size_t)f * d.LL + q] = e;
    const size_t row = ((size_t)f * d.H + ((size_t)br << n) + r) * d.W + ((size_t)bc << n);
    for (int c = 0; c < B; c += V) {
        float2 dp[V];
        load_detail<V>(a.det, row + c, dp);
        write_maps<V>(a.hb, a.hbo2, a.thb, a.so2, a.thb_eps, row + c, e, dp);
    }
}

}  // namespace

hipError_t launch_tikhonov_fp64(const double *d_in, double *d_out, float *d_mf, hipStream_t s) {
    hipLaunchKernelGGL(k_tikhonov_fp64, dim3(1), dim3(64), 0, s, d_in, d_out, d_mf);
    return hipGetLastError();
}

namespace {

template <typename T, int N, bool MAPS>
void launch_df(const void *frames, const HaarArgs &b, bool aligned, hipStream_t s) {
    constexpr int kPerBlock = 1 << (2 * (N < 2 ? 0 : N - 2));   // threads
    const dim3 g((unsigned)((b.d.LL * kPerBlock + kBlockThreads - 1) / kBlockThreads), (unsigned)b.n_frames);
    if (aligned)
        hipLaunchKernelGGL((k_log_haar_df<T, N, true, MAPS>), g, dim3(kBlockThreads), 0, s, (const T *)frames, b);
    else
        hipLaunchKernelGGL((k_log_haar_df<T, N, false, MAPS>), g, dim3(kBlockThreads), 0, s, (const T *)frames, b);
}

template <typename T, int N, bool MAPS>
void launch_reg(const void *frames, const HaarArgs &b, hipStream_t s) {
    const dim3 g((unsigned)((b.d.LL + kBlockThreads - 1) / kBlockThreads), (unsigned)b.n_frames);
    hipLaunchKernelGGL((k_log_haar_reg<T, N, MAPS>), g, dim3(kBlockThreads), 0, s, (const T *)frames, b);
}

template <typename T, bool MAPS>
void launch_blocks(const void *frames, const HaarArgs &b, bool aligned, hipStream_t s) {
    const bool df = b.d.levels >= 3 || b.df;
    switch (b.d.levels) {
        case 0: df ? launch_df<T, 0, MAPS>(frames, b, aligned, s) : launch_reg<T, 0, MAPS>(frames, b, s); break;
        case 1: df ? launch_df<T, 1, MAPS>(frames, b, aligned, s) : launch_reg<T, 1, MAPS>(frames, b, s); break;
        case 2: df ? launch_df<T, 2, MAPS>(frames, b, aligned, s) : launch_reg<T, 2, MAPS>(frames, b, s); break;
        case 3: launch_df<T, 3, MAPS>(frames, b, aligned, s); break;
        case 4: launch_df<T, 4, MAPS>(frames, b, aligned, s); break;
        default: launch_df<T, 5, MAPS>(frames, b, aligned, s); break;
    }
}

template <typename T>
void launch_k1(const void *frames, const HaarArgs &b, hipStream_t s) {
    const bool aligned = vector_frames(frames, b);
    if (b.maps) {
        launch_blocks<T, true>(frames, b, aligned, s);
    } else if (log_haar_takes_blocks(frames, b)) {
        launch_blocks<T, false>(frames, b, aligned, s);
    } else {
        // the strip kernel keeps the register kernel's bits
        HaarArgs c = b;
        c.vec4 = ((uintptr_t)frames % (4 * sizeof(T))) == 0;
        const long long grid = (long long)b.n_frames * b.d.hl * b.d.strips_per_row;
        hipLaunchKernelGGL((k_log_haar<T>), dim3((unsigned)grid), dim3(kBlockThreads), 0, s, (const T *)frames, c);
    }
}

}  // namespace

hipError_t launch_log_haar(const void *frames, int n_frames, const HaarArgs &a, hipStream_t s) {
    if (n_frames <= 0) return hipSuccess;
    HaarArgs b = a;
    b.n_frames = n_frames;
    switch (a.dtype) {
        case HB_F32: launch_k1<float>(frames, b, s); break;
        case HB_F16: launch_k1<__half>(frames, b, s); break;
        default: launch_k1<uint16_t>(frames, b, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_reference(const PosteriorArgs &a, hipStream_t s) {
    const long long n = (long long)a.n_frames * a.LL;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reference, dim3((unsigned)((n + kBlockThreads - 1) / kBlockThreads)), dim3(kBlockThreads),
                       0, s, a);
    return hipGetLastError();
}

namespace {

template <int NW, int RT>
void launch_mfma(const PosteriorArgs &a, long long regions, hipStream_t s) {
    const dim3 g((unsigned)(regions * (kRegionTiles / RT))), blk(64 * NW * RT);
    if (a.dfc)
        hipLaunchKernelGGL((k_posterior<NW, RT, true>), g, blk, 0, s, a);
    else
        hipLaunchKernelGGL((k_posterior<NW, RT, false>), g, blk, 0, s, a);
}

}  // namespace

// Chunk tables up to twice an XCD's L2 (4 MB).
constexpr size_t kTableNearL2 = 8 << 20;

// Run length (log2, in blocks) in which a launch is dealt to the XCDs.  An XCD's
// contiguous eighth of a few frames is one part of a picture, and costs differ
// between the parts by more than short runs lose in L2: us a call with an eighth
// and with runs of 8, 1080p frames on a 256 x 256 grid: one 179.5 and 175.4, two
// 303 and 294, four 552 and 542, six 786 and 788, eight 1024 and 1033.  From six
// on the eighth stays.  Tables past twice an XCD's L2 (4 MB) want longer runs:
// 1280x1024 pair, eighth, runs of 8 and of 64: 320 x 320 grid (7 MB) 949, 918 and
// 921; 384 x 384 (10 MB) 1317, 1303 and 1276; 448 x 448 1763, 1820 and 1715.
static int xcd_run_log2(int n_frames, size_t table_bytes) {
    if (n_frames >= 6) return 0;
    return table_bytes <= kTableNearL2 ? 3 : 6;
}

hipError_t launch_posterior(const PosteriorArgs &args, bool mfma, hipStream_t s) {
    const int bw = mfma ? kRegionW : kDirectSide, bh = mfma ? kRegionH : kDirectSide;
    const int cols = (args.wl + bw - 1) / bw, rows = (args.hl + bh - 1) / bh;
    const long long blocks = (long long)cols * rows * args.n_frames * args.split;
    if (blocks <= 0) return hipSuccess;
    PosteriorArgs a = args;
    a.order = BlockOrder(cols, rows, a.split);
    const size_t table = (size_t)a.n_supers * a.chunks_per_super * kChunkRecordBytes;
    a.run_log2 = xcd_run_log2(a.n_frames, table);
    if (mfma) {
        // Tiles that would all be resident at once with one wave each: the
        // launch would last as long as its busiest tile (2.3 times the mean on
        // 1080p frames).  Few of them take four waves each, in a workgroup of
        // their own so that few regions still reach every CU (the region is
        // then ranked by each of its four tiles' workgroups).  One 640x480
        // frame (600 tiles, 256 x 256 grid): 155 us a call with one wave per
        // tile and four tiles per workgroup, 72 this way.  With more of them
        // what the waves of a tile repeat weighs more than balance, and two
        // waves a tile in a region's workgroup are faster: us a call with four
        // and with two waves, one 1080p frame (4080 tiles) 181 and 175.5, on a
        // 128 x 128 grid 97 and 87, 5904 tiles 242 and 227; but 3800 tiles 171
        // and 172, 2560 tiles 131 and 139.  Small super-tiles repeat more per
        // chunk and change over earlier (2560 tiles on a 128 x 128 grid 72.2 and
        // 68.4, 3200 on 96 x 96 50.1 and 48.4), large tables never do (4080
        // tiles on 384 x 384 319 and 334).  Past the residents one wave a tile:
        // 7680 tiles 303 and 305.5 with two, 9600 (128 x 128 grid) 159 and 168.
        const long long tiles = blocks * kRegionTiles;
        const long long pairs_from = a.chunks_per_super <= 16 ? 2048 : 4000;
        if (tiles > kResidentWaves) {
            launch_mfma<1, kRegionTiles>(a, blocks, s);
        } else if (tiles > pairs_from && table <= kTableNearL2) {
            launch_mfma<2, kRegionTiles>(a, blocks, s);
        } else {
            if (a.run_log2) a.run_log2 += 2;   // four workgroups a region
            launch_mfma<4, 1>(a, blocks, s);
        }
    } else if (a.precise) {
        hipLaunchKernelGGL(k_posterior_direct<true>, dim3((unsigned)blocks), dim3(kBlockThreads), 0, s, a);
    } else {
        hipLaunchKernelGGL(k_posterior_direct<false>, dim3((unsigned)blocks), dim3(kBlockThreads), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_recompose(int n_frames, const RecomposeArgs &a, hipStream_t s) {
    if (n_frames <= 0) return hipSuccess;
    RecomposeArgs b = a;
    b.n_frames = n_frames;
    const int B = 1 << a.d.levels;
    const dim3 blocks((unsigned)((a.d.LL * B + kBlockThreads - 1) / kBlockThreads), (unsigned)n_frames);
    // widest vector the block width and every map pointer allow
    auto fits = [&](int v) {
        if (B % v) return false;
        for (const float *m : {a.hb, a.hbo2, a.thb, a.so2})
            if (m && ((uintptr_t)m % (sizeof(float) * v)) != 0) return false;
        return true;
    };
    if (fits(4))
        hipLaunchKernelGGL(k_recompose<4>, blocks, dim3(kBlockThreads), 0, s, b);
    else if (fits(2))
        hipLaunchKernelGGL(k_recompose<2>, blocks, dim3(kBlockThreads), 0, s, b);
    else
        hipLaunchKernelGGL(k_recompose<1>, blocks, dim3(kBlockThreads), 0, s, b);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Static scratch of hb_estimate_frames_noalloc: the per-call buffers
// (low-pass observation, detail part, posterior partials, global reference,
// low-pass estimate) are carved out of this array instead of the plan's own
// allocations.  Each device holds its own copy for the life of the process.
// Host code never passes the array's name to a kernel (on the host it is only
// a registration handle): static_scratch() looks up the device address once
// per device, with that device current, and every launch uses that address.
// ---------------------------------------------------------------------------
namespace {
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

hipError_t static_scratch(int device, void **ptr) {
    *ptr = nullptr;
    if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = p;
    }
    *ptr = g_scratch_ptr[device];
    return hipSuccess;
}

}  // namespace hb
