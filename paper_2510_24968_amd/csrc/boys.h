// Boys function F_n(T) = int_0^1 exp(-T t^2) t^(2n) dt on the device
// (definition in Sec. 2.3.3; the paper gives no evaluation method).
//
// Grid T_k = k * BOYS_DT, k < BOYS_NT.  A class kernel of total angular
// momentum L stages the orders L .. L+7 of the FP64 grid into LDS, each
// pre-divided by j!, so that
//     F_L(T) = sum_j F_{L+j}(T_k) (T_k - T)^j / j!       (dF_n/dT = -F_{n+1})
// is one 8-term Horner polynomial in (T_k - T) about the nearest grid point,
// and the lower orders follow from the downward recursion
//     F_{n-1} = (2 T F_n + exp(-T)) / (2n - 1).
// For T >= BOYS_TMAX, F_0 = sqrt(pi / T) / 2 (erfc(sqrt T) < 1e-16 there)
// and the upward recursion F_{n+1} = ((2n + 1) F_n - exp(-T)) / (2T), which
// is stable for 2T > 2n + 1.  Everything here is FP64 except the Taylor
// step of boys_eval_mixed (FP32 tiles).
#pragma once

#include "fsim_internal.h"

namespace fsim {

__host__ __device__ constexpr double inv_factorial(int j) {
    double f = 1.0;
    for (int k = 2; k <= j; ++k) f *= k;
    return 1.0 / f;
}

// LDS footprint of one staged table, in doubles.
constexpr int BOYS_LDS = BOYS_NT * BOYS_NTAYLOR;

// n doubles (even) from 16-byte aligned global memory into LDS.
__device__ __forceinline__ void boys_copy(double *lds, const double *__restrict__ g, int n) {
    const double2 *__restrict__ src = (const double2 *)g;
    for (int i = threadIdx.x; i < n / 2; i += blockDim.x) ((double2 *)lds)[i] = src[i];
}

__device__ inline void boys_stage(double *lds, const double *__restrict__ g, int L) {
    boys_copy(lds, g + boys_base(L), BOYS_LDS);
}

// 1 / sqrt(x) for finite x > 0: the hardware estimate and one step of
// y (1 + e/2 + 3 e^2 / 8), e = 1 - x y^2.
__device__ __forceinline__ double rsqrt_pos(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Large-T branch shared by the evaluators: F_0 = sqrt(pi)/2 / sqrt(T) and
// the upward recursion with 1/(2T) taken from the same reciprocal square
// root (a product of two roundings instead of a division).
template <int L>
__device__ __forceinline__ void boys_large_t(double T, double e, double *F) {
    const double rs = rsqrt(T);
    F[0] = 0.88622692545275801365 * rs;
    if constexpr (L > 0) {
        const double h = 0.5 * rs * rs;
#pragma unroll
        for (int n = 0; n < L; ++n) F[n + 1] = ((2 * n + 1) * F[n] - e) * h;
    }
}

// The ket-outer kernels' table of order L: boys_nt(L) rows of the grid and
// the column exp(-T_k).  On the grid exp(-T) = exp(-T_k) exp(d) with
// d = T_k - T, |d| <= 0.05, already at hand from the Taylor step, and exp(d)
// from its series through d^8/8! (truncation below 6e-18 relative); beyond
// it the asymptotic form needs no exponential at all.  Evaluating exp(-T)
// inside the grid branch and not ahead of both, and ending the grid where
// the large-T branch is a plain recursion, took the 64-water FP64 s/p build
// from 291.8 to 273.1 ms, its mixed build from 252.6 to 214.8.
//
// The nearest grid point comes from one FMA onto 1.5 2^52, whose last place is
// one: the sum's low bits are the index and the difference the rounded value.
// FP64 rounding and integer conversions issue at a quarter of the FMA rate
// (64-water FP64 s/p build 228.0 -> 221.7 ms, 1024 C/H molecules 303.0 -> 296.6).
struct BoysPoint {
    int k;
    double d;   // T_k - T
};
__device__ __forceinline__ BoysPoint boys_point(double T) {
    constexpr double M = 6755399441055744.0;
    const double t = fma(T, BOYS_INV_DT, M);
    return BoysPoint{(int)__double_as_longlong(t), fma(t - M, BOYS_DT, -T)};
}

template <int L>
struct BoysLong {
    static constexpr int ECOL = boys_ecol(L), SIZE = boys_block(L);
    static __device__ __forceinline__ void stage(double *lds, const double *__restrict__ g) {
        boys_copy(lds, g + boys_base(L), SIZE);
    }
    // exp(-T) at grid point k, d = T_k - T
    static __device__ __forceinline__ double expm(const double *ecol, int k, double d) {
        double p = inv_factorial(8);
#pragma unroll
        for (int j = 7; j >= 0; --j) p = fma(p, d, inv_factorial(j));
        return ecol[k] * p;
    }
    static __device__ __forceinline__ void down(double T, double e, double *F) {
        const double t2 = 2.0 * T;
#pragma unroll
        for (int n = L; n > 0; --n) F[n - 1] = fma(t2, F[n], e) * (1.0 / (2 * n - 1));
    }
    static __device__ __forceinline__ void asymptotic(double T, double *F) {
        const double rs = rsqrt(T);
        F[0] = 0.88622692545275801365 * rs;
        if constexpr (L > 0) {
            const double h = 0.5 * rs * rs;
#pragma unroll
            for (int n = 0; n < L; ++n) F[n + 1] = (2 * n + 1) * F[n] * h;
        }
    }
    static __device__ __forceinline__ void eval(double T, const double *tab, double *F) {
        if (T < boys_tmax(L)) {
            const auto [k, d] = boys_point(T);
            const double *c = tab + k * BOYS_NTAYLOR;
            double f = c[BOYS_NTAYLOR - 1];
#pragma unroll
            for (int j = BOYS_NTAYLOR - 2; j >= 0; --j) f = fma(f, d, c[j]);
            F[L] = f;
            if constexpr (L > 0) down(T, expm(tab + ECOL, k, d), F);
        } else {
            asymptotic(T, F);
        }
    }
};

// F_0..F_L at T from a table staged for order L.  exp(-T), which both branches need for L > 0, is evaluated once ahead
// of the branch: the lanes of a wave often take both branches, which would
// otherwise run it twice.
template <int L>
__device__ __forceinline__ void boys_eval(double T, const double *tab, double *F) {
    double e = 0.0;
    if constexpr (L > 0) e = exp(-T);
    if (T < BOYS_TMAX) {
        const int k = __double2int_rn(T * BOYS_INV_DT);
        const double d = k * BOYS_DT - T;
        const double *c = tab + k * BOYS_NTAYLOR;
        double f = c[BOYS_NTAYLOR - 1];
#pragma unroll
        for (int j = BOYS_NTAYLOR - 2; j >= 0; --j) f = fma(f, d, c[j]);
        F[L] = f;
        if constexpr (L > 0) {
            const double t2 = 2.0 * T;
#pragma unroll
            for (int n = L; n > 0; --n) F[n - 1] = fma(t2, F[n], e) * (1.0 / (2 * n - 1));
        }
    } else {
        boys_large_t<L>(T, e, F);
    }
}

// Evaluation for the FP32 tiles (quartets whose Schwarz bound is below the
// FP32 threshold).  Only the small-T Taylor step runs in FP32: the same grid
// rounded to FP32 and 5 Taylor terms (truncation at most 0.05^5/5! relative
// to F_L, below FP32 rounding), which gives F_L to FP32 accuracy.  The
// downward recursion to F_0..F_{L-1} and the whole large-T branch
// (asymptotic F_0 and the upward recursion) stay FP64; the caller rounds
// the R^n_000 sources to FP32 afterwards.
constexpr int BOYS_NTAYLOR32 = 5;
constexpr int BOYS_LDS32 = BOYS_NT * BOYS_NTAYLOR32;

__device__ inline void boys_stage32(float *lds, const double *__restrict__ g, int L) {
    for (int i = threadIdx.x; i < BOYS_LDS32; i += blockDim.x) {
        const int k = i / BOYS_NTAYLOR32, j = i - k * BOYS_NTAYLOR32;
        lds[i] = (float)g[boys_base(L) + k * BOYS_NTAYLOR + j];
    }
}

template <int L>
__device__ __forceinline__ void boys_eval_mixed(double T, const float *tab, double *F) {
    double e = 0.0;
    if constexpr (L > 0) e = exp(-T);
    if (T < BOYS_TMAX) {
        const float Tf = (float)T;
        const int k = __float2int_rn(Tf * (float)BOYS_INV_DT);
        const float d = k * (float)BOYS_DT - Tf;
        const float *c = tab + k * BOYS_NTAYLOR32;
        float f = c[BOYS_NTAYLOR32 - 1];
#pragma unroll
        for (int j = BOYS_NTAYLOR32 - 2; j >= 0; --j) f = fmaf(f, d, c[j]);
        F[L] = (double)f;
        if constexpr (L > 0) {
            const double t2 = 2.0 * T;
#pragma unroll
            for (int n = L; n > 0; --n) F[n - 1] = fma(t2, F[n], e) * (1.0 / (2 * n - 1));
        }
    } else {
        boys_large_t<L>(T, e, F);
    }
}

// The ket-outer kernels' form of it: the exp column (FP64) first, then the
// FP32 rows.
template <int L>
struct BoysLongMixed {
    static constexpr int NE = boys_block(L) - boys_ecol(L);             // doubles
    static constexpr int NF = boys_nt(L) * BOYS_NTAYLOR32;              // floats
    static constexpr int SIZE = NE + (NF + 1) / 2;                      // doubles
    static __device__ __forceinline__ void stage(double *lds, const double *__restrict__ g) {
        boys_copy(lds, g + boys_base(L) + boys_ecol(L), NE);
        float *__restrict__ f = (float *)(lds + NE);
        for (int i = threadIdx.x; i < NF; i += blockDim.x) {
            const int k = i / BOYS_NTAYLOR32, j = i - k * BOYS_NTAYLOR32;
            f[i] = (float)g[boys_base(L) + k * BOYS_NTAYLOR + j];
        }
    }
    static __device__ __forceinline__ void eval(double T, const double *tab, double *F) {
        if (T < boys_tmax(L)) {
            const auto [k, dk] = boys_point(T);
            const float d = (float)dk;
            const float *c = (const float *)(tab + NE) + k * BOYS_NTAYLOR32;
            float f = c[BOYS_NTAYLOR32 - 1];
#pragma unroll
            for (int j = BOYS_NTAYLOR32 - 2; j >= 0; --j) f = fmaf(f, d, c[j]);
            F[L] = (double)f;
            if constexpr (L > 0)
                BoysLong<L>::down(T, BoysLong<L>::expm(tab, k, dk), F);
        } else {
            BoysLong<L>::asymptotic(T, F);
        }
    }
};

// Runtime-L variant reading the full global grid (setup kernels only).
__device__ inline void boys_eval_rt(int L, double T, const double *__restrict__ g, double *F) {
    if (T < BOYS_TMAX) {
        const int k = __double2int_rn(T * BOYS_INV_DT);
        const double d = k * BOYS_DT - T;
        double f = 0.0;
        for (int j = BOYS_NTAYLOR - 1; j >= 0; --j)
            f = fma(f, d, g[k * BOYS_NORD + L + j] * inv_factorial(j));
        F[L] = f;
        const double e = exp(-T), t2 = 2.0 * T;
        for (int n = L; n > 0; --n) F[n - 1] = (t2 * F[n] + e) / (2 * n - 1);
    } else {
        F[0] = 0.88622692545275801365 * rsqrt(T);
        const double e = exp(-T), h = 0.5 / T;
        for (int n = 0; n < L; ++n) F[n + 1] = ((2 * n + 1) * F[n] - e) * h;
    }
}

}  // namespace fsim
