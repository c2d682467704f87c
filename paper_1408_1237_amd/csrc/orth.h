// Gram-Schmidt and the Givens step of one short vector in one block (device
// code shared by the single and the batched solvers).
//
// At a few thousand points an Arnoldi step's orthogonalisation is a serial chain
// of launches, not of memory traffic: MGS against j + 1 basis vectors took j + 2
// launches (two per vector in the batched solver) of about 4.7 us each, for
// vectors of 16-64 KB.  One block of 1024 threads keeps the vector in registers
// (up to ORTH_MAX_N entries), reads each basis vector once (the next one is
// requested before the current sum is reduced) and does the whole chain: about
// 1 us per basis vector.
#pragma once

#include "krr_internal.h"

namespace krr {

constexpr int ORTH_THREADS = 1024;
constexpr int ORTH_PER = 8;                              // vector entries per thread
constexpr int ORTH_MAX_N = ORTH_THREADS * ORTH_PER;      // longest vector of the one-block form
constexpr int ORTH_MAX_M = 1000;                         // largest restart length (krr.h)

struct OrthShared {
    double part[2][ORTH_THREADS / WAVE];
    double h[ORTH_MAX_M + 2];  // the Hessenberg column
    double cs[ORTH_MAX_M], sn[ORTH_MAX_M];
};

// Block sum of v, the same in every thread; buf alternates between calls.
__device__ __forceinline__ double orth_sum(double v, OrthShared &sh, int &buf) {
    v = wave_total64(v);
    if (threadIdx.x % WAVE == 0) sh.part[buf][threadIdx.x / WAVE] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < ORTH_THREADS / WAVE; ++k) s += sh.part[buf][k];
    buf ^= 1;
    return s;
}

// Orthogonalises the vector x (entry tid + 1024 k in x[k], n entries) against
// V_0 .. V_j (V_i at V + i ld): MGS as printed, or classical Gram-Schmidt twice.
// On return sh.h[0 .. j + 1] is the Hessenberg column (after the caller's next
// barrier), wnorm0 = ||x|| before, and the return value ||x|| after.
template <bool CGS2>
__device__ __forceinline__ double orth_column(double (&x)[ORTH_PER], int n, const double *__restrict__ V, int64_t ld,
                                              int j, OrthShared &sh, double &wnorm0) {
    const int tid = threadIdx.x;
    int buf = 0;
    auto load = [&](int i, double (&v)[ORTH_PER]) {
#pragma unroll
        for (int k = 0; k < ORTH_PER; ++k) {
            const int e = tid + k * ORTH_THREADS;
            v[k] = e < n ? V[static_cast<int64_t>(i) * ld + e] : 0.0;
        }
    };
    auto dot = [&](const double (&a)[ORTH_PER], const double (&b)[ORTH_PER]) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < ORTH_PER; ++k) s = __builtin_fma(a[k], b[k], s);
        return s;
    };
    double v[ORTH_PER], nx[ORTH_PER];
    load(0, v);
    wnorm0 = sqrt(orth_sum(dot(x, x), sh, buf));
    for (int pass = 0; pass < (CGS2 ? 2 : 1); ++pass) {
        if (pass > 0) load(0, v);
        for (int i = 0; i <= j; ++i) {
            if (i < j) load(i + 1, nx);
            const double h = orth_sum(dot(x, v), sh, buf);
            if constexpr (CGS2) {
                // pass 0 leaves the coefficients in h, pass 1 in cs (added to h below)
                if (tid == 0) (pass == 0 ? sh.h : sh.cs)[i] = h;
            } else {
                if (tid == 0) sh.h[i] = h;
#pragma unroll
                for (int k = 0; k < ORTH_PER; ++k) x[k] = __builtin_fma(-h, v[k], x[k]);
            }
#pragma unroll
            for (int k = 0; k < ORTH_PER; ++k) v[k] = nx[k];
        }
        if constexpr (CGS2) {
            __syncthreads();
            for (int i = 0; i <= j; ++i) {
                load(i, v);
                const double h = (pass == 0 ? sh.h : sh.cs)[i];
#pragma unroll
                for (int k = 0; k < ORTH_PER; ++k) x[k] = __builtin_fma(-h, v[k], x[k]);
            }
            if (pass == 1) {
                for (int i = tid; i <= j; i += ORTH_THREADS) sh.h[i] += sh.cs[i];
                __syncthreads();
            }
        }
    }
    const double hn = sqrt(orth_sum(dot(x, x), sh, buf));
    if (tid == 0) sh.h[j + 1] = hn;
    return hn;
}

// Rotates the Hessenberg column in sh.h with the j previous rotations and forms
// rotation j; called by one thread with sh.cs / sh.sn holding rotations
// 0 .. j - 1.  Returns rho (the new diagonal entry, left in sh.h[j]; sh.h[j + 1]
// becomes 0) and the rotation.
__device__ __forceinline__ double orth_givens(OrthShared &sh, int j, double &cj, double &sj) {
    double a = sh.h[0];
    for (int i = 0; i < j; ++i) {
        const double b = sh.h[i + 1], c = sh.cs[i], s = sh.sn[i];
        sh.h[i] = c * a + s * b;
        a = -s * a + c * b;
    }
    const double b = sh.h[j + 1];
    const double rho = sqrt(a * a + b * b);
    cj = a / rho;
    sj = b / rho;
    sh.h[j] = rho;
    sh.h[j + 1] = 0.0;
    return rho;
}

}  // namespace krr
