// Adjoint pass for the gradient of a loss l(w), w = K^{-1} y, with respect to
// the points, log sigma and log gamma (hyperparameters by maximum likelihood,
// section 2.1).  With lambda = K^{-1} dl/dw, dl/dtheta = -lambda^T (dK/dtheta) w:
//   dl/dx_i   = (1/sigma^2) sum_j (lambda_i w_j + lambda_j w_i) K_hat_ij (x_i - x_j)
//   dl/dlogs  = -(1/sigma^2) sum_ij lambda_i w_j K_hat_ij ||x_i - x_j||^2
//   dl/dlogg  = -gamma lambda^T w.
// The coefficient c_ij = (lambda_i w_j + lambda_j w_i) K_hat_ij is symmetric, so
// one pass over the pairs needs one vector and one scalar per target row,
//   A_i = sum_j c_ij D_ij,   S_i = sum_j c_ij ||D_ij||^2,
// with D_ij = x_i - x_j in scaled coordinates, and
//   dl/dx_i = A_i / (sigma^2 c),  dl/dlogs = -1/2 sum_i S_i / (sigma^2 c^2)
// (c the coordinate scale; lambda == w: c_ij = 2 w_i w_j K_hat_ij, whose 2 w_i the
// finish applies, once per row).  The FP32 pass keeps the sums with w and with lambda
// apart (sum_j w_j K_hat_ij D_ij, the same with lambda_j, and sum_j w_j K_hat_ij
// ||D_ij||^2) and multiplies by lambda_i and w_i in FP64.  Precision: FP64 throughout, or FP32 offsets, kernel
// values and sums.  At a solution w of an ill-conditioned system (|w| large with
// alternating signs) the row sums cancel heavily, so the FP32 gradient carries
// relative row errors far above FP32 rounding; FP64 is small beside the solve
// that produces w.
#include <type_traits>

#include "krylov.h"

namespace krr {

template <typename T>
struct GP;
template <>
struct GP<float> {
    static __device__ __forceinline__ float ex2(float a) { return __builtin_amdgcn_exp2f(a); }
    static __device__ __forceinline__ float fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
};
template <>
struct GP<double> {
    static __device__ __forceinline__ double ex2(double a) { return exp2_f64(a); }
    static __device__ __forceinline__ double fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
};

struct GArgs {
    int64_t n, n_pad;
    int ntiles, nrowblocks, splits, tps;
    const double *anchor;
    const double *tile_r2;
    const double *box;  // tile boxes (krr_internal.h)
    bool rest = false;  // VALU form: only the row tiles that mg_tile refuses
    const void *off;  // offsets in the pass's precision, SoA
    const void *ws;   // w in sorted order
    const void *ls;   // lambda in sorted order
    void *parts;      // [splits][n_pad][grad_sums]: A_i, S_i of a column range
};

// Sums of a row: A_i and S_i; FP32 with lambda != w two vectors and S_i.
template <typename T>
__host__ __device__ constexpr int grad_sums(int dpad, bool same) {
    return sizeof(T) == 8 || same ? dpad + 1 : 2 * dpad + 1;
}

// Row tiles up to this R^2, all coordinates finite, take the matrix-core form.
constexpr double MG_R2 = 4.0;
template <int D>
__device__ __forceinline__ bool finite_tile(const GArgs &a, int J) {
    return a.box[static_cast<int64_t>(J) * BOX * D] != -INFINITY;
}
template <int D>
__device__ __forceinline__ bool mg_tile(const GArgs &a, int I) {
    return a.tile_r2[I] <= MG_R2 && finite_tile<D>(a, I);
}

// VALU form: one lane per target row, sources at wave-uniform addresses (scalar
// loads); explicit differences.
template <int D, bool SAME, typename T>
__global__ __launch_bounds__(BLOCK) void k_grad(GArgs a) {
    constexpr int NA = grad_sums<T>(D, SAME);
    constexpr bool TWO = NA > D + 1;      // sums with lambda apart
    constexpr bool APART = sizeof(T) == 4;  // row factors left to the finish
    constexpr int U = D <= 4 ? 8 : D <= 8 ? 4 : 2;
    using G = GP<T>;
    const T *__restrict__ off = static_cast<const T *>(a.off);
    const T *__restrict__ wsrc = static_cast<const T *>(a.ws);
    const T *__restrict__ lsrc = static_cast<const T *>(a.ls);
    const int64_t n_pad = a.n_pad;
    const int bx = blockIdx.x % a.nrowblocks, by = blockIdx.x / a.nrowblocks;
    if (a.rest && mg_tile<D>(a, bx)) return;
    const int64_t i = static_cast<int64_t>(bx) * BLOCK + threadIdx.x;
    double aI[D];
    T oi[D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
        aI[k] = a.anchor[static_cast<int64_t>(bx) * D + k];
        oi[k] = off[k * n_pad + i];
    }
    const T wi = SAME || APART ? T(0) : wsrc[i], li = SAME || APART ? T(0) : lsrc[i];
    T A[D], Al[TWO ? D : 1], S = T(0);
#pragma unroll
    for (int k = 0; k < D; ++k) {
        A[k] = T(0);
        if (TWO) Al[k] = T(0);
    }
    const int J0 = by * a.tps;
    const int J1 = min(a.ntiles, J0 + a.tps);
    for (int J = J0; J < J1; ++J) {
        T t[D];
#pragma unroll
        for (int k = 0; k < D; ++k)
            t[k] = static_cast<T>((aI[k] - a.anchor[static_cast<int64_t>(J) * D + k]) + static_cast<double>(oi[k]));
        const int64_t j0 = static_cast<int64_t>(J) * TILE;
        for (int jb = 0; jb < TILE; jb += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t j = j0 + jb + u;
                T dl[D];
                T r2 = T(0);
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    dl[k] = t[k] - off[k * n_pad + j];
                    r2 = G::fma(dl[k], dl[k], r2);
                }
                const T kv = G::ex2(-r2);
                const T c = kv * (SAME || APART ? wsrc[j] : G::fma(li, wsrc[j], lsrc[j] * wi));
                S = G::fma(c, r2, S);
#pragma unroll
                for (int k = 0; k < D; ++k) A[k] = G::fma(c, dl[k], A[k]);
                if constexpr (TWO) {
                    const T cl = kv * lsrc[j];
#pragma unroll
                    for (int k = 0; k < D; ++k) Al[k] = G::fma(cl, dl[k], Al[k]);
                }
            }
        }
    }
    T *out = static_cast<T *>(a.parts) + (static_cast<int64_t>(by) * n_pad + i) * NA;
#pragma unroll
    for (int k = 0; k < D; ++k) out[k] = A[k];
    if constexpr (TWO)
#pragma unroll
        for (int k = 0; k < D; ++k) out[D + k] = Al[k];
    out[NA - 1] = S;
}

// FP64 matrix-core form, compiled dimensions 12 and 16.  Both contractions of a
// pair run on v_mfma_f64_16x16x4f64: the squared distance, -TN ||t' - o'||^2 =
// [2 TN t', -TN |t'|^2, TN, TN] . [o', 1, -e0, -e1], and the row sums c_ij o'_j
// (c as A operand straight from the exponents' accumulator layout, the sources'
// coordinates as the 16 columns of B).  All coordinates are taken from the row
// tile's anchor, x' = x - a_I (sources shifted when they are staged, |o'|^2 =
// e0 + e1 in the two halves the staging threads hold), so the target operand is
// built once per block and A_i = t'_i sum_j c_ij - sum_j c_ij o'_j.  The VALU does
// the table exponential and the coefficient.  A pair costs no subtraction and no
// fused multiply-add per coordinate: at N = 50,000, d = 16 the pass took 7.7 ms in
// the VALU form with lambda and w summed apart.
//
// The expanded distance carries an absolute error of a few 2^-53 |t'|^2, whatever
// the distance.  So a row tile takes this form only up to R^2 = MG_R2 (its
// own |t'|^2; the sources that matter are within a few scaled units of it), and
// pairs closer than r^2 = R^2 MG_NEAR, whose r^2 would lose its relative accuracy,
// are formed again from their differences (rare: the wave looks at the smallest of
// its 512 exponents; a fixed line of 1/64 met every pair of smooth kernels, N = 20,000,
// d = 12, sigma = 5 sqrt(d) 1.5 ms against 0.8); wider row tiles are left to k_grad.  Relative error of gx
// against the explicit form's, N about 1000:
//   N(0, I), d = 9-16, R^2 2-4.6: 6.6e-16 - 1.0e-15, against 6.8e-16 - 1.2e-15
//   (R^2 11-31: 0.9-2.3e-15 against 0.8-1.3e-15: beyond the line);
//   40 clusters spread by 1e4 (R^2 1e9): 2e-7 against 2e-12 without the line.
// A wave owns 2 groups of 16 targets, a block 128 rows of a row tile; sources are
// staged 128 at a time, double-buffered (45 KB, two blocks per CU by registers).
typedef double gdx4 __attribute__((ext_vector_type(4)));
typedef double gdx2 __attribute__((ext_vector_type(2)));

constexpr double MG_NEAR = 1.0 / 256.0;
__device__ __forceinline__ unsigned high_word(double v) {
    return static_cast<unsigned>(__builtin_bit_cast(unsigned long long, v) >> 32);
}

template <int D, bool SAME>
__global__ __launch_bounds__(BLOCK, 2) void k_grad_mg(GArgs a) {
    static_assert(D == 12 || D == 16, "one 16-column block of coordinates; whole chunks");
    constexpr int NA = D + 1, TN = 256, RG = 2, ROWS = 128, SC = 128, CPT = TILE / SC;
    constexpr int DK = D / 4 + 1;
    constexpr int LDO = SC + 18;  // row stride 144 mod 256 bytes: both operands' reads spread over the banks
    constexpr int PER = D / 2;    // coordinates staged per thread
    __shared__ __align__(16) double s_o[2][16][LDO];
    __shared__ __align__(16) double s_w[2][SC], s_l[SAME ? 1 : 2][SC];
    __shared__ double s_e[2][2][SC];
    __shared__ double s_tab[TN];
    const double *__restrict__ off = static_cast<const double *>(a.off);
    const double *__restrict__ wsrc = static_cast<const double *>(a.ws);
    const double *__restrict__ lsrc = static_cast<const double *>(a.ls);
    const int64_t n_pad = a.n_pad;
    const int nrb = 2 * a.nrowblocks;
    const int bh = blockIdx.x % nrb, by = blockIdx.x / nrb;
    const int I = bh / 2;
    if (!mg_tile<D>(a, I)) return;
    // x > -TN R^2 MG_NEAR (and x > 0, from rounding): high words below that of the
    // bound, as unsigned numbers
    const unsigned near_hi = __builtin_amdgcn_readfirstlane(high_word(-TN * MG_NEAR * a.tile_r2[I]));
    const int tid = threadIdx.x, lane = tid % WAVE, r16 = lane % 16, g = lane / 16;
    // source of A row r16, so that lane l's four exponents are sources 4 g + v
    const int asrc = (r16 % 4) * 4 + r16 / 4;
    const int64_t row0 = static_cast<int64_t>(I) * TILE + (bh % 2) * ROWS + (tid / WAVE) * (16 * RG);
    for (int k = tid; k < TN; k += BLOCK) s_tab[k] = EXP2_TABLE256[k];
    if constexpr (D < 16) {  // the unused coordinate columns stay zero
        for (int k = D * LDO + tid; k < 16 * LDO; k += BLOCK) s_o[0][0][k] = s_o[1][0][k] = 0.0;
    }

    // the target operand of each group: coordinate 4 kc + g of its slots
    double bval[RG][DK], li[RG], wi[RG];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        const int64_t i = row0 + rg * 16 + r16;
        double tt = 0.0;
#pragma unroll
        for (int kc = 0; kc < D / 4; ++kc) {
            const double t = off[(4 * kc + g) * n_pad + i];
            bval[rg][kc] = 2.0 * TN * t;
            tt = __builtin_fma(t, t, tt);
        }
        tt += __shfl_xor(tt, 16, WAVE);
        tt += __shfl_xor(tt, 32, WAVE);
        bval[rg][D / 4] = g == 0 ? -TN * tt : (g < 3 ? static_cast<double>(TN) : 0.0);
        li[rg] = SAME ? 0.0 : lsrc[i];
        wi[rg] = wsrc[i];
    }
    // staging: source tid % 128, coordinates PER (tid / 128) .. + PER - 1
    const int scol = tid % SC, shalf = tid / SC;
    double st_o[PER], st_w = 0.0, st_l = 0.0;
    auto stage_load = [&](int ci) {
        const int J = ci / CPT;
        const int64_t j = static_cast<int64_t>(ci) * SC + scol;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int kk = shalf * PER + k;
            const double sh = a.anchor[static_cast<int64_t>(J) * D + kk] - a.anchor[static_cast<int64_t>(I) * D + kk];
            st_o[k] = off[kk * n_pad + j] + sh;
        }
        if (shalf == 0) st_w = wsrc[j];
        if (!SAME && shalf == 1) st_l = lsrc[j];
    };
    auto stage_store = [&](int ci, int buf) {
        const int64_t j = static_cast<int64_t>(ci) * SC + scol;
        double e = 0.0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            s_o[buf][shalf * PER + k][scol] = st_o[k];
            e = __builtin_fma(st_o[k], st_o[k], e);
        }
        // the padding, which would lie at its tile's anchor, goes far away
        s_e[buf][shalf][scol] = j < a.n ? -e : -e - 1e6;
        if (shalf == 0) s_w[buf][scol] = st_w;
        if (!SAME && shalf == 1) s_l[SAME ? 0 : buf][scol] = st_l;
    };
    gdx4 acc[RG];
    double cs[RG], S[RG];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        acc[rg] = gdx4{0.0, 0.0, 0.0, 0.0};
        cs[rg] = S[rg] = 0.0;
    }
    const int C0 = by * a.tps * CPT, C1 = min(a.ntiles, (by + 1) * a.tps) * CPT;
    if (C0 < C1) {
        stage_load(C0);
        stage_store(C0, 0);
    }
    __syncthreads();
    for (int ci = C0; ci < C1; ++ci) {
        const int buf = (ci - C0) & 1;
        if (ci + 1 < C1) stage_load(ci + 1);
        auto exponents = [&](int st, gdx4 (&G)[RG]) {
            double av[DK];
#pragma unroll
            for (int kc = 0; kc < D / 4; ++kc) av[kc] = s_o[buf][4 * kc + g][st + asrc];
            // slots [1, -e0, -e1, 0]
            const double e = s_e[buf][g == 2 ? 1 : 0][st + asrc];
            av[D / 4] = g == 0 ? 1.0 : (g < 3 ? e : 0.0);
#pragma unroll
            for (int rg = 0; rg < RG; ++rg) {
                G[rg] = gdx4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int kc = 0; kc < DK; ++kc)
                    G[rg] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[kc], bval[rg][kc], G[rg], 0, 0, 0);
            }
        };
        auto near_pairs = [&](auto diag_c, int st, gdx4 (&G)[RG]) {
            auto near = [&](int rg, int v) {
                const int64_t j = static_cast<int64_t>(ci) * SC + st + 4 * g + v;
                return high_word(G[rg][v]) < near_hi && !(decltype(diag_c)::value && j == row0 + rg * 16 + r16);
            };
            bool any = false;
            if constexpr (decltype(diag_c)::value) {
#pragma unroll
                for (int e = 0; e < 4 * RG; ++e) any = any || near(e / 4, e % 4);
            } else {
                unsigned least = high_word(G[0][0]);
#pragma unroll
                for (int e = 1; e < 4 * RG; ++e) least = min(least, high_word(G[e / 4][e % 4]));
                any = least < near_hi;
            }
            if (__builtin_expect(__ballot(any) == 0, 1)) return;
            // every pair of the lane at once: copies of ten points, N = 50,000, d = 16, 5.6 ms
            // (one close pair after the other 7.9; distinct points 4.5)
#pragma unroll
            for (int rg = 0; rg < RG; ++rg) {
                double r2[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
                for (int k = 0; k < D; ++k) {
                    const double t = off[k * n_pad + row0 + rg * 16 + r16];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const double dl = t - s_o[buf][k][st + 4 * g + v];
                        r2[v] = __builtin_fma(dl, dl, r2[v]);
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) G[rg][v] = near(rg, v) ? -TN * r2[v] : G[rg][v];
            }
        };
        // DIAG: the chunk holds the rows' own points, whose D_ii = 0 adds nothing;
        // their (largest) coefficient is left out so that it does not have to cancel
        // between t'_i sum c and sum c o'
        auto accumulate = [&](auto diag_c, int st, gdx4 (&G)[RG]) {
            constexpr bool DIAG = decltype(diag_c)::value;
            near_pairs(diag_c, st, G);
            // this lane's sources 4 g + v: weights, and coordinate r16 for the second contraction
            double wv[4], lv[4], ov[4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const gdx2 w2 = *reinterpret_cast<const gdx2 *>(&s_w[buf][st + 4 * g + 2 * h]);
                const gdx2 o2 = *reinterpret_cast<const gdx2 *>(&s_o[buf][r16][st + 4 * g + 2 * h]);
                wv[2 * h] = w2[0];
                wv[2 * h + 1] = w2[1];
                ov[2 * h] = o2[0];
                ov[2 * h + 1] = o2[1];
                if constexpr (!SAME) {
                    const gdx2 l2 = *reinterpret_cast<const gdx2 *>(&s_l[buf][st + 4 * g + 2 * h]);
                    lv[2 * h] = l2[0];
                    lv[2 * h + 1] = l2[1];
                }
            }
#pragma unroll
            for (int rg = 0; rg < RG; ++rg)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    // far pairs: the exponential is 0 from -1100 on; keeps x in int range
                    const double x = __builtin_fmax(G[rg][v], -2000.0 * TN);
                    const double e = exp2_tab<TN>(x, s_tab);
                    double u;
                    if constexpr (SAME)
                        u = wv[v];
                    else
                        u = __builtin_fma(li[rg], wv[v], lv[v] * wi[rg]);
                    double c = e * u;
                    if constexpr (DIAG) {
                        const int64_t j = static_cast<int64_t>(ci) * SC + st + 4 * g + v;
                        c = j == row0 + rg * 16 + r16 ? 0.0 : c;
                    }
                    cs[rg] += c;
                    S[rg] = __builtin_fma(c, x, S[rg]);
                    acc[rg] = __builtin_amdgcn_mfma_f64_16x16x4f64(c, ov[v], acc[rg], 0, 0, 0);
                }
        };
        // the matrix cores form a step's exponents while the VALU takes the one
        // before; not unrolled further (the compiler would spill 150 registers)
        auto chunk = [&](auto diag_c) {
            gdx4 G0[RG], G1[RG];
            exponents(0, G0);
#pragma unroll 1
            for (int st = 0; st < SC; st += 32) {
                exponents(st + 16, G1);
                accumulate(diag_c, st, G0);
                if (st + 32 < SC) exponents(st + 32, G0);
                accumulate(diag_c, st + 16, G1);
            }
        };
        // the clamp of x below hides a NaN distance, whose r^2 belongs into S
        if (!finite_tile<D>(a, ci / CPT)) S[0] = S[1] = NAN;
        if (ci / CPT == I)
            chunk(std::true_type{});
        else
            chunk(std::false_type{});
        if (ci + 1 < C1) stage_store(ci + 1, buf ^ 1);
        __syncthreads();
    }
    // A_i = t'_i C_i - sum c o'; accumulator lane l: target g + 4 v, coordinate r16
    double *__restrict__ parts = static_cast<double *>(a.parts) + static_cast<int64_t>(by) * n_pad * NA;
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        double c = cs[rg], s = S[rg];
        c += __shfl_xor(c, 16, WAVE);
        c += __shfl_xor(c, 32, WAVE);
        s += __shfl_xor(s, 16, WAVE);
        s += __shfl_xor(s, 32, WAVE);
        if (g == 0) parts[(row0 + rg * 16 + r16) * NA + D] = s * (-1.0 / TN);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int it = g + 4 * v;
            const double ct = __shfl(c, it, WAVE);
            const int64_t i = row0 + rg * 16 + it;
            if (r16 < D) {
                const double t = off[r16 * n_pad + i];
                parts[i * NA + r16] = __builtin_fma(t, ct, -acc[rg][v]);
            }
        }
    }
}

// Sorted copies of lambda and w in the pass's precision (0 on the padding).
template <typename T>
__global__ __launch_bounds__(BLOCK) void k_grad_gather(const int32_t *__restrict__ perm, int64_t n_pad,
                                                       const double *__restrict__ lam, const double *__restrict__ w,
                                                       T *ls, T *ws) {
    const int64_t i = blockIdx.x * static_cast<int64_t>(BLOCK) + threadIdx.x;
    if (i >= n_pad) return;
    const int32_t p = perm[i];
    ls[i] = p >= 0 ? static_cast<T>(lam[p]) : T(0);
    ws[i] = p >= 0 ? static_cast<T>(w[p]) : T(0);
}

template <typename T>
__device__ __forceinline__ T gwave_sum(T v) {
#pragma unroll
    for (int o = WAVE / 2; o > 0; o /= 2) v += __shfl_xor(v, o, WAVE);
    return v;
}

// gx[p_i, k] = A_ik / (sigma^2 c) (FP32: lambda_i and w_i times the row's two sums;
// FP64 with lambda == w: 2 w_i times the row's sum.  In the pass itself that factor cost
// 30 more spilled registers at d = 60, N = 25,000 30.9 ms against 25.4),
// the column ranges added in order; sums S_i (lambda_i S_i) and lambda_p w_p over the
// rows (last block writes the two scalars).  One thread per (row, k) entry, so the reads run along memory
// (one row per thread walking its 2 D + 1 entries took 614 us at N = 50,000,
// d = 16).
template <typename T>
__global__ __launch_bounds__(BLOCK) void k_grad_finish(int64_t n, int64_t n_pad, int d, int dpad, int splits,
                                                       bool same, const int32_t *__restrict__ perm,
                                                       const T *__restrict__ parts, const double *__restrict__ lam,
                                                       const double *__restrict__ w, double inv_s2c,
                                                       double inv_s2c2, double gamma, double *gx, double *g_ls,
                                                       double *g_lg, double *partials, unsigned *counter) {
    constexpr bool APART = sizeof(T) == 4;
    const int ne = dpad + 1, NA = grad_sums<T>(dpad, same);
    double accS = 0.0, accG = 0.0;
    for (int64_t e = blockIdx.x * static_cast<int64_t>(BLOCK) + threadIdx.x; e < n * ne;
         e += static_cast<int64_t>(gridDim.x) * BLOCK) {
        const int64_t i = e / ne;
        const int k = static_cast<int>(e - i * ne);
        if (k >= d && k < dpad) continue;
        const int64_t p = perm[i];
        auto sum = [&](int c) {
            double v = 0.0;
            for (int u = 0; u < splits; ++u)
                v += static_cast<double>(parts[(static_cast<int64_t>(u) * n_pad + i) * NA + c]);
            return v;
        };
        double s = sum(k < d ? k : NA - 1);
        if constexpr (APART)
            s = k < d ? lam[p] * s + w[p] * (same ? s : sum(dpad + k)) : lam[p] * s;
        else if (same)
            s *= 2.0 * w[p];
        if (k < d) {
            gx[p * d + k] = s * inv_s2c;
        } else {
            accS += s;
            accG += lam[p] * w[p];
        }
    }
    // deterministic grid reduction of the two scalars (last block)
    __shared__ double sh[2][BLOCK / WAVE];
    __shared__ int is_last;
    accS = gwave_sum(accS);
    accG = gwave_sum(accG);
    if (threadIdx.x % WAVE == 0) {
        sh[0][threadIdx.x / WAVE] = accS;
        sh[1][threadIdx.x / WAVE] = accG;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a0 = 0.0, a1 = 0.0;
        for (int k = 0; k < BLOCK / WAVE; ++k) {
            a0 += sh[0][k];
            a1 += sh[1][k];
        }
        partials[blockIdx.x] = a0;
        partials[gridDim.x + blockIdx.x] = a1;
        __threadfence();
        is_last = (atomicAdd(counter, 1u) == gridDim.x - 1);
    }
    __syncthreads();
    if (!is_last || threadIdx.x >= WAVE) return;
    __threadfence();
    double s0 = 0.0, s1 = 0.0;
    for (unsigned b = threadIdx.x; b < gridDim.x; b += WAVE) {
        s0 += __hip_atomic_load(&partials[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s1 += __hip_atomic_load(&partials[gridDim.x + b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    s0 = gwave_sum(s0);
    s1 = gwave_sum(s1);
    if (threadIdx.x != 0) return;
    *g_ls = (APART ? -1.0 : -0.5) * s0 * inv_s2c2;
    *g_lg = -gamma * s1;
    *counter = 0u;
}

__global__ void k_zero_u32(unsigned *p) {
    if (threadIdx.x == 0) *p = 0u;
}

// ---------------------------------------------------------------- host

// Column ranges: about 4096 blocks of 256 rows (2048 x 2 half tiles).
static int grad_splits(const Prepared &P) {
    int s = (4096 + P.ntiles - 1) / P.ntiles;
    int mx = P.ntiles / 2 > 1 ? P.ntiles / 2 : 1;
    if (mx > 32) mx = 32;
    if (s > mx) s = mx;
    return s < 1 ? 1 : s;
}

size_t grad_scratch_bytes(const Prepared &P) {
    const int mx = (P.ntiles / 2 > 1 ? (P.ntiles / 2 < 32 ? P.ntiles / 2 : 32) : 1);
    return align_up(static_cast<size_t>(mx) * P.n_pad * (P.dpad + 1) * 8, 256) +
           2 * align_up(static_cast<size_t>(P.n_pad) * 8, 256) + align_up(2 * VEC_BLOCKS * 8, 256) + 256;
}

template <int D, typename T>
static hipError_t launch_grad(const GArgs &a, bool same, hipStream_t s) {
    // FP64 at the compiled dimensions 12 and 16: below, the matrix-core form's 16
    // coordinate columns and padded slots cost more than the VALU's d subtractions
    // and 2 d fused multiply-adds on large sets (d = 8, VALU / matrix cores: N = 50,000
    // 3.60 / 3.78 ms, N = 10,000 0.30 / 0.29, N = 1000 0.17 / 0.09); above 16 its
    // operands do not fit.  FP32 stays on the VALU, which keeps D_ij = x_i - x_j
    // itself in FP32.  The wide row tiles are
    // a launch of their own (its blocks return at once on compact ones; inside the
    // matrix-core kernel, at 2 waves per SIMD, they took 2.5 times as long).
    GArgs v = a;
    if constexpr (sizeof(T) == 8 && (D == 12 || D == 16)) {
        v.rest = true;
        const dim3 g(2 * a.nrowblocks * a.splits);
        if (same)
            hipLaunchKernelGGL((k_grad_mg<D, true>), g, dim3(BLOCK), 0, s, a);
        else
            hipLaunchKernelGGL((k_grad_mg<D, false>), g, dim3(BLOCK), 0, s, a);
        KRR_HIP(hipGetLastError());
    }
    if (same)
        hipLaunchKernelGGL((k_grad<D, true, T>), dim3(a.nrowblocks * a.splits), dim3(BLOCK), 0, s, v);
    else
        hipLaunchKernelGGL((k_grad<D, false, T>), dim3(a.nrowblocks * a.splits), dim3(BLOCK), 0, s, v);
    return hipGetLastError();
}

template <typename T>
static hipError_t grad_pass(const Prepared &P, double sigma, double gamma, const double *lam, const double *w,
                            double *gx, double *g_ls, double *g_lg, void *scratch, hipStream_t s) {
    const bool same = (lam == w);
    const int mx = (P.ntiles / 2 > 1 ? (P.ntiles / 2 < 32 ? P.ntiles / 2 : 32) : 1);
    Carver cv(scratch);
    GArgs a;
    T *parts = cv.take<T>(static_cast<size_t>(mx) * P.n_pad * grad_sums<T>(P.dpad, same));
    T *ls = cv.take<T>(P.n_pad);
    T *wsv = cv.take<T>(P.n_pad);
    double *partials = cv.take<double>(2 * VEC_BLOCKS);
    unsigned *counter = cv.take<unsigned>(1);
    const int splits_req = grad_splits(P);
    a.n = P.n;
    a.n_pad = P.n_pad;
    a.ntiles = P.ntiles;
    a.nrowblocks = P.ntiles;
    a.tps = (P.ntiles + splits_req - 1) / splits_req;
    a.splits = (P.ntiles + a.tps - 1) / a.tps;
    a.anchor = P.anchor;
    a.tile_r2 = P.tile_r2;
    a.box = P.box;
    a.off = sizeof(T) == 8 ? static_cast<const void *>(P.off64) : static_cast<const void *>(P.off32);
    a.ws = wsv;
    a.ls = ls;
    a.parts = parts;
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, s, counter);
    hipLaunchKernelGGL(k_grad_gather<T>, dim3((P.n_pad + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, P.perm, P.n_pad, lam,
                       w, ls, wsv);
    KRR_HIP(hipGetLastError());
    hipError_t e;
    switch (P.dpad) {
        case 1: e = launch_grad<1, T>(a, same, s); break;
        case 2: e = launch_grad<2, T>(a, same, s); break;
        case 3: e = launch_grad<3, T>(a, same, s); break;
        case 4: e = launch_grad<4, T>(a, same, s); break;
        case 6: e = launch_grad<6, T>(a, same, s); break;
        case 8: e = launch_grad<8, T>(a, same, s); break;
        case 12: e = launch_grad<12, T>(a, same, s); break;
        case 16: e = launch_grad<16, T>(a, same, s); break;
        case 24: e = launch_grad<24, T>(a, same, s); break;
        case 32: e = launch_grad<32, T>(a, same, s); break;
        case 48: e = launch_grad<48, T>(a, same, s); break;
        case 64: e = launch_grad<64, T>(a, same, s); break;
        default: e = hipErrorInvalidValue;
    }
    KRR_HIP(e);
    const double c = P.scale;
    const double s2 = sigma * sigma;
    hipLaunchKernelGGL(k_grad_finish<T>, dim3(vec_blocks(P.n_pad * (P.dpad + 1))), dim3(BLOCK), 0, s, P.n, P.n_pad, P.d, P.dpad,
                       a.splits, same, P.perm, parts, lam, w, 1.0 / (s2 * c), 1.0 / (s2 * c * c), gamma,
                       gx, g_ls, g_lg, partials, counter);
    return hipGetLastError();
}

hipError_t kmvp_grad_run(const Prepared &P, int prec, double sigma, double gamma, const double *lam,
                         const double *w, double *gx, double *g_ls, double *g_lg, void *scratch, hipStream_t s) {
    if (prec == KRR_FP64) return grad_pass<double>(P, sigma, gamma, lam, w, gx, g_ls, g_lg, scratch, s);
    return grad_pass<float>(P, sigma, gamma, lam, w, gx, g_ls, g_lg, scratch, s);
}

}  // namespace krr
