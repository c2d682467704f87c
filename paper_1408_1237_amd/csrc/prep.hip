// Point preparation for the kernel products: scaling, Morton ordering, tile
// anchors and per-precision offsets and weights (layout described in
// krr_internal.h).  Runs once per solve; O(N log N) and negligible next to the
// O(N^2) products.
#include <rocprim/device/device_radix_sort.hpp>

#include <cmath>

#include "krr_internal.h"
#include "split16.h"

namespace krr {

constexpr int BBOX_BLOCKS = 64;  // slices of the bounding box pass (one lane each in k_morton)
constexpr int BBOX_THREADS = 1024;

static const int kDims[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64};

int dim_instance(int d) {
    for (int v : kDims)
        if (v >= d) return v;
    return 0;
}

Prepared carve_prepared(Carver &cv, int64_t n, int d) {
    Prepared P;
    P.n = n;
    P.d = d;
    P.dpad = dim_instance(d);
    P.n_pad = (n + TILE - 1) / TILE * TILE;
    P.ntiles = static_cast<int>(P.n_pad / TILE);
    P.perm = cv.take<int32_t>(P.n_pad);
    P.anchor = cv.take<double>(static_cast<size_t>(P.ntiles) * P.dpad);
    P.tile_r2 = cv.take<double>(P.ntiles);
    P.tile_nj = cv.take<double>(P.ntiles);
    P.tile_far = cv.take<float>(P.ntiles);
    P.tile_far64 = cv.take<float>(P.ntiles);
    P.off64 = cv.take<double>(static_cast<size_t>(P.dpad) * P.n_pad);
    P.off32 = cv.take<float>(static_cast<size_t>(P.dpad) * P.n_pad);
    P.offb = cv.take<float>(static_cast<size_t>(P.dpad) * P.n_pad);
    P.w64 = cv.take<double>(P.n_pad);
    P.w32 = cv.take<float>(P.n_pad);
    P.w16 = cv.take<float>(P.n_pad);
    P.sq64 = cv.take<double>(P.n_pad);
    if (P.dpad > 16) {
        P.pm64 = cv.take<double>(static_cast<size_t>(P.dpad) * P.n_pad);
        P.pm32 = cv.take<float>(static_cast<size_t>(P.dpad) * P.n_pad);
        P.pmb = cv.take<float>(static_cast<size_t>(P.dpad) * P.n_pad);
    }
    const int oct = 2 * split_chunks(P.dpad);
    if (oct > 0) {
        P.slot32 = cv.take<half8_t>(static_cast<size_t>(oct) * P.n_pad);
        P.slot16 = cv.take<half8_t>(static_cast<size_t>(oct) * P.n_pad);
    }
    if (P.dpad <= 16) {
        P.box = cv.take<double>(BOX * static_cast<size_t>(P.ntiles) * P.dpad);
        P.sub_reach = cv.take<int>(static_cast<size_t>(P.ntiles) * (TILE / SUB));
    }
    P.flags = cv.take<int>(4);
    return P;
}

size_t prepared_bytes(int64_t n, int d) {
    Carver cv(nullptr);
    carve_prepared(cv, n, d);
    return cv.off + 256;
}

// keys (2 buffers) + values (2 buffers) + bbox + sort scratch bound
static size_t sort_scratch_bound(int64_t n) { return (size_t(16) << 20) + static_cast<size_t>(n) * 16; }

size_t prep_temp_bytes(int64_t n) {
    Carver cv(nullptr);
    cv.take<uint64_t>(n);
    cv.take<uint64_t>(n);
    cv.take<int32_t>(n);
    cv.take<int32_t>(n);
    cv.take<double>(2 * KRR_MAX_DIM * BBOX_BLOCKS);
    cv.take<int>(KRR_MAX_DIM * BBOX_BLOCKS);
    cv.take<char>(sort_scratch_bound(n));
    return cv.off + 256;
}

// ---------------------------------------------------------------- reductions

template <typename T, class Op>
__device__ T block_reduce(T v, Op op, T *lds /* >= BLOCK/WAVE */) {
#pragma unroll
    for (int off = WAVE / 2; off > 0; off /= 2) v = op(v, __shfl_xor(v, off, WAVE));
    const int w = threadIdx.x / WAVE;
    if ((threadIdx.x % WAVE) == 0) lds[w] = v;
    __syncthreads();
    T r = lds[0];
    for (int k = 1; k < static_cast<int>(blockDim.x) / WAVE; ++k) r = op(r, lds[k]);
    __syncthreads();
    return r;
}

struct MaxOp { __device__ double operator()(double a, double b) const { return fmax(a, b); } };

// ---------------------------------------------------------------- kernels

// Bounding box, first half: block (blk, t) takes the min / max of the scaled
// coordinate t over its slice of the points; part[(t * 2 + 0|1) * nblk + blk].
// bad[t * nblk + blk]: a non-finite coordinate in the slice.  The few partials
// (at most BBOX_BLOCKS per coordinate) are combined by every block of k_morton,
// which takes the place of a kernel whose one thread per coordinate walked up to
// 1024 of them (N = 1e5, d = 3: 55 us; with the fill of the flags, three launches
// became one).
__global__ __launch_bounds__(BBOX_THREADS) void k_bbox_partial(const double *__restrict__ x, int64_t n, int d,
                                                               double scale, double *part, int *bad) {
    __shared__ double s_lo[BBOX_THREADS / WAVE], s_hi[BBOX_THREADS / WAVE];
    const int t = blockIdx.y;
    const int nblk = gridDim.x;
    double lo = INFINITY, hi = -INFINITY;
    int nf = 0;
#pragma unroll 4
    for (int64_t i = blockIdx.x * static_cast<int64_t>(BBOX_THREADS) + threadIdx.x; i < n;
         i += static_cast<int64_t>(nblk) * BBOX_THREADS) {
        double v = x[i * d + t];
        nf |= isfinite(v) ? 0 : 1;
        v *= scale;
        lo = fmin(lo, v);
        hi = fmax(hi, v);
    }
#pragma unroll
    for (int off = WAVE / 2; off > 0; off /= 2) {
        lo = fmin(lo, __shfl_xor(lo, off, WAVE));
        hi = fmax(hi, __shfl_xor(hi, off, WAVE));
    }
    if (threadIdx.x % WAVE == 0) {
        s_lo[threadIdx.x / WAVE] = lo;
        s_hi[threadIdx.x / WAVE] = hi;
    }
    nf = __syncthreads_or(nf);
    if (threadIdx.x == 0) {
        for (int w = 1; w < BBOX_THREADS / WAVE; ++w) {
            lo = fmin(lo, s_lo[w]);
            hi = fmax(hi, s_hi[w]);
        }
        part[(t * 2 + 0) * nblk + blockIdx.x] = lo;
        part[(t * 2 + 1) * nblk + blockIdx.x] = hi;
        bad[t * nblk + blockIdx.x] = nf;
    }
}

// Morton code: the first dm = min(d, 63) scaled coordinates quantised to
// bits = min(63 / dm, 31) bits each over the bounding box, bits interleaved.
// Every block combines the box partials itself (one wave per coordinate bound;
// min and max do not depend on the order); block 0 also stores the flags.
__global__ __launch_bounds__(BLOCK) void k_morton(const double *__restrict__ x, int64_t n, int d, double scale,
                                                  const double *__restrict__ part, const int *__restrict__ bad,
                                                  int nblk, int dm, int bits, uint64_t *keys, int32_t *vals,
                                                  int *flags) {
    __shared__ double s_box[2 * KRR_MAX_DIM];
    const int wv = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
    for (int b = wv; b < 2 * dm; b += BLOCK / WAVE) {
        const bool mx = b & 1;
        double v = lane < nblk ? part[b * nblk + lane] : (mx ? -INFINITY : INFINITY);
#pragma unroll
        for (int off = WAVE / 2; off > 0; off /= 2) {
            const double u = __shfl_xor(v, off, WAVE);
            v = mx ? fmax(v, u) : fmin(v, u);
        }
        if (lane == 0) s_box[b] = v;
    }
    if (blockIdx.x == 0) {
        int nf = 0;
        for (int k = threadIdx.x; k < d * nblk; k += BLOCK) nf |= bad[k];
        nf = __syncthreads_or(nf);
        if (threadIdx.x < 4) flags[threadIdx.x] = threadIdx.x == 0 && nf ? 1 : 0;
    }
    __syncthreads();
    const int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x;
    if (i >= n) return;
    const double qmax = static_cast<double>((uint64_t(1) << bits) - 1);
    uint64_t code = 0;
    for (int t = 0; t < dm; ++t) {
        const double lo = s_box[2 * t], hi = s_box[2 * t + 1];
        const double ext = hi - lo;
        double f = ext > 0 ? (x[i * d + t] * scale - lo) / ext : 0.0;
        f = fmin(fmax(f, 0.0), 1.0);
        const uint64_t qt = static_cast<uint64_t>(f * qmax);
        for (int b = 0; b < bits; ++b) code |= ((qt >> b) & 1u) << (b * dm + t);
    }
    keys[i] = code;
    vals[i] = static_cast<int32_t>(i);
}

// Sorted order of a small set by counting: the rank of a key is the number of
// keys below it (ties by index: the stable order of the radix sort).  A block
// ranks 64 keys, one per lane; its 16 waves share the comparisons by chunks of
// 64 keys, read at wave-uniform addresses (scalar loads), two VALU operations
// per comparison.  One launch in place of four to eight.
constexpr int RANK_THREADS = 1024;
constexpr int64_t RANK_MAX_N = 8192;
__global__ __launch_bounds__(RANK_THREADS) void k_rank(const uint64_t *__restrict__ keys, int n, int32_t *order) {
    constexpr int NW = RANK_THREADS / WAVE;
    __shared__ int s_cnt[NW][WAVE];
    const int lane = threadIdx.x % WAVE;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / WAVE);
    const int i = blockIdx.x * WAVE + lane;
    const uint64_t key = i < n ? keys[i] : 0;
    int cnt = 0;
    for (int c = wv; c * WAVE < n; c += NW) {
        const uint64_t *kc = keys + c * WAVE;
        const int m = min(WAVE, n - c * WAVE);
        if (c == static_cast<int>(blockIdx.x)) {
            for (int u = 0; u < m; ++u) cnt += kc[u] < key || (kc[u] == key && u < lane) ? 1 : 0;
        } else {
            // before this block's keys: equal keys come first (key + 1 <= 2^63)
            const uint64_t lim = c < static_cast<int>(blockIdx.x) ? key + 1 : key;
            if (m == WAVE) {
#pragma unroll 16
                for (int u = 0; u < WAVE; ++u) cnt += kc[u] < lim ? 1 : 0;
            } else {
                for (int u = 0; u < m; ++u) cnt += kc[u] < lim ? 1 : 0;
            }
        }
    }
    s_cnt[wv][lane] = cnt;
    __syncthreads();
    if (threadIdx.x < WAVE && i < n) {
        int r = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) r += s_cnt[w][threadIdx.x];
        order[r] = i;
    }
}

// One block per tile: anchor, offsets, radius, normaliser and weights, and the
// slot vectors (split16.h) of the FP32 and BF16 offsets, in the precisions of
// `need` (a product call uses one of the three).
//
// The anchor is the centre of the tile's bounding box, which minimises the
// largest offset, whenever that keeps the tile narrow enough to fold its
// exponent.  A tile too wide to fold anyway (typically a dense group plus a few
// far points that a space-filling order put together) takes the
// coordinate-wise (lower) median instead: it stays inside the group, whose
// offsets then stay short and keep their absolute precision when rounded to
// FP32 or BF16 (with the box centre the group's offsets would be as long as the
// tile, and its pairs' distances would carry that rounding).
//
// What bounds it is latency: a point's coordinates stay in registers (one read),
// the box goes through LDS 16 coordinates at a time with 16 lanes per
// coordinate, and the medians (256 comparisons per point and coordinate) are
// ranked on the wide tiles alone.  Ranking every tile and reducing the box one
// coordinate at a time took 805 us at N = 44,484, d = 41 and 155 us at
// N = 50,021, d = 8, beside products of 749 and 430 us.
//
// Slots.  Gaussian: the offsets o and no source constant.  Matern: o' = log2(e) o
// and the constant |o'|^2, so that the product forms (log2(e) r)^2.
template <int D, bool BF, bool MAT>
__device__ __forceinline__ void store_slots(const Prepared &P, int64_t j, const float (&of)[D]) {
    constexpr int KC = split_chunks(D);
    if constexpr (KC > 0) {
        HiLo v[D];
        double so = 0.0;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            float o = of[k];
            if (MAT) {
                o *= LOG2E_F;
                so = __builtin_fma(static_cast<double>(o), static_cast<double>(o), so);
            }
            v[k] = split_f16(o);
        }
        const HiLo one{static_cast<_Float16>(1.f), static_cast<_Float16>(1.f)};
        const HiLo zero{static_cast<_Float16>(0.f), static_cast<_Float16>(0.f)};
        const HiLo e = MAT ? split_f16(static_cast<float>(so)) : zero;
        half8_t *out = static_cast<half8_t *>(BF ? P.slot16 : P.slot32);
#pragma unroll
        for (int w = 0; w < 2 * KC; ++w) out[w * P.n_pad + j] = slot_octet<D, true>(w, v, one, e);
    }
}

template <int D, bool MAT>
__global__ __launch_bounds__(TILE) void k_tiles(const double *__restrict__ x, int64_t n, int d, double scale,
                                                const int32_t *__restrict__ sorted_idx, Prepared P, int need,
                                                PrepVec pv) {
    constexpr int CH = D < 16 ? D : 16;  // coordinates per pass of the box
    constexpr int LANES = 16;            // lanes per coordinate
    __shared__ double s_v[CH][TILE + 4];
    __shared__ double s_lo[D], s_hi[D], s_median[D];
    __shared__ double lds[TILE / WAVE];
    // D <= 16: per 32 points, the squared extent of each coordinate
    __shared__ double s_ext[D <= 16 ? TILE / SUB : 1][D <= 16 ? D : 1];
    const int J = blockIdx.x, tid = threadIdx.x;
    const int64_t j = static_cast<int64_t>(J) * TILE + tid;
    const bool real = j < n;
    const int32_t idx = real ? sorted_idx[j] : -1;
    const int64_t t0 = static_cast<int64_t>(J) * TILE;
    const int nreal = static_cast<int>(n - t0 < TILE ? n - t0 : TILE);  // real points come first in a tile
    P.perm[j] = idx;
    double xr[D];  // the point's coordinates, unscaled (0 beyond d and on the padding)
#pragma unroll
    for (int t = 0; t < D; ++t) xr[t] = (real && t < d) ? x[static_cast<int64_t>(idx) * d + t] : 0.0;
    // the minima and maxima below pass a NaN over (the anchor is that of the finite
    // points); a tile with a non-finite coordinate stores unbounded boxes
    bool unbounded = false;
    if constexpr (D <= 16) {
        int nf = 0;
#pragma unroll
        for (int t = 0; t < D; ++t) nf |= isfinite(xr[t] * scale) ? 0 : 1;
        unbounded = __syncthreads_or(nf) != 0;
    }
#pragma unroll
    for (int c0 = 0; c0 < D; c0 += CH) {
#pragma unroll
        for (int k = 0; k < CH; ++k)
            if (c0 + k < D) s_v[k][tid] = real ? xr[c0 + k] * scale : NAN;  // fmin / fmax pass a NaN over
        __syncthreads();
        const int k = tid / LANES, part = tid % LANES;
        if (D > 16 && k < CH && c0 + k < D) {
            double lo = INFINITY, hi = -INFINITY;
#pragma unroll
            for (int i = 0; i < TILE / LANES; ++i) {
                const double v = s_v[k][i * LANES + part];
                lo = fmin(lo, v);
                hi = fmax(hi, v);
            }
#pragma unroll
            for (int off = LANES / 2; off > 0; off /= 2) {
                lo = fmin(lo, __shfl_xor(lo, off, WAVE));
                hi = fmax(hi, __shfl_xor(hi, off, WAVE));
            }
            if (part == 0) {
                s_lo[c0 + k] = lo;
                s_hi[c0 + k] = hi;
            }
        }
        if constexpr (D <= 16) {
            const int sub = tid % (TILE / SUB), kk = tid / (TILE / SUB);
            if (kk < D) {
                double lo = INFINITY, hi = -INFINITY;
#pragma unroll
                for (int i = 0; i < SUB; ++i) {
                    // rotated by the eighth: its 8 lanes of a coordinate read other banks
                    const double v = s_v[kk][sub * SUB + ((i + 2 * sub) & (SUB - 1))];
                    lo = fmin(lo, v);
                    hi = fmax(hi, v);
                }
                s_ext[sub][kk] = (hi - lo) * (hi - lo);
                // the eighths' boxes (neighbouring lanes) make those of the halves and
                // of the tile
                double *bx = P.box + static_cast<int64_t>(J) * BOX * D + kk;
#pragma unroll
                for (int off = 1; off < TILE / SUB; off *= 2) {
                    if (off == TILE / SUB / 2 && (sub & (off - 1)) == 0) {
                        bx[(2 + sub / off * 2) * D] = unbounded ? -INFINITY : lo;
                        bx[(3 + sub / off * 2) * D] = unbounded ? INFINITY : hi;
                    }
                    lo = fmin(lo, __shfl_xor(lo, off, WAVE));
                    hi = fmax(hi, __shfl_xor(hi, off, WAVE));
                }
                if (sub == 0) {
                    s_lo[kk] = lo;
                    s_hi[kk] = hi;
                    bx[0] = unbounded ? -INFINITY : lo;
                    bx[D] = unbounded ? INFINITY : hi;
                }
            }
        }
        __syncthreads();
    }
    if constexpr (D <= 16) {
        if (tid < TILE / SUB) {
            double d2 = 0.0;
            for (int k = 0; k < D; ++k) d2 += s_ext[tid][k];
            // 1e-6: the products' kernel values carry their own rounding
            const double r = ceil(neglog2_kernel(d2 * 1.000001, MAT) + 1e-3);
            P.sub_reach[J * (TILE / SUB) + tid] = tid * SUB >= nreal ? -1 : (r < 1e6 ? static_cast<int>(r) : 1000000);
        }
    }
    // the radius about the box centre decides between the two anchors
    double sqc = 0.0;
#pragma unroll
    for (int t = 0; t < D; ++t) {
        const double o = (real && t < d) ? __builtin_fma(xr[t], scale, -0.5 * (s_lo[t] + s_hi[t])) : 0.0;
        sqc = __builtin_fma(o, o, sqc);
    }
    const bool median = block_reduce(sqc, MaxOp(), lds) > WIDE_R2_FP32;
    if (median) {
        // rank of this point's coordinate among the tile's real points (ties by
        // position); the point of rank (nreal - 1) / 2 is the median.  Against the
        // points of the waves before (after) this one a tie counts (does not), one
        // comparison each; only within the wave is the position compared too.
        const int w0 = tid / WAVE * WAVE;
        auto below = [](double u, double v, bool tie) { return u < v || (tie && u == v) ? 1 : 0; };
#pragma unroll 1
        for (int c0 = 0; c0 < d; c0 += CH) {
            for (int k = 0; k < CH && c0 + k < d; ++k)  // the padding ranks last
                s_v[k][tid] = real ? x[static_cast<int64_t>(idx) * d + c0 + k] * scale : INFINITY;
            // kept if a non-finite value breaks the ranks
            if (tid < CH && c0 + tid < d) s_median[c0 + tid] = 0.5 * (s_lo[c0 + tid] + s_hi[c0 + tid]);
            __syncthreads();
            for (int k = 0; k < CH && c0 + k < d; ++k) {
                const double v = s_v[k][tid];
                int rank = 0;
#pragma unroll 16
                for (int i = 0; i < w0; ++i) rank += s_v[k][i] <= v ? 1 : 0;
#pragma unroll 16
                for (int i = 0; i < WAVE; ++i) rank += below(s_v[k][w0 + i], v, i < tid - w0);
#pragma unroll 16
                for (int i = w0 + WAVE; i < TILE; ++i) rank += s_v[k][i] < v ? 1 : 0;
                if (real && rank == (nreal - 1) / 2) s_median[c0 + k] = v;
            }
            __syncthreads();  // s_v is rewritten for the next coordinates
        }
    }
    // offsets from the chosen anchor (padding coordinates and points are zero)
    double sq64 = 0.0, sq32 = 0.0, sq16 = 0.0;
    float of[D];
#pragma unroll
    for (int t = 0; t < D; ++t) {
        const double a = t < d ? (median ? s_median[t] : 0.5 * (s_lo[t] + s_hi[t])) : 0.0;
        const double o = (real && t < d) ? __builtin_fma(xr[t], scale, -a) : 0.0;
        of[t] = static_cast<float>(o);
        if (tid == 0) P.anchor[static_cast<size_t>(J) * D + t] = a;
        if (need & PREP_FP64) P.off64[t * P.n_pad + j] = o;
        if (need & PREP_FP32) P.off32[t * P.n_pad + j] = of[t];
        if constexpr (D > 16) {
            if (need & PREP_PM) {
                P.pm64[j * D + t] = o;
                P.pm32[j * D + t] = of[t];
            }
        }
        sq64 = __builtin_fma(o, o, sq64);
        sq32 = __builtin_fma(static_cast<double>(of[t]), static_cast<double>(of[t]), sq32);
    }
    if (need & PREP_FP32) store_slots<D, false, MAT>(P, j, of);
    // offsets of the BF16 products: rounded to BF16 on a compact tile
    const bool compact = block_reduce(sq64, MaxOp(), lds) <= COMPACT_R2_BF16;
#pragma unroll
    for (int t = 0; t < D; ++t) {
        if (compact) of[t] = bf16_to_f32(f32_to_bf16_rne(of[t]));
        if (need & PREP_BF16) P.offb[t * P.n_pad + j] = of[t];
        if constexpr (D > 16) {
            if (need & PREP_PM) P.pmb[j * D + t] = of[t];
        }
        sq16 = __builtin_fma(static_cast<double>(of[t]), static_cast<double>(of[t]), sq16);
    }
    if (need & PREP_BF16) store_slots<D, true, MAT>(P, j, of);
    const double r2 = block_reduce(fmax(sq64, fmax(sq32, sq16)), MaxOp(), lds);
    const double nj = floor(0.5 * r2);
    if (tid == 0) {
        P.tile_r2[J] = r2;
        P.tile_nj[J] = nj;
        // Gaussian: a target at |t| from the anchor has exponent
        // <= -(|t| - R)^2 + R^2 - N_J against every source of the tile, <= -200
        // beyond this |t|^2; Matern: scaled distance >= 111 (exp2 of -log2(e) s
        // is 0 in FP32) beyond (R + 111)^2; 1e-4 margin
        const double u = MAT ? sqrt(r2) + 111.0 : sqrt(r2) + sqrt(200.0 + r2 - nj);
        P.tile_far[J] = static_cast<float>(1.0001 * u * u);
        // FP64: exponents <= -1100, or for Matern e^-s at s >= 760 (0 in FP64)
        const double u64 = MAT ? sqrt(r2) + 760.0 : sqrt(r2) + sqrt(1100.0 + r2 - nj);
        P.tile_far64[J] = static_cast<float>(1.0001 * u64 * u64);
    }
    double w64 = 0.0;
    float w32 = 0.f, w16 = 0.f;
    if (need & PREP_FP64) {
        P.sq64[j] = sq64;
        P.w64[j] = w64 = (real && r2 <= WIDE_R2_FP64) ? exp2(nj - sq64) : 0.0;
    }
    if (need & PREP_FP32) P.w32[j] = w32 = (real && r2 <= WIDE_R2_FP32) ? static_cast<float>(exp2(nj - sq32)) : 0.0f;
    if (need & PREP_BF16) P.w16[j] = w16 = (real && r2 <= WIDE_R2_FP32) ? static_cast<float>(exp2(nj - sq16)) : 0.0f;
    // the product's vector: sorted copy, prescaled copy and the tile's bounds
    // (what a gather, a rounding and a prescale launch did, about 4.7 us each)
    if (pv.q != nullptr) {
        double aq;
        if (pv.prec == KRR_FP64) {
            const double q = real ? static_cast<const double *>(pv.q)[idx] : 0.0;
            static_cast<double *>(pv.qs)[j] = q;
            static_cast<double *>(pv.qw)[j] = q * w64;
            aq = fabs(q);
        } else {
            float q = real ? static_cast<const float *>(pv.q)[idx] : 0.f;
            if (pv.prec == KRR_BF16) {
                const uint16_t h = f32_to_bf16_rne(q);
                static_cast<uint16_t *>(pv.qs)[j] = h;
                q = bf16_to_f32(h);
                static_cast<float *>(pv.qw)[j] = q * w16;
            } else {
                static_cast<float *>(pv.qs)[j] = q;
                static_cast<float *>(pv.qw)[j] = q * w32;
            }
            aq = fabs(static_cast<double>(q));
        }
        if constexpr (D <= 16) {
            __threadfence_block();
            __syncthreads();  // sub_reach was written above by this block
            tile_bounds(tid, true, aq, P.sub_reach + J * (TILE / SUB), real, pv.up + J, pv.lo + J, &s_v[0][0]);
        }
    }
}

template <int D>
static hipError_t launch_tiles(const Prepared &P, const double *x, const int32_t *order, int need, const PrepVec &v,
                               hipStream_t s) {
    if (P.kernel == KRR_KERNEL_MATERN32)
        hipLaunchKernelGGL((k_tiles<D, true>), dim3(P.ntiles), dim3(TILE), 0, s, x, P.n, P.d, P.scale, order, P, need,
                           v);
    else
        hipLaunchKernelGGL((k_tiles<D, false>), dim3(P.ntiles), dim3(TILE), 0, s, x, P.n, P.d, P.scale, order, P,
                           need, v);
    return hipGetLastError();
}

static hipError_t build_tiles(const Prepared &P, const double *x, const int32_t *order, int need, const PrepVec &v,
                              hipStream_t s) {
    switch (P.dpad) {
        case 1: return launch_tiles<1>(P, x, order, need, v, s);
        case 2: return launch_tiles<2>(P, x, order, need, v, s);
        case 3: return launch_tiles<3>(P, x, order, need, v, s);
        case 4: return launch_tiles<4>(P, x, order, need, v, s);
        case 6: return launch_tiles<6>(P, x, order, need, v, s);
        case 8: return launch_tiles<8>(P, x, order, need, v, s);
        case 12: return launch_tiles<12>(P, x, order, need, v, s);
        case 16: return launch_tiles<16>(P, x, order, need, v, s);
        case 24: return launch_tiles<24>(P, x, order, need, v, s);
        case 32: return launch_tiles<32>(P, x, order, need, v, s);
        case 48: return launch_tiles<48>(P, x, order, need, v, s);
        case 64: return launch_tiles<64>(P, x, order, need, v, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t prepare_points(Prepared &P, const double *x, double sigma, void *temp, size_t temp_bytes,
                          hipStream_t s, int kernel, int need, const PrepVec *v) {
    const int64_t n = P.n;
    const int d = P.d;
    P.kernel = kernel;
    // Gaussian: exp(-r^2 / (2 sigma^2)) = 2^(-||x~_i - x~_j||^2); Matern: the
    // scaled distance ||x~_i - x~_j|| is sqrt(3) r / h
    P.scale = kernel == KRR_KERNEL_MATERN32 ? std::sqrt(3.0) / sigma
                                            : std::sqrt(std::log2(std::exp(1.0))) / (sigma * std::sqrt(2.0));
    // the point-major copies feed the VALU cross-check kernels only
    if (P.dpad > 16 && use_valu_kernel()) need |= PREP_PM;
    Carver cv(temp);
    uint64_t *k0 = cv.take<uint64_t>(n);
    uint64_t *k1 = cv.take<uint64_t>(n);
    int32_t *v0 = cv.take<int32_t>(n);
    int32_t *v1 = cv.take<int32_t>(n);
    double *part = cv.take<double>(2 * KRR_MAX_DIM * BBOX_BLOCKS);
    int *bad = cv.take<int>(KRR_MAX_DIM * BBOX_BLOCKS);
    const size_t sort_cap = sort_scratch_bound(n);
    char *sort_tmp = cv.take<char>(sort_cap);
    if (cv.off > temp_bytes) return hipErrorInvalidValue;

    const int nblk = static_cast<int>(std::min<int64_t>(BBOX_BLOCKS, (n + BBOX_THREADS - 1) / BBOX_THREADS));
    hipLaunchKernelGGL(k_bbox_partial, dim3(nblk, d), dim3(BBOX_THREADS), 0, s, x, n, d, P.scale, part, bad);
    const int dm = d < 63 ? d : 63;
    const int bits = (63 / dm) < 31 ? 63 / dm : 31;
    hipLaunchKernelGGL(k_morton, dim3((n + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, x, n, d, P.scale, part, bad, nblk,
                       dm, bits, k0, v0, P.flags);
    KRR_HIP(hipGetLastError());
    // counting ranks grows with n^2; measured against the radix sort it is ahead
    // up to RANK_MAX_N
    if (n <= RANK_MAX_N) {
        hipLaunchKernelGGL(k_rank, dim3(static_cast<unsigned>((n + WAVE - 1) / WAVE)), dim3(RANK_THREADS), 0, s, k0,
                           static_cast<int>(n), v1);
        KRR_HIP(hipGetLastError());
        return build_tiles(P, x, v1, need, v ? *v : PrepVec{}, s);
    }
    rocprim::double_buffer<uint64_t> keys(k0, k1);
    rocprim::double_buffer<int32_t> vals(v0, v1);
    size_t bytes = 0;
    KRR_HIP(rocprim::radix_sort_pairs(nullptr, bytes, keys, vals, static_cast<size_t>(n), 0u,
                                      static_cast<unsigned>(dm * bits), s));
    if (bytes > sort_cap) return hipErrorInvalidValue;
    KRR_HIP(rocprim::radix_sort_pairs(sort_tmp, bytes, keys, vals, static_cast<size_t>(n), 0u,
                                      static_cast<unsigned>(dm * bits), s));
    return build_tiles(P, x, static_cast<const int32_t *>(vals.current()), need, v ? *v : PrepVec{}, s);
}

// ---------------------------------------------------------------- gather / scatter

template <typename T>
__device__ inline T cvt(double v);
template <>
__device__ inline double cvt<double>(double v) { return v; }
template <>
__device__ inline float cvt<float>(double v) { return static_cast<float>(v); }

template <typename Tin, typename Tout>
__global__ __launch_bounds__(BLOCK) void k_gather(const int32_t *__restrict__ perm, int64_t n_pad,
                                                  const Tin *__restrict__ src, Tout *__restrict__ dst) {
    const int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x;
    if (i >= n_pad) return;
    const int32_t p = perm[i];
    dst[i] = p >= 0 ? static_cast<Tout>(src[p]) : Tout(0);
}

template <typename Tin, typename Tout>
__global__ __launch_bounds__(BLOCK) void k_scatter(const int32_t *__restrict__ perm, int64_t n_pad,
                                                   const Tin *__restrict__ src, Tout *__restrict__ dst) {
    const int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x;
    if (i >= n_pad) return;
    const int32_t p = perm[i];
    if (p >= 0) dst[p] = static_cast<Tout>(src[i]);
}

template <typename Tin, typename Tout>
hipError_t gather_sorted(const Prepared &P, const Tin *src, Tout *dst, hipStream_t s) {
    hipLaunchKernelGGL((k_gather<Tin, Tout>), dim3((P.n_pad + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, P.perm,
                       P.n_pad, src, dst);
    return hipGetLastError();
}
template <typename Tin, typename Tout>
hipError_t scatter_sorted(const Prepared &P, const Tin *src, Tout *dst, hipStream_t s) {
    hipLaunchKernelGGL((k_scatter<Tin, Tout>), dim3((P.n_pad + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, P.perm,
                       P.n_pad, src, dst);
    return hipGetLastError();
}

template hipError_t gather_sorted<double, double>(const Prepared &, const double *, double *, hipStream_t);
template hipError_t gather_sorted<float, float>(const Prepared &, const float *, float *, hipStream_t);
template hipError_t gather_sorted<double, float>(const Prepared &, const double *, float *, hipStream_t);
template hipError_t scatter_sorted<double, double>(const Prepared &, const double *, double *, hipStream_t);
template hipError_t scatter_sorted<float, float>(const Prepared &, const float *, float *, hipStream_t);
template hipError_t scatter_sorted<float, double>(const Prepared &, const float *, double *, hipStream_t);
template hipError_t gather_sorted<float, double>(const Prepared &, const float *, double *, hipStream_t);
template hipError_t scatter_sorted<double, float>(const Prepared &, const double *, float *, hipStream_t);

__global__ __launch_bounds__(BLOCK) void k_to_bf16(const float *__restrict__ src, uint16_t *__restrict__ dst,
                                                   int64_t n) {
    const int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x;
    if (i < n) dst[i] = f32_to_bf16_rne(src[i]);
}

hipError_t to_bf16(const float *src, uint16_t *dst, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_to_bf16, dim3((n + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, src, dst, n);
    return hipGetLastError();
}

}  // namespace krr
