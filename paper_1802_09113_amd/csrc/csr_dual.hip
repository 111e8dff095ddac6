// Newton directions on CSR samples in the sample's row space.
//
// Alg. 2 started from r_0 = -g never leaves span{g} + X_S^T R^(nS x K): with z = X_S s the product is
// H_S s = scale X_S^T U(z) + lambda s, U(z) the rows of eq. (12).  So every vector of the method is kept as
//   v = a g + X_S^T Y,  a scalar a and an nS x K block Y of coefficients,
// and what the method asks of a vector needs no column of the matrix:
//   X_S v = a (X_S g) + A Y,  A = X_S X_S^T (nS x nS, once per sample),   <v, v> = a (a g.g + Y . X_S g) + Y . X_S v.
// A text sample of 1000 rows of 450 entries touches 127 000 columns; with 19 weight columns a vector of Alg. 2 on those is
// 2.4 million numbers, and 19 000 here.  A CG iteration is two launches: the new direction's X_S s = X_S r + beta X_S s,
// U(X_S s) and A U on the matrix cores (dual_product_kernel), then the step and all updates (dual_update_kernel, the
// counterpart of finalize_cg_kernel: every dot product is left as partials by the launch before).  The curvature is that of s
// itself, sum of X_S s . U(X_S s) + lambda s . s: formed from the residual's, r . H r + 2 beta r . H s + beta^2 s . H s, as the
// dense paths do, it cancels where lambda is small, and the directions were 3 (lambda 1e-3) to 16 times (1e-4) as far from
// extended precision as those of CG on the columns.  The direction is p g + X_S^T Y_p at the end: one gather.  Everything
// here is in fp64 whatever the data's precision.
//
// 20000 x 1355191, 450 entries a row, K 19, fp64, 1000 sampled rows: an iteration 85 -> 14 us (product 8.0, update 5.0), the
// Gram matrix 75, a direction of ten products with its preparation 1222 -> 600; two Newton steps 4291 -> 3020 us.
// Precision: what the scalars lose is the part of g that the sampled rows span, as r . r forms from terms of the size of
// rho^2 g.g; but rho falls with r (it is the residual on every coordinate outside the rows' span).  On 25 text samples of five
// shapes the directions are as far from extended precision as those of CG on the columns: 1e-16 to 1e-7 by shape, the ratio of
// the two between 0.07 and 10, 0.80 in the geometric mean; on well conditioned samples of 100 to 400 short rows 0.84 (lambda
// 1e-2), 2.0 (1e-3) and 4.4 (1e-4: 1.2e-15 against 2.8e-16).
#include "ssn_internal.h"
#include "ssn_math.h"
#include "csr_margin.h"

namespace ssn {

typedef double dv4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ dv4 dmfma(double a, double b, dv4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// the value of v in lane src (the same for the whole wave)
__device__ __forceinline__ double lane_value(double v, int src)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), src), hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ __forceinline__ double lane_value(float v, int src)
{
    return (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}

int64_t gram_ld(int64_t rows) { return (rows + 63) / 64 * 64; }

// ---- the Gram matrix -------------------------------------------------------------------------------------
// Frequent columns (gram_freq_min entries and more: the few hundred words that most of the pairs of rows share) go through
// a dense copy and the matrix cores; the pairs of rows that share one of the others are added row by row in LDS.  The line
// is an eighth of the rows (64 and more): there a dense column's n^2 / 2 products, eight per cycle and SIMD, and a sparse column's n^2 / 64,
// a wave of them in some hundred cycles, cost about the same.  1000 rows of text, 127 000 columns: from 125 entries on 404
// columns with 92 % of the 80 million products.

static int gram_freq_min(int64_t rows) { return rows > 512 ? (int)(rows / 8) : 64; }

// xf[h][i] = the entry of frequent column h in sampled row i (one at most: the caller serves no matrix whose rows store a
// column twice); rows of zeros behind them up to a multiple of sixteen
template <typename T>
__global__ __launch_bounds__(256) void gram_dense_kernel(const int32_t *freq, const int32_t *nfreq_dev, const int32_t *cstart, const int32_t *row,
                                                         const T *val, double *xf, int ld)
{
    extern __shared__ double gram_lds[];
    const int h = blockIdx.x, nfreq = *nfreq_dev;
    if (h >= (nfreq + 15) / 16 * 16) return;
    for (int i = threadIdx.x; i < ld; i += 256) gram_lds[i] = 0.0;
    __syncthreads();
    if (h < nfreq) {
        const int c = freq[h], t1 = cstart[c + 1];
        for (int t = cstart[c] + threadIdx.x; t < t1; t += 256) gram_lds[row[t]] = (double)val[t];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < ld; i += 256) xf[(int64_t)h * ld + i] = gram_lds[i];
}

// gram = xf^T xf by tiles of 32 x 32, a workgroup of four waves per tile on and above the diagonal; the waves share the
// frequent columns, sixteen at a time, and their sums are added in wave order.  (Tiles of 64 x 64, a
// quarter per wave and the columns in shares, were slower: 48 against 34 us for 811 columns of 1000 rows.)
__global__ __launch_bounds__(256) void gram_frequent_kernel(const double *xf, const int32_t *nfreq_dev, int ld, double *gram)
{
    __shared__ double lds[4 * 4 * 256];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, f = lane & 15;
    const int nt = ld / 32, groups = (*nfreq_dev + 15) / 16;
    int I = 0, J = blockIdx.x;
    while (J >= nt - I) {
        J -= nt - I;
        ++I;
    }
    J += I;
    dv4 acc[2][2] = {{dv4{0, 0, 0, 0}, dv4{0, 0, 0, 0}}, {dv4{0, 0, 0, 0}, dv4{0, 0, 0, 0}}};
    double a[4][2], b[4][2];
    auto fetch = [&](int g) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double *x = xf + (int64_t)(16 * g + 4 * s + q) * ld + f;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                a[s][m] = x[I * 32 + 16 * m];
                b[s][m] = x[J * 32 + 16 * m];
            }
        }
    };
    if (w < groups) fetch(w);
    for (int g = w; g < groups; g += 4) {
        double ca[4][2], cb[4][2];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int m = 0; m < 2; ++m) ca[s][m] = a[s][m], cb[s][m] = b[s][m];
        if (g + 4 < groups) fetch(g + 4);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = dmfma(ca[s][i], cb[s][j], acc[i][j]);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) lds[(w * 4 + t) * 256 + v * 64 + lane] = acc[t >> 1][t & 1][v];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const double x = (lds[t * 256 + tid] + lds[(4 + t) * 256 + tid]) + (lds[(8 + t) * 256 + tid] + lds[(12 + t) * 256 + tid]);
        const int r = I * 32 + 16 * (t >> 1) + 4 * w + q, c = J * 32 + 16 * (t & 1) + f;       // w: accumulator element here
        gram[(int64_t)r * ld + c] = x;
        if (I != J) gram[(int64_t)c * ld + r] = x;
    }
}

// gram[i] += the products of row i with the rows it shares its other columns with; a workgroup per row, each wave adds
// every fourth of the row's entries into a copy of its own (one order of additions), a column's entries one to a lane, eight
// columns in flight (quarters of consecutive entries, whose waves differ a lot in work, and a column at a time: 82 -> 28 us
// for 1000 rows of 450)
template <typename T>
__global__ __launch_bounds__(256) void gram_rare_kernel(const int32_t *off, const int32_t *ccol, const T *val_in, const int32_t *cstart,
                                                        const int32_t *row, const T *val, int n, int ld, int fmin, double *gram)
{
    extern __shared__ double gram_lds[];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = blockIdx.x;
    double *acc = gram_lds + w * n;
    double *gi = gram + (int64_t)i * ld;
    for (int j = lane; j < n; j += 64) acc[j] = 0.0;
    const int b = off[i], e = off[i + 1];
    double single = 0.0;
    for (int t0 = b; t0 < e; t0 += 256) {
        const int t = t0 + 4 * lane + w;
        int s = 0, len = 0;
        T v = T(0);
        if (t < e) {
            const int c = ccol[t];
            v = val_in[t];
            s = cstart[c];
            len = cstart[c + 1] - s;
        }
        if (len == 1) single += (double)v * (double)v;               // no other row has this column
        unsigned long long m = __ballot(len >= 2 && len <= 64 && len < fmin), ml = __ballot(len > 64 && len < fmin);
        while (m) {
            constexpr int U = 8;
            int j[U], lk[U];
            T x[U];
            double vk[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int src = m ? __ffsll((long long)m) - 1 : 0;
                const int sk = __builtin_amdgcn_readlane(s, src);
                lk[k] = m ? __builtin_amdgcn_readlane(len, src) : 0;
                vk[k] = lane_value(v, src);
                m &= m - 1;
                const int at = sk + (lane < lk[k] ? lane : 0);
                j[k] = row[at];
                x[k] = val[at];
            }
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (lane < lk[k])
                    (void)__hip_atomic_fetch_add(&acc[j[k]], vk[k] * (double)x[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        for (; ml; ml &= ml - 1) {
            const int src = __ffsll((long long)ml) - 1;
            const int sk = __builtin_amdgcn_readlane(s, src), lk = __builtin_amdgcn_readlane(len, src);
            const double vk = lane_value(v, src);
            for (int r = 0; r < lk; r += 256) {
                int j[4];
                T x[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int o = r + 64 * k + lane, at = sk + (o < lk ? o : 0);
                    j[k] = row[at];
                    x[k] = val[at];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (r + 64 * k + lane < lk)
                        (void)__hip_atomic_fetch_add(&acc[j[k]], vk * (double)x[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    single = wave_inclusive_scan(single);
    if (lane == 63) (void)__hip_atomic_fetch_add(&acc[i], single, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += 256)
        gi[j] += (gram_lds[j] + gram_lds[n + j]) + (gram_lds[2 * n + j] + gram_lds[3 * n + j]);
}

static hipError_t dual_grow(double **ptr, int64_t *cap, int64_t need)
{
    if (*cap >= need) return hipSuccess;
    if (*ptr) {
        const hipError_t e = hipFree(*ptr);
        if (e != hipSuccess) return e;
    }
    *ptr = nullptr;
    *cap = 0;
    const hipError_t e = hipMalloc((void **)ptr, (size_t)(need + need / 8) * sizeof(double));
    if (e != hipSuccess) return e;
    *cap = need + need / 8;
    return hipSuccess;
}

template <typename T> static hipError_t gram_go(CscView *v, int ld, int fpad, hipStream_t st)
{
    static const hipError_t attr =
        hipFuncSetAttribute((const void *)gram_rare_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * GRAM_ROWS_MAX * 8);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(gram_dense_kernel<T>, dim3((unsigned)fpad), dim3(256), (size_t)ld * 8, st, v->freq, v->nfreq_dev, v->cstart, v->row,
                       (const T *)v->val, v->xfreq, ld);
    const int nt = ld / 32;
    hipLaunchKernelGGL(gram_frequent_kernel, dim3((unsigned)(nt * (nt + 1) / 2)), dim3(256), 0, st, v->xfreq, v->nfreq_dev, ld, v->gram);
    const int n = (int)v->nrows;
    hipLaunchKernelGGL(gram_rare_kernel<T>, dim3((unsigned)n), dim3(256), (size_t)n * 4 * 8, st, v->off, v->ccol, (const T *)v->val_in,
                       v->cstart, v->row, (const T *)v->val, n, ld, gram_freq_min(v->nrows), v->gram);
    return hipGetLastError();
}

hipError_t csc_gram(CscView *v, int dtype, hipStream_t st)
{
    // how many columns are frequent stays on the device: the buffers take what the entries allow, and the columns
    const int ld = (int)gram_ld(v->nrows);
    const int64_t by_nnz = v->nnz / gram_freq_min(v->nrows), most = by_nnz < v->ncols ? by_nnz : v->ncols;
    const int fpad = most > 0 ? (int)((most + 15) / 16 * 16) : 16;
    hipError_t e = csc_frequent_columns(v, gram_freq_min(v->nrows), st);
    if (e == hipSuccess) e = dual_grow(&v->gram, &v->cap_gram, (int64_t)ld * ld);
    if (e == hipSuccess) e = dual_grow(&v->xfreq, &v->cap_xfreq, (int64_t)fpad * ld);
    if (e != hipSuccess) return e;
    e = dtype == SSN_F32 ? gram_go<float>(v, ld, fpad, st) : gram_go<double>(v, ld, fpad, st);
    if (e == hipSuccess) v->gram_rows = v->nrows;
    return e;
}

// ---- Alg. 2 ------------------------------------------------------------------------------------------------
// X_S g, and the start: r_0 = -g; a workgroup per row, its waves share the row's entries (a sample's rows are few)
constexpr int START_WAVES = 8;
template <typename T, int VEC> __global__ __launch_bounds__(64 * START_WAVES) void dual_start_kernel(DualCg a)
{
    __shared__ double zs[START_WAVES * 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, K = a.K, NS = 64 / ((K + VEC - 1) / VEC);
    const int64_t r = a.S[blockIdx.x], b = a.rowptr[r], e = a.rowptr[r + 1];
    const int64_t per = ((e - b + START_WAVES * NS - 1) / (START_WAVES * NS)) * NS;
    const int64_t wb = b + w * per < e ? b + w * per : e, we = wb + per < e ? wb + per : e;
    zs[w * 64 + lane] = csr_row_margin_vec<T, double, VEC>(a.colidx, (const T *)a.vals, (const T *)a.G, a.ldg, wb, we, lane, K);
    __syncthreads();
    if ((int)threadIdx.x >= K) return;
    double z = 0.0;
#pragma unroll
    for (int k = 0; k < START_WAVES; ++k) z += zs[k * 64 + lane];
    const int64_t o = (int64_t)blockIdx.x * K + lane;
    a.zg[o] = z;
    a.w[o] = -z;
    a.yr[o] = a.yp[o] = a.ybest[o] = 0.0;
}

// sums of N values over the block, the same bits in every thread
template <int N> __device__ __forceinline__ void dual_sums(double (&v)[N])
{
    __shared__ double sm[N][4];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        v[i] = wave_inclusive_scan(v[i]);
        if ((threadIdx.x & 63) == 63) sm[i][threadIdx.x >> 6] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = (sm[i][0] + sm[i][1]) + (sm[i][2] + sm[i][3]);
    __syncthreads();
}

// r_k . r_k from the state behind product k - 1 and the sums of Y_r . X_S g and Y_r . X_S r_k.  What cancels is the part
// of g that the sampled rows span; a sum below zero is rounding around a residual of nothing.
__device__ __forceinline__ double dual_rr(double rho, double gg, double yz, double yw)
{
    const double rr = rho * (rho * gg + yz) + yw;
    return rr < 0.0 ? 0.0 : rr;
}

// the state before product k: lines 10-11 of Alg. 2 for the residual product k - 1 left
struct DualState {
    double rr, rbest, gnorm, pibest;
    int done, iters, flags, better;
};
__device__ __forceinline__ DualState dual_advance(const CgSlot &prev, double rr_new, double theta)
{
    const bool ended = prev.done || prev.brk, broke = prev.brk && !prev.done;
    const double rnorm = sqrt(rr_new);
    const bool better = !ended && rnorm <= prev.rbest, stop = !ended && rnorm <= theta * prev.gnorm;
    DualState s;
    s.rr = ended ? prev.rr : rr_new;
    s.rbest = better ? rnorm : prev.rbest;
    s.gnorm = prev.gnorm;
    s.pibest = better ? prev.pi : prev.pibest;
    s.done = (ended || stop) ? 1 : 0;
    s.iters = (ended && !broke) ? prev.iters : prev.iters + 1;
    s.flags = prev.flags | (stop ? 1 : 0) | (broke ? 2 : 0);
    s.better = better ? 1 : 0;
    return s;
}

// What both launches of product k form alike from the state before product k - 1 (product 0: that of the initialisation,
// whose residual is -g) and the partials of Y_r . X_S g and Y_r . X_S r_k behind it.
struct DualBefore {
    DualState s;
    double rho, sigma, gg, beta;
};
__device__ __forceinline__ DualBefore dual_before(const CgSlot &prev, bool first, double yz, double yw, double theta)
{
    DualBefore b;
    b.gg = first ? prev.rr : prev.goff;
    b.rho = first ? -1.0 : prev.rho;
    b.sigma = first ? 0.0 : prev.sigma;
    b.s = dual_advance(prev, dual_rr(b.rho, b.gg, yz, yw), theta);
    if (first) {
        b.s.rr = prev.rr;
        b.s.rbest = prev.rbest;
        b.s.pibest = prev.pibest;
        b.s.done = prev.done;
        b.s.iters = 0;
        b.s.flags = prev.flags;
        b.s.better = 0;
    }
    b.beta = (first || b.s.done) ? 0.0 : b.s.rr / prev.rr;
    return b;
}

// X_S s of the new direction (line 12) and its U for the rows [ks * kper, + kper) of the sample, 64 at a time, and their share
// of gram * U for 64 rows: a workgroup of four waves, one 16-row tile each; part[ks] receives the share.  Both operands of the
// matrix instruction come in whole lines: gram is symmetric, so its rows serve as columns, and U goes through LDS.  The
// workgroups of the first row tile also store X_S s (beside the one before, which the others still read) and U and leave
// their sum of X_S s . U.
template <typename T, int NB>
__global__ __launch_bounds__(256) void dual_product_kernel(DualCg a, const CgSlot *prev_p, int k, const double *din, int nb)
{
    const bool first = k == 0;
    const CgSlot prev = *prev_p;
    if (prev.done || (!first && prev.brk)) return;
    constexpr int UL = NB * 16 + 1;
    __shared__ double us[64 * UL];
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, f = lane & 15;
    const int K = a.K, n = a.n, it = blockIdx.x, ks = blockIdx.y;
    const T *P = (const T *)a.P;
    const double *xs_old = k & 1 ? a.xs[0] : a.xs[1];
    double *xs_new = k & 1 ? a.xs[1] : a.xs[0];
    const int k0 = ks * a.kper, k1 = k0 + a.kper < a.ld ? k0 + a.kper : a.ld;
    double g[16];
    auto fetch = [&](int kb) {
#pragma unroll
        for (int s = 0; s < 16; ++s) g[s] = a.gram[(int64_t)(kb + 4 * s + q) * a.ld + it * 64 + w * 16 + f];
    };
    fetch(k0);                               // on the way while the scalars are formed
    double v[2] = {0.0, 0.0};
    if (!first)
        for (int i = tid; i < nb; i += 256) {
            v[0] += din[i];
            v[1] += din[nb + i];
        }
    dual_sums<2>(v);
    const DualBefore b = dual_before(prev, first, v[0], v[1], a.theta);
    if (b.s.done) return;                    // the same in every workgroup
    dv4 acc[NB];
#pragma unroll
    for (int nb_ = 0; nb_ < NB; ++nb_) acc[nb_] = dv4{0, 0, 0, 0};
    double zu = 0.0;
    for (int kb = k0; kb < k1; kb += 64) {
        if (kb > k0) fetch(kb);
        const int r = kb + (tid >> 2), sub = tid & 3;
        double pv[NB * 4], xv[NB * 4], t = 0.0;
#pragma unroll
        for (int m = 0; m < NB * 4; ++m) {
            const int c = sub + 4 * m;
            const bool in = r < n && c < K;
            pv[m] = in ? (double)P[(int64_t)r * a.KP + c] : 0.0;
            xv[m] = in ? a.w[(int64_t)r * K + c] : 0.0;
            if (!first && in) xv[m] += b.beta * xs_old[(int64_t)r * K + c];
        }
#pragma unroll
        for (int m = 0; m < NB * 4; ++m) t += pv[m] * xv[m];
        t += __shfl_xor(t, 1);
        t += __shfl_xor(t, 2);
        if (kb > k0) __syncthreads();                                // the rows before these have been used
#pragma unroll
        for (int m = 0; m < NB * 4; ++m) {
            const int c = sub + 4 * m;
            const double u = pv[m] * xv[m] - pv[m] * t;              // eq. (12); zero in padded rows and classes
            us[(tid >> 2) * UL + c] = u;
            if (it == 0 && r < n && c < K) {
                xs_new[(int64_t)r * K + c] = xv[m];
                a.u[(int64_t)r * K + c] = u;
                zu += xv[m] * u;
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 16; ++s)
#pragma unroll
            for (int i = 0; i < NB; ++i) acc[i] = dmfma(g[s], us[(4 * s + q) * UL + i * 16 + f], acc[i]);
    }
    double *out = a.part + (int64_t)ks * n * K;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = it * 64 + w * 16 + 4 * e + q, c = i * 16 + f;
            if (r < n && c < K) out[(int64_t)r * K + c] = acc[i][e];
        }
    if (it != 0) return;                                             // the whole workgroup
    zu = wave_inclusive_scan(zu);
    if (lane == 63) red[w] = zu;
    __syncthreads();
    if (tid == 0) a.zu_part[ks] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Behind product k: the scalars and lines 7-12 of Alg. 2 (see finalize_cg_kernel).  A state slot holds rho of r_{k+1}, sigma
// of s_k, pi of p_{k+1} (r = rho g + X_S^T Y_r and so on), g.g in goff and s_k . s_k in sHs; product 0 starts from slot *prev
// of the initialisation.
__global__ __launch_bounds__(256) void dual_update_kernel(DualCg a, const CgSlot *prev_p, CgSlot *cur, int k, const double *din,
                                                          double *dout)
{
    const bool first = k == 0;
    const CgSlot prev = *prev_p;
    const int64_t total = (int64_t)a.n * a.K, e = (int64_t)blockIdx.x * 256 + threadIdx.x, eo = e < total ? e : 0;
    const int nb = gridDim.x;
    const double *xs = k & 1 ? a.xs[1] : a.xs[0];
    double w = a.w[eo], yr = a.yr[eo], yp = a.yp[eo], ys = first ? 0.0 : a.ys[eo], gu = 0.0;
    const double u = a.u[eo], x = xs[eo], zg = a.zg[eo];
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < a.nks; i += 256) v[0] += a.zu_part[i];
    if (!first)
        for (int i = threadIdx.x; i < nb; i += 256) {
#pragma unroll
            for (int j = 0; j < 3; ++j) v[1 + j] += din[j * nb + i];
        }
    for (int c = 0; c < a.nks; c += 8) {
        double t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = a.part[(int64_t)(c + i < a.nks ? c + i : c) * total + eo];
#pragma unroll
        for (int i = 0; i < 8; ++i) gu += (c + i < a.nks) ? t[i] : 0.0;
    }
    dual_sums<4>(v);
    const DualBefore b = dual_before(prev, first, v[1], v[2], a.theta);
    const DualState &s = b.s;
    const double beta = b.beta;
    // s_k . s_k from r_k . s_{k-1} = sigma (rho g.g + Y_r . X_S g) + Y_s . X_S r_k, which is rounding and no more
    const double ss = first ? s.rr : s.rr + 2.0 * beta * (b.sigma * (b.rho * b.gg + v[1]) + v[3]) + beta * beta * prev.sHs;
    const double sHs = a.scale * v[0] + a.lambda * ss;
    const bool brk = !s.done && !(sHs > 0.0), update = !s.done && !brk;
    const double alpha = update ? s.rr / sHs : 0.0;
    const double sig_n = update ? b.rho + beta * b.sigma : b.sigma, pi = first ? 0.0 : prev.pi;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        cur->rr = s.rr;
        cur->rbest = s.rbest;
        cur->gnorm = s.gnorm;
        cur->done = s.done;
        cur->iters = s.iters;
        cur->flags = s.flags;
        cur->brk = brk ? 1 : 0;
        cur->alpha = alpha;
        cur->best_cur = 0;
        cur->best_pending = 0;
        cur->sHs = ss;
        cur->goff = b.gg;
        cur->rho = b.rho - alpha * a.lambda * sig_n;
        cur->sigma = sig_n;
        cur->pi = pi + alpha * sig_n;
        cur->pibest = s.pibest;
        if (a.trace) {
            if (!first && !prev.done && !prev.brk) a.trace[3 * (k - 1) + 1] = sqrt(s.rr);
            if (!s.done) {
                a.trace[3 * k] = alpha;
                a.trace[3 * k + 2] = sHs;
                if (brk) a.trace[3 * k + 1] = sqrt(s.rr);
            }
        }
    }
    if (s.better && e < total) a.ybest[e] = yp;                      // line 10 for the iterate the last product left
    if (!update) return;
    double d[3] = {0.0, 0.0, 0.0};
    if (e < total) {
        ys = yr + beta * ys;                                         // line 12
        yp += alpha * ys;                                            // line 8
        yr -= alpha * (a.scale * u + a.lambda * ys);                 // line 9
        w -= alpha * (a.scale * gu + a.lambda * x);
        a.ys[e] = ys;
        a.yp[e] = yp;
        a.yr[e] = yr;
        a.w[e] = w;
        d[0] = yr * zg;
        d[1] = yr * w;
        d[2] = ys * w;
    }
    dual_sums<3>(d);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int j = 0; j < 3; ++j) dout[j * nb + blockIdx.x] = d[j];
    }
}

// After the last product: lines 10-11 for r_T, the coefficients of the best iterate (in the data's precision: the
// operand of the gather), the partials of their product with X_S g for the slope, the final state
template <typename T>
__global__ __launch_bounds__(256) void dual_tail_kernel(DualCg a, const CgSlot *prev_p, CgSlot *fin, int k, const double *din, T *yout,
                                                        int KP, double *slope_part)
{
    const CgSlot prev = *prev_p;
    const int64_t total = (int64_t)a.n * a.K, e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int nb = gridDim.x;
    double v[2] = {0.0, 0.0};
    for (int i = threadIdx.x; i < nb; i += 256) {
        v[0] += din[i];
        v[1] += din[nb + i];
    }
    dual_sums<2>(v);
    const DualState s = dual_advance(prev, dual_rr(prev.rho, prev.goff, v[0], v[1]), a.theta);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        fin->rr = s.rr;
        fin->rbest = s.rbest;
        fin->gnorm = s.gnorm;
        fin->done = s.done;
        fin->iters = s.iters;
        fin->flags = s.flags;
        fin->brk = 0;
        fin->alpha = 0.0;
        fin->best_cur = 0;
        fin->best_pending = 0;
        fin->sHs = prev.sHs;
        fin->goff = prev.goff;               // all of g.g: the slope is pibest * goff + the partials below
        fin->rho = prev.rho;
        fin->sigma = prev.sigma;
        fin->pi = prev.pi;
        fin->pibest = s.pibest;
        if (a.trace && !prev.done && !prev.brk) a.trace[3 * (k - 1) + 1] = sqrt(s.rr);
    }
    double d[1] = {0.0};
    if (e < total) {
        const double y = s.better ? a.yp[e] : a.ybest[e];
        const int64_t i = e / a.K;
        yout[i * KP + (e - i * a.K)] = (T)y;
        d[0] = y * a.zg[e];
    }
    dual_sums<1>(d);
    if (slope_part && threadIdx.x == 0) slope_part[blockIdx.x] = d[0];
}

int64_t dual_doubles(int64_t n, int K, int *nks, int *kper)
{
    const int64_t ld = gram_ld(n);
    *kper = n <= 1024 ? 64 : 128;
    *nks = (int)((ld + *kper - 1) / *kper);
    return (9 + *nks) * n * K + 64 + 2 * 4 * RED_MAX_PARTS;
}

template <typename T> static hipError_t dual_go(DualCg a, CgSlot *slots, int T_, T *yout, int KP, double *parts, double *slope_part, hipStream_t st)
{
    const int nb = dual_blocks(a.n, a.K);
    const dim3 grid((unsigned)(a.ld / 64), (unsigned)a.nks), block(256);
    const int vec = row_vec<T>(a.K);
    const dim3 rows((unsigned)a.n), waves(64 * START_WAVES);
    if (vec == 1) hipLaunchKernelGGL((dual_start_kernel<T, 1>), rows, waves, 0, st, a);
    else if (vec == 2) hipLaunchKernelGGL((dual_start_kernel<T, 2>), rows, waves, 0, st, a);
    else hipLaunchKernelGGL((dual_start_kernel<T, 16 / (int)sizeof(T)>), rows, waves, 0, st, a);
    for (int k = 0; k < T_; ++k) {
        const CgSlot *prev = k ? slots + (k - 1) : slots + T_;       // the initial state waits in the last slot
        double *in = parts + (size_t)((k + 1) & 1) * 4 * RED_MAX_PARTS, *out = parts + (size_t)(k & 1) * 4 * RED_MAX_PARTS;
        if (a.K <= 16) hipLaunchKernelGGL((dual_product_kernel<T, 1>), grid, block, 0, st, a, prev, k, in, nb);
        else if (a.K <= 32) hipLaunchKernelGGL((dual_product_kernel<T, 2>), grid, block, 0, st, a, prev, k, in, nb);
        else hipLaunchKernelGGL((dual_product_kernel<T, 4>), grid, block, 0, st, a, prev, k, in, nb);
        hipLaunchKernelGGL(dual_update_kernel, dim3((unsigned)nb), block, 0, st, a, prev, slots + k, k, in, out);
    }
    hipLaunchKernelGGL(dual_tail_kernel<T>, dim3((unsigned)nb), block, 0, st, a, slots + (T_ - 1), slots + T_, T_,
                       parts + (size_t)((T_ - 1) & 1) * 4 * RED_MAX_PARTS, yout, KP, slope_part);
    return hipGetLastError();
}

int dual_blocks(int64_t n, int K) { return (int)((n * K + 255) / 256); }

hipError_t launch_dual_cg(int dtype, DualCg a, CgSlot *slots, int T, double *work, void *yout, int KP, double *slope_part, hipStream_t st)
{
    (void)dual_doubles(a.n, a.K, &a.nks, &a.kper);
    const int64_t d = (int64_t)a.n * a.K;
    if (dual_blocks(a.n, a.K) > RED_MAX_PARTS || a.K > 64 || T < 1) return hipErrorInvalidValue;
    a.ld = (int32_t)gram_ld(a.n);
    double *vecs[] = {work, work + d, work + 2 * d, work + 3 * d, work + 4 * d, work + 5 * d, work + 6 * d, work + 7 * d, work + 8 * d};
    a.zg = vecs[0];
    a.w = vecs[1];
    a.u = vecs[2];
    a.xs[0] = vecs[3];
    a.xs[1] = vecs[4];
    a.yr = vecs[5];
    a.ys = vecs[6];
    a.yp = vecs[7];
    a.ybest = vecs[8];
    a.part = work + 9 * d;
    a.zu_part = a.part + a.nks * d;
    double *parts = a.zu_part + 64;
    if (dtype == SSN_F32) return dual_go<float>(a, slots, T, (float *)yout, KP, parts, slope_part, st);
    return dual_go<double>(a, slots, T, (double *)yout, KP, parts, slope_part, st);
}

}  // namespace ssn
