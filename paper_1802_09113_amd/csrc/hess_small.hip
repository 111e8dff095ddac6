// Newton directions of small problems on the dense layout: the sub-sampled Hessian is formed once and Alg. 2 runs on it
// in one workgroup.
//
// With d = p K of a few hundred, a matrix-free CG iteration is two dependent launches of some 5 us for a few hundred
// thousand multiply-adds: the launches and the trips to memory inside them are all of it.  H_S itself is small enough for
// the registers of ONE compute unit.  It is a K x K arrangement of p x p blocks
//   B_ab = X_S^T diag(q_a (delta_ab - q_b)) X_S        (eqs. (11)-(13) with the class sums written out),
// each symmetric, with B_ab = B_ba: K (K + 1) / 2 blocks are formed (hess_form_kernel, matrix cores) and every element
// serves both class pairs it stands for.  hess_cg_kernel then keeps them in registers and runs all of Alg. 2 without
// another launch, barriers of a workgroup in place of kernel boundaries, and leaves what the tail launches of the
// matrix-free form leave.  2000 x 50, three classes, 100 rows, fp64: direction of ten products 122 -> 45 us (forming 6,
// CG 21); 581012 x 54, seven classes, 5810 rows, fp32: 125 -> 89 us (forming 20, sum of its row chunks 4, CG 49).
#include "ssn_internal.h"
#include "ssn_math.h"

namespace ssn {

// ---- the plan ------------------------------------------------------------------------------------------
constexpr int HC_THREADS = 1024;
constexpr int HC_L = 8;                      // features per register strip of the CG kernel

// Strips per thread that are compiled.  The blocks are held in fp64 where that fits, up to four strips, whatever the data's
// precision; those of fp32 data beyond it in fp32, six or nine strips.
static constexpr int hc_upts[] = {1, 2, 4, 6, 9};
constexpr int HC_LDS = 150 * 1024;           // of 160 KB: the kernel's own arrays take 9

bool hess_small_plan(int dtype, int64_t p, int K, int64_t nS, int T, int num_cus, HessSmall *h)
{
    if (p * K > HC_THREADS || p > 512) return false;
    h->pairs = K * (K + 1) / 2;
    h->nc = (int)((p + HC_L - 1) / HC_L);
    h->pl = h->nc * HC_L;
    h->upt = 0;
    for (int u : hc_upts) {
        if (u > 4 && dtype != SSN_F32) break;
        if ((int64_t)h->pairs * h->nc * ((p + u - 1) / u) <= HC_THREADS) {
            h->upt = u;
            break;
        }
    }
    if (!h->upt) return false;
    const int64_t es = dtype == SSN_F32 ? 4 : 8;
    const int64_t pp = (p + h->upt - 1) / h->upt * h->upt, lds = ((int64_t)K * h->pl + (int64_t)K * K * h->nc * pp) * 8;
    if (lds > HC_LDS) return false;
    h->lds = (int)lds;
    const int nt = (int)((p + 63) / 64);
    h->nsup = nt * (nt + 1) / 2;
    // four waves of 16 rows and more; up to four chunks are added by the CG kernel as it loads
    int64_t chunks = nS <= 256 ? (nS + 63) / 64 : nS <= 512 ? 4 : (nS + 127) / 128, most = (int64_t)num_cus * 2 / ((int64_t)h->pairs * h->nsup);
    if (most < 1) most = 1;
    if (chunks > most) chunks = most;
    h->rows_per_chunk = ((nS + chunks - 1) / chunks + 63) / 64 * 64;
    h->chunks = (int)((nS + h->rows_per_chunk - 1) / h->rows_per_chunk);
    h->elems = (int64_t)h->pairs * p * h->pl;
    // fewer chunks: the CG kernel adds them as it loads; blocks held in fp32 are rounded by the launch that adds them (one
    // compute unit reads a megabyte of fp64 in 7 us more: p 54, K 6, 100 rows, T 4, direction 58 -> 51 us)
    h->summed = h->chunks > 4 || h->upt > 4;
    h->work = (h->chunks + (h->summed ? 1 : 0)) * h->elems;
    // Where the line lies: forming costs a time per row, class pair and pair of feature blocks and saves most of a
    // matrix-free product, T times; an iteration on blocks in fp32 takes 4 us (their elements are converted each time), and
    // matrix-free products of more than sixteen weight columns take two class tiles.  Directions of nS rows, matrix-free /
    // formed, in us:
    //   fp64, p 50, K 2:   T 10: nS 100 121/45, 200000 380/131;  T 4: 62/37, 165/119
    //   fp64, p 36, K 6:   T 10: nS 5000 129/75;                 T 4: nS 1000 61/44, 5000 64/65
    //   fp64, p 176, K 1:  T 10: nS 1000 126/61, 200000 1410/438
    //   fp32, p 54, K 6:   T 10: nS 5000 124/89, 60000 225/215;  T 4: nS 1000 59/51, 5000 62/65 (not)
    //   fp32, p 16, K 18:  T 10: nS 5000 167/136;                T 4: nS 1000 78/63
    //   fp32, p 153, K 2:  T 10: nS 5000 133/100, 60000 303/354 (not); T 4: nS 1000 61/57, 5000 65/80 (not)
    //   fp32, p 270, K 1:  T 10: nS 60000 538/303, 200000 1116/830
    //   fp32, p 8, K 31:   T 10: nS 1000 160/86;                 T 4: nS 100 79/44, 1000 77/76
    const bool f32 = dtype == SSN_F32, small = p <= 32;
    const double per = small ? (f32 ? 0.075e-3 : 0.1e-3) : h->nsup == 1 ? (f32 ? 0.11e-3 : 0.18e-3) : (f32 ? 0.25e-3 : 0.3e-3);
    const double forming = 15.0 + per * (double)nS * (double)h->pairs * (double)h->nsup;
    const double each = f32 && K > 16 ? 9.5 : h->upt <= 4 ? 6.5 : 5.3;
    const double saved = (double)T * (each + (double)nS * (double)p * (double)es / 3e6);
    return forming < saved;
}

// ---- forming the blocks --------------------------------------------------------------------------------
struct HessForm {
    const void *X;
    int64_t ldx, p;
    const int32_t *S;
    int64_t nS;
    const void *P;           // probabilities of the sample's rows, row stride KP
    int32_t KP, K;
    int32_t pairs, nsup, pl;
    int64_t rows_per_chunk;
    double *part;            // chunk x pair x p x pl
};

typedef double hv4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ hv4 hmfma(double a, double b, hv4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
// row of the 16 x 16 tile in accumulator element v of a lane in 16-lane group g
__device__ __forceinline__ int h_row(int g, int v) { return 4 * v + g; }

// The rows [lo, hi) of the sample into the NT x NT tiles of feature blocks I and J.  Both operands of the matrix
// instruction hold a feature per lane and a row per 16-lane group, so a loaded element is the left operand as it is and
// the right one after a multiplication with its row's weight: nothing is transposed.  The next 16 rows are on their way
// while the matrix cores work on these, their row numbers one step further ahead.
// Weights, products and sums are in fp64 whatever the data's precision.
template <typename T, int NT, bool DIAG>
__device__ __forceinline__ void form_rows(const HessForm &a, int64_t lo, int64_t hi, int I, int J, int ca, int cb,
                                          hv4 (&acc)[NT][NT])
{
    const int lane = threadIdx.x & 63, f = lane & 15, q = lane >> 4;
    const T *X = (const T *)a.X, *P = (const T *)a.P;
    int fi[NT], fj[NT];
    bool oi[NT], oj[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        fi[t] = I * 64 + t * 16 + f;
        fj[t] = J * 64 + t * 16 + f;
        oi[t] = fi[t] < a.p;
        oj[t] = fj[t] < a.p;
        if (!oi[t]) fi[t] = 0;
        if (!oj[t]) fj[t] = 0;
    }
    if (lo >= hi) return;
    T xi[4][NT], xj[DIAG ? 1 : 4][NT], pa[4], pb[4];
    int64_t src[4];
    auto rows = [&](int64_t r0) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int64_t r = r0 + 4 * s + q;
            src[s] = (int64_t)a.S[r < hi ? r : hi - 1];
        }
    };
    auto fetch = [&](int64_t r0) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int64_t r = r0 + 4 * s + q, rc = r < hi ? r : hi - 1;
            pa[s] = P[rc * a.KP + ca];
            pb[s] = P[rc * a.KP + cb];
            const T *x = X + src[s] * a.ldx;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                xi[s][t] = x[fi[t]];
                if constexpr (!DIAG) xj[s][t] = x[fj[t]];
            }
        }
    };
    rows(lo);
    fetch(lo);
    rows(lo + 16);
    for (int64_t r0 = lo; r0 < hi; r0 += 16) {
        double ai[4][NT], bj[4][NT];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bool in = r0 + 4 * s + q < hi;
            const double a1 = (double)pa[s], b1 = (double)pb[s], d = in ? (ca == cb ? a1 * (1.0 - a1) : -(a1 * b1)) : 0.0;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                ai[s][t] = (in && oi[t]) ? (double)xi[s][t] : 0.0;
                if constexpr (DIAG) bj[s][t] = d * ai[s][t];
                else bj[s][t] = (in && oj[t]) ? d * (double)xj[s][t] : 0.0;
            }
        }
        if (r0 + 16 < hi) {
            fetch(r0 + 16);
            rows(r0 + 32);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    if (!DIAG || i <= j) acc[i][j] = hmfma(ai[s][i], bj[s][j], acc[i][j]);
    }
}

template <typename T, int NT, bool DIAG> __device__ __forceinline__ void form_block(const HessForm &a, double *lds, int chunk, int pair, int I, int J,
                                                                              int ca, int cb)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t share = a.rows_per_chunk / 4;
    const int64_t lo = (int64_t)chunk * a.rows_per_chunk + w * share;
    const int64_t hi = lo + share < a.nS ? lo + share : a.nS;
    hv4 acc[NT][NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = hv4{0, 0, 0, 0};
    form_rows<T, NT, DIAG>(a, lo, hi, I, J, ca, cb, acc);
    // the four waves' tiles side by side in LDS, element (v, lane) of a tile at v * 64 + lane: a thread then adds the four
    // values of its place in every tile, in wave order
    constexpr int NTILES = DIAG ? NT * (NT + 1) / 2 : NT * NT;
    {
        int t = 0;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                if (DIAG && i > j) continue;
#pragma unroll
                for (int v = 0; v < 4; ++v) lds[(w * NTILES + t) * 256 + v * 64 + lane] = acc[i][j][v];
                ++t;
            }
    }
    __syncthreads();
    double *out = a.part + ((int64_t)chunk * a.pairs + pair) * a.p * a.pl;
    const int r = h_row(lane >> 4, w), c = lane & 15;             // here w stands for the accumulator element
    int t = 0;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            if (DIAG && i > j) continue;
            double x = lds[t * 256 + tid];
#pragma unroll
            for (int k = 1; k < 4; ++k) x += lds[(k * NTILES + t) * 256 + tid];
            const int64_t fr = I * 64 + i * 16 + r, fc = J * 64 + j * 16 + c;
            if (fr < a.p && fc < a.pl) out[fr * a.pl + fc] = x;
            if (!(DIAG && i == j) && fc < a.p && fr < a.pl) out[fc * a.pl + fr] = x;      // the block is symmetric
            ++t;
        }
}

// A workgroup of four waves per (row chunk, pair of feature blocks of 64, class pair); the waves share the chunk's rows
// and their sums are added in a fixed order.  What bounds it is the number of workgroups a sample gives and the chain
// row number -> row -> matrix instruction; its partials (one block per chunk) are kept few by the cap on the chunks.
// Two waves per SIMD: 27 -> 20 us for 5810 rows, p 54, K 6 in fp32 (15 us on fp32 matrix instructions).
// PAIRS: more than one feature block (NT = 4); a kernel of its own, as its sixteen tiles leave room for one wave per SIMD.
template <typename T, int NT, bool PAIRS> __global__ __launch_bounds__(256, PAIRS ? 1 : 2) void hess_form_kernel(HessForm a)
{
    extern __shared__ __align__(16) unsigned char hess_lds[];
    const int pair = blockIdx.x % a.pairs, rest = blockIdx.x / a.pairs;
    const int sup = rest % a.nsup, chunk = rest / a.nsup;
    int ca = 0, cb = pair;
    while (cb >= a.K - ca) {
        cb -= a.K - ca;
        ++ca;
    }
    cb += ca;
    const int nt = (int)((a.p + 63) / 64);
    int I = 0, J = sup;
    while (J >= nt - I) {
        J -= nt - I;
        ++I;
    }
    J += I;
    if (!PAIRS || I == J) form_block<T, NT, true>(a, (double *)hess_lds, chunk, pair, I, J, ca, cb);
    else if constexpr (PAIRS) form_block<T, NT, false>(a, (double *)hess_lds, chunk, pair, I, J, ca, cb);
}

// the blocks from the sums of their chunks, in chunk order
template <typename T> __global__ __launch_bounds__(VEC_BLOCK) void hess_sum_kernel(const double *part, T *H, int64_t total, int chunks)
{
    const int64_t e = (int64_t)blockIdx.x * VEC_BLOCK + threadIdx.x;
    if (e >= total) return;
    double s = 0.0;
    for (int c = 0; c < chunks; c += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(c + u < chunks ? c + u : c) * total + e];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += (c + u < chunks) ? v[u] : 0.0;
    }
    H[e] = (T)s;
}

// ---- Alg. 2 in one workgroup ---------------------------------------------------------------------------
// The wave sums red[0..16) added by a scan over a row of lanes, the same bits in every thread (one LDS read and four
// additions in sequence; sixteen reads would take 32 registers the strips need).
__device__ __forceinline__ double hc_total(const double *red)
{
    static_assert(HC_THREADS == 16 * 64, "a row of 16 lanes adds the wave sums");
    double r = red[threadIdx.x & 15];
    r += dpp_or_zero<0x111, 0xf>(r);
    r += dpp_or_zero<0x112, 0xf>(r);
    r += dpp_or_zero<0x114, 0xf>(r);
    r += dpp_or_zero<0x118, 0xf>(r);
    const long long b = __double_as_longlong(r);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), 15), hi = __builtin_amdgcn_readlane((int)(b >> 32), 15);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ __forceinline__ void hc_leave(double v, double *red)      // this wave's sum for hc_total behind a barrier
{
    v = wave_inclusive_scan(v);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
}

__device__ __forceinline__ void hc_state(CgSlot *w, double rr, double rbest, double gnorm, int done, int iters, int flags, double sHs)
{
    w->rr = rr;                              // field by field: a struct temporary would live in scratch memory
    w->rbest = rbest;
    w->gnorm = gnorm;
    w->done = done;
    w->iters = iters;
    w->flags = flags;
    w->brk = 0;
    w->alpha = 0.0;
    w->best_cur = 0;
    w->best_pending = 0;
    w->sHs = sHs;
    w->goff = 0.0;
    w->rho = w->sigma = w->pi = w->pibest = 0.0;
}

// Thread t holds UPT strips of eight features of the blocks: of block (ca, cb), features 8 chunk .. 8 chunk + 7, rows
// jb, jb + njb, ..  A product reads s (class-major, rows padded with zeros to whole strips) from LDS eight values at a
// time, every strip of the thread uses the same eight, and leaves two partial sums per strip, one for each of the
// classes: at (class, other class, chunk, row), so that the K * nc partials of an element are one stride apart.  Element e
// is feature e % p of class e / p, so that neighbouring threads read neighbouring partials.  What bounds it is instruction
// issue on one compute unit: hence the waves without elements skip the sums and scalars, and the partials are added by all
// threads.
// Precision (T: of the data and the vectors, HT: of the blocks): a product adds in fp64 all the way.  With fp32 multiplications
// and strip sums, and fp32 sums over rows behind them, directions of fp32 data were up to 3.6 times as far from fp64 ones as
// those of the matrix-free form, whose roundings, one per row and feature, average out over the sample.  Of 36 problems of
// fp32 data whose blocks do not fit in fp64 (HT = float) the error is 0.11 to 1.24 of the matrix-free one, 0.76 in the
// geometric mean.  Conversions and fp64 partials cost 1.4 us per product at p 54, K 6 (ten products 34 -> 49 us).
template <typename T, typename HT, int UPT> __global__ __launch_bounds__(HC_THREADS) void hess_cg_kernel(HessCg a)
{
    extern __shared__ __align__(16) unsigned char hess_lds[];
    __shared__ double red[2][HC_THREADS / 64], fold[HC_THREADS];
    __shared__ int ended;
    __shared__ double norm0, last_sHs;       // for the final state (registers less in the loop)
    const int K = a.K, p = a.p, nc = a.nc, pl = a.pl;
    double *sl = (double *)hess_lds, *pt = sl + K * pl;
    const int tid = threadIdx.x;
    // the strips
    const int njb = (p + UPT - 1) / UPT, pp = njb * UPT;             // pp: partials per strip column, rows past p are zeros
    const int jb = tid % njb, grp = tid / njb;
    const int chunk = grp % nc, pair = grp / nc;
    const bool mine = pair < a.pairs;
    int ca = 0, cb = mine ? pair : 0;
    while (cb >= K - ca) {
        cb -= K - ca;
        ++ca;
    }
    cb += ca;
    HT H[UPT][HC_L];
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
        const int j = jb + u * njb;
        const bool in = mine && j < p;
        const int64_t at = in ? ((int64_t)pair * p + j) * pl + chunk * HC_L : 0;
        if (sizeof(HT) == 4 || a.nsum == 0) {
            const HT *src = (const HT *)a.H + at;
#pragma unroll
            for (int k = 0; k < HC_L; ++k) H[u][k] = src[k];
        } else {
            const double *src = a.part + at;
#pragma unroll
            for (int k = 0; k < HC_L; ++k) H[u][k] = (HT)src[k];
            for (int c = 1; c < a.nsum; ++c) {
                src += a.elems;
#pragma unroll
                for (int k = 0; k < HC_L; ++k) H[u][k] += (HT)src[k];
            }
        }
#pragma unroll
        for (int k = 0; k < HC_L; ++k) H[u][k] = in ? H[u][k] : HT(0);
    }
    // this thread's element of the vectors
    const int N = p * K;
    const bool el = tid < N;
    const int ec = el ? tid / p : 0, ej = el ? tid - ec * p : 0;
    const int64_t off = (int64_t)ej * a.ld + ec;
    const T gv = el ? ((const T *)a.G)[off] : T(0);
    // the threads that add element ge's partials: rep 0 is the element's own thread
    const int Np = (N + 63) / 64 * 64, nrep = HC_THREADS / Np, npart = K * nc;
    const int rep = tid / Np, gi = tid - rep * Np, ge = gi < N ? gi : 0, gc = ge / p, gj = ge - gc * p;
    const bool ew = tid < Np;                // waves that hold elements; the others only multiply and wait at the barriers
    T pe = T(0), re = -gv, se = -gv, pb = -gv;
    for (int i = tid; i < K * pl; i += HC_THREADS) sl[i] = 0.0;
    if (tid < 2 * (HC_THREADS / 64)) (&red[0][0])[tid] = 0.0;
    __syncthreads();
    if (el) sl[ec * pl + ej] = (double)se;
    if (ew) hc_leave((double)gv * (double)gv, red[0]);
    __syncthreads();
    double rr = hc_total(red[0]);
    double rbest = sqrt(rr);
    const double stop_at = a.theta * rbest;
    int iters = 0, flags = 0;
    if (tid == 0) {
        ended = rr == 0.0 ? 1 : 0;
        norm0 = rbest;
        last_sHs = 0.0;
    }
    __syncthreads();
    while (!ended) {                         // the same in every thread: written behind a barrier, read in front of the next
        auto multiply = [&](int from, int to) {                      // the share of class `from` in class `to`
            double x[HC_L];
#pragma unroll
            for (int i = 0; i < HC_L; ++i) x[i] = sl[from * pl + chunk * HC_L + i];
            double *o = pt + ((to * K + from) * nc + chunk) * pp + jb;
#pragma unroll
            for (int u = 0; u < UPT; ++u) {
                if constexpr (sizeof(HT) == 4) {                     // converted here: left to itself the compiler keeps them all in fp64
#pragma unroll
                    for (int i = 0; i < HC_L; ++i) asm volatile("" : "+v"(H[u][i]));
                }
                double y = (double)H[u][0] * x[0];
#pragma unroll
                for (int i = 1; i < HC_L; ++i) y += (double)H[u][i] * x[i];
                o[u * njb] = y;
            }
        };
        if (mine) {
            multiply(cb, ca);
            if (ca != cb) multiply(ca, cb);
        }
        __syncthreads();
        // element e's K * nc partials, shared out among the threads e, e + Np, ..; their sums meet in LDS
        double t = 0.0;
        if (rep < nrep) {
            const double *o = pt + (gc * npart + rep) * pp + gj;
            const int step = nrep * pp;
            int i = rep;
            for (; i + 3 * nrep < npart; i += 4 * nrep, o += 4 * step) {
                const double v0 = o[0], v1 = o[step], v2 = o[2 * step], v3 = o[3 * step];
                t += v0 + v1;
                t += v2 + v3;
            }
            for (; i < npart; i += nrep, o += step) t += o[0];
        }
        if (nrep > 1) {
            if (!ew) fold[tid] = t;
            __syncthreads();
            if (ew)
                for (int i = 1; i < nrep; ++i) t += fold[i * Np + tid];
        }
        T hs = T(0);
        if (ew) {
            hs = el ? (T)(a.scale * t + a.lambda * (double)se) : T(0);
            hc_leave((double)se * (double)hs, red[0]);
        }
        __syncthreads();
        bool brk = false;
        double alpha = 0.0;
        if (ew) {
            const double sHs = hc_total(red[0]);
            if (tid == 0) last_sHs = sHs;
            brk = !(sHs > 0.0);              // not positive definite in floating point: stop, keep p_best
            if (!brk) {
                alpha = rr / sHs;
                pe = (T)((double)pe + alpha * (double)se);            // lines 8, 9
                re = (T)((double)re - alpha * (double)hs);
                hc_leave((double)re * (double)re, red[1]);
            }
        }
        __syncthreads();
        if (ew) {
            const double rrn = brk ? rr : hc_total(red[1]), rnorm = sqrt(rrn);
            const bool stop = !brk && rnorm <= stop_at;              // line 11
            if (tid == 0) {
                if (a.trace) {
                    a.trace[3 * iters] = alpha;
                    a.trace[3 * iters + 1] = rnorm;
                    a.trace[3 * iters + 2] = last_sHs;
                }
                ended = (brk || stop || iters + 1 >= a.T) ? 1 : 0;
            }
            ++iters;
            flags |= (stop ? 1 : 0) | (brk ? 2 : 0);
            if (!brk && rnorm <= rbest) {                             // line 10
                pb = pe;
                rbest = rnorm;
            }
            se = (T)((double)re + rrn / rr * (double)se);     // line 12
            rr = rrn;
            if (el) sl[ec * pl + ej] = (double)se;
        }
        __syncthreads();
    }
    if (el) ((T *)a.P)[off] = pb;
    double slope = 0.0;
    if (a.trial) {                           // inside ssn_solve: the first trial point, the slope, and what the host waits for
        if (el) ((T *)a.trial)[off] = (T)(1.0 * (double)pb + (double)((const T *)a.W)[off]);
        const T gl = el ? ((const T *)a.G)[off] : T(0);              // again: not held through the loop
        if (ew) hc_leave((double)pb * (double)gl, red[0]);
        __syncthreads();
        slope = hc_total(red[0]);
    }
    if (tid != 0) return;
    const double gnorm = norm0, sHs = last_sHs;
    const bool zero = gnorm == 0.0;
    hc_state(a.fin, rr, rbest, gnorm, zero || flags, iters, flags, sHs);
    if (!a.trial) return;
    *a.slope_dev = slope;
    a.host_out[0] = *a.f_dev;
    a.host_out[1] = slope;
    hc_state((CgSlot *)(a.host_out + 2), rr, rbest, gnorm, zero || flags, iters, flags, sHs);
}

template <typename T, int NT, bool PAIRS> static hipError_t form_go(const HessForm &f, int blocks, hipStream_t st)
{
    constexpr int lds = (int)sizeof(double) * 4 * 256 * (PAIRS ? NT * NT : NT * (NT + 1) / 2);       // the four waves' tiles
    static const hipError_t attr =
        hipFuncSetAttribute((const void *)hess_form_kernel<T, NT, PAIRS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((hess_form_kernel<T, NT, PAIRS>), dim3((unsigned)blocks), dim3(256), lds, st, f);
    return hipGetLastError();
}

template <typename T> static hipError_t form(const HessForm &f, int blocks, hipStream_t st)
{
    if (f.p <= 32) return form_go<T, 2, false>(f, blocks, st);
    return f.nsup > 1 ? form_go<T, 4, true>(f, blocks, st) : form_go<T, 4, false>(f, blocks, st);
}

template <typename T, typename HT, int UPT> static hipError_t cg_go(const HessCg &a, int lds, hipStream_t st)
{
    static const hipError_t attr =
        hipFuncSetAttribute((const void *)hess_cg_kernel<T, HT, UPT>, hipFuncAttributeMaxDynamicSharedMemorySize, HC_LDS);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((hess_cg_kernel<T, HT, UPT>), dim3(1), dim3(HC_THREADS), (size_t)lds, st, a);
    return hipGetLastError();
}

hipError_t launch_hess_small(int dtype, const HessSmall &h, const RowsArgs &r, const void *P, double *part, HessCg a, hipStream_t st)
{
    HessForm f{};
    f.X = r.X;
    f.ldx = r.ldx;
    f.p = r.p;
    f.S = r.S;
    f.nS = r.nrows;
    f.P = P;
    f.KP = r.KP;
    f.K = r.K;
    f.pairs = h.pairs;
    f.nsup = h.nsup;
    f.pl = h.pl;
    f.rows_per_chunk = h.rows_per_chunk;
    f.part = part;
    const int blocks = h.pairs * h.nsup * h.chunks;
    hipError_t e = dtype == SSN_F32 ? form<float>(f, blocks, st) : form<double>(f, blocks, st);
    if (e != hipSuccess) return e;
    a.part = part;
    a.nsum = h.chunks;
    if (h.summed) {
        void *H = part + h.chunks * h.elems;
        const unsigned b = (unsigned)((h.elems + VEC_BLOCK - 1) / VEC_BLOCK);
        if (h.upt > 4) hipLaunchKernelGGL(hess_sum_kernel<float>, dim3(b), dim3(VEC_BLOCK), 0, st, part, (float *)H, h.elems, h.chunks);
        else hipLaunchKernelGGL(hess_sum_kernel<double>, dim3(b), dim3(VEC_BLOCK), 0, st, part, (double *)H, h.elems, h.chunks);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        a.H = H;
        a.nsum = 0;
    }
    a.elems = h.elems;
    a.p = (int32_t)r.p;
    a.K = r.K;
    a.pairs = h.pairs;
    a.nc = h.nc;
    a.pl = h.pl;
    if (dtype == SSN_F32) {
        if (h.upt == 1) return cg_go<float, double, 1>(a, h.lds, st);
        if (h.upt == 2) return cg_go<float, double, 2>(a, h.lds, st);
        if (h.upt == 4) return cg_go<float, double, 4>(a, h.lds, st);
        if (h.upt == 6) return cg_go<float, float, 6>(a, h.lds, st);
        return cg_go<float, float, 9>(a, h.lds, st);
    }
    if (h.upt == 1) return cg_go<double, double, 1>(a, h.lds, st);
    if (h.upt == 2) return cg_go<double, double, 2>(a, h.lds, st);
    return cg_go<double, double, 4>(a, h.lds, st);
}

}  // namespace ssn
