// The margins of one CSR row (device code, shared by csr.hip and csr_dual.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace ssn {

// Weight columns per lane: 16 bytes of a row where it is that long
template <typename T> inline int row_vec(int K)
{
    const int most = 16 / (int)sizeof(T);
    return K >= most ? most : K >= 2 ? 2 : 1;
}

// z_c = sum over the stored entries b .. e - 1 (the same for the whole wave) of x * M[col, c], in lane c; zero in lanes from
// K on.  VEC weight columns to a lane, 16 bytes of a row of M where it is that long: ceil(K / VEC) lanes take an entry, the
// last one the last VEC columns (those its neighbour has, too, are not used).  What bounds a pass is the gathers a wave has
// on the way to memory: with a lane per column and eight bytes per load there were three entries per load instruction at
// K = 19, now six (fp64) or twelve (fp32).  20000 rows of 450 entries, 1.36 million columns, K 19, all rows: objective 286
// -> 198 us, margins 277 -> 186 us in fp64, gradient pass 165 -> 116 us in fp32.  A: what the products are added up in.
template <typename T, typename A, int VEC>
__device__ __forceinline__ A csr_row_margin_vec(const int32_t *colidx, const T *vals, const T *M0, int64_t ldm, int64_t b, int64_t e, int lane,
                                                int K)
{
    struct __attribute__((packed, aligned(sizeof(T)))) pack { T v[VEC]; };      // rows of M start at any element
    const int L = (K + VEC - 1) / VEC, NS = 64 / L;
    const int s = lane / L, cl = lane - s * L, c0 = cl * VEC < K - VEC ? cl * VEC : K - VEC;
    const T *M = M0 + c0;
    A acc[2][VEC];
#pragma unroll
    for (int m = 0; m < VEC; ++m) acc[0][m] = acc[1][m] = A(0);
    // N entries per slot from place t on, added up in two sums of their own (a row's chain of additions is one per round, and
    // four within).  ALL: every slot has its N; otherwise places behind the row's end read its last entry and count as 0 * 0
    // -- not as 0 * M, which is no zero where a weight is infinite.
    auto take = [&](auto n, auto all, int64_t t) {
        constexpr int N = decltype(n)::value;
        constexpr bool ALL = decltype(all)::value;
        int64_t cc[N];
        T vv[N];
        pack mm[N];
#pragma unroll
        for (int u = 0; u < N; ++u) cc[u] = colidx[ALL || t + u * NS < e ? t + u * NS : e - 1];
#pragma unroll
        for (int u = 0; u < N; ++u) vv[u] = vals[ALL || t + u * NS < e ? t + u * NS : e - 1];
#pragma unroll
        for (int u = 0; u < N; ++u) mm[u] = *(const pack *)(M + cc[u] * ldm);
        A sum[2][VEC];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const bool in = ALL || t + u * NS < e;
            const A x = in ? (A)vv[u] : A(0);
#pragma unroll
            for (int m = 0; m < VEC; ++m) {
                const A w = in ? (A)mm[u].v[m] : A(0);
                sum[u & 1][m] = u < 2 ? x * w : sum[u & 1][m] + x * w;
            }
        }
#pragma unroll
        for (int m = 0; m < VEC; ++m) {
            acc[0][m] += sum[0][m];
            if constexpr (N > 1) acc[1][m] += sum[1][m];
        }
    };
    if (s < NS) {
        int64_t t = b;                                          // (t and e are the same for the whole wave)
        for (; t + 8 * NS <= e; t += 8 * NS) take(std::integral_constant<int, 8>{}, std::true_type{}, t + s);
        const int64_t left = e - t;
        if (left > 4 * NS) take(std::integral_constant<int, 8>{}, std::false_type{}, t + s);
        else if (left > 2 * NS) take(std::integral_constant<int, 4>{}, std::false_type{}, t + s);
        else if (left > NS) take(std::integral_constant<int, 2>{}, std::false_type{}, t + s);
        else if (left > 0) take(std::integral_constant<int, 1>{}, std::false_type{}, t + s);
    }
    int top = 1;
    while (top < NS) top <<= 1;
    A tot[VEC];
#pragma unroll
    for (int m = 0; m < VEC; ++m) tot[m] = acc[0][m] + acc[1][m];
    for (int h = top >> 1; h >= 1; h >>= 1) {
#pragma unroll
        for (int m = 0; m < VEC; ++m) {
            const A o = __shfl(tot[m], (lane + h * L) & 63);
            if (s + h < NS) tot[m] += o;
        }
    }
    // column c from its lane of the first slot to lane c
    const int src = lane / VEC < L ? lane / VEC : 0, at = lane - (src * VEC < K - VEC ? src * VEC : K - VEC);
    A z = A(0);
#pragma unroll
    for (int m = 0; m < VEC; ++m) {
        const A o = __shfl(tot[m], src);
        if (at == m) z = o;
    }
    return (lane < K) ? z : A(0);
}

}  // namespace ssn
