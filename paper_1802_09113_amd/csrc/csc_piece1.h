// One weight column: the sums of the columns' pieces, a lane per piece (device code, shared by csc.hip and vecops.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ssn_math.h"

namespace ssn {

template <typename T> struct Piece1 {
    T x;                // the piece's sum
    int col, nextc;     // its column (-1 in lanes without a piece) and the next piece's
    bool head, more;    // the column's first piece; the column has further ones behind it
};

// Piece base + lane.  ALL: the sums of every piece; otherwise those of the columns of several pieces only (0 elsewhere).
template <typename T, bool ALL>
__device__ __forceinline__ Piece1<T> piece1_load(const int32_t *piece_col, int64_t npieces, const T *pp, int64_t base, int lane)
{
    const int64_t pid = base + lane;
    const bool have = pid < npieces;
    Piece1<T> q;
    q.col = have ? piece_col[pid] : -1;
    const int prevc = (have && pid > 0) ? piece_col[pid - 1] : -2;
    q.nextc = have ? piece_col[pid + 1] : -3;                    // (sentinels -1 behind the last piece)
    q.head = have && q.col != prevc;
    q.more = have && q.nextc == q.col;
    q.x = (ALL ? have : have && !(q.head && !q.more)) ? pp[pid] : T(0);
    return q;
}

// The sum of a column in the lane of its first piece, in a fixed order.  Every lane of the wave calls it.
template <typename T>
__device__ __forceinline__ T piece1_column_sum(const Piece1<T> &q, const int32_t *piece_col, int64_t npieces, const T *pp,
                                               int64_t base, int lane)
{
    T x = q.x;
    const int below = __shfl_up(q.col, 1);                       // (every lane takes part in the exchange)
    const bool start = lane == 0 || q.col != below;
    const unsigned long long starts = __ballot(start);
    const unsigned long long above = (lane == 63) ? 0ull : ((starts >> (lane + 1)) << (lane + 1));
    const int send = above ? (__ffsll((long long)above) - 2) : 63;
    for (int d = 1; d < 64; d <<= 1) {
        const T y = __shfl_down(x, d);
        if (lane + d <= send) x += y;
    }
    // The column of the wave's last piece may run on behind it; this wave follows it if the column starts here
    // (the wave where it starts does otherwise).
    const int lastcol = __shfl(q.col, 63);
    const int lastnext = __shfl(q.nextc, 63);
    const int laststart = 63 - __clzll(starts);                  // first lane of the last segment (lane 0 always starts one)
    const int lasthead = __shfl((int)q.head, laststart);
    T csum = T(0);
    if (lastcol >= 0 && lastnext == lastcol && lasthead) {       // uniform over the wave
        // 256 pieces per step, all their loads requested together (a piece that is not this column's is read and
        // dropped); the step's sum is the last lane's value of a scan over the lanes
        for (int64_t j0 = base + 64;; j0 += 256) {
            T y[4];
            bool m[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t j = j0 + 64 * k + lane, jc = j < npieces ? j : npieces - 1;
                const int c = piece_col[jc];
                const T pv = pp[jc];
                m[k] = j < npieces && c == lastcol;
                y[k] = m[k] ? pv : T(0);
            }
            const double t = ((double)y[0] + (double)y[1]) + ((double)y[2] + (double)y[3]);
            csum += (T)__shfl(wave_inclusive_scan(t), 63);
            if (!__all(m[3])) break;
        }
    }
    return send == 63 ? x + csum : x;
}

}  // namespace ssn
