// Device-side evaluation of a sharing polynomial at the party IDs 1, 2, ...
#pragma once
#include "field.hpp"

// values a0 + a[0] x + ... at x = 1..m (m <= M <= 8), canonical, handed to emit(x - 1, value); a0, a[] may be
// unreduced sums: a0 < 2 * 2^61 + 2^8, a[] < 2^61 + 2^8 (over the 45-bit prime: below 2^57).  Forward differences;
// in the bounds below one unit is 2^61 + 2^8 and a word holds less than eight.  PACED: the longer form of the
// reduction, which a kernel bound by its stores may prefer.
template <int T, int M, bool PACED = false, typename F>
__device__ __forceinline__ void eval_points(u64 a0, const u64 (&a)[T], F &&emit, int m = M)
{
    static_assert(T >= 1 && T <= 3 && M <= 8, "degrees 1 to 3, up to 8 points");
    auto reduce = [](u64 x) { return PACED ? ss_canon(ss_fold(x)) : ss_reduce(x); };
    u64 s = a0;
    if constexpr (T == 1) {
#pragma unroll
        for (int x = 1; x <= M; x++) {
            if (x > m) break;
            s = reduce(s + a[0]);
            emit(x - 1, s);
        }
    } else if constexpr (T == 2) {
        // d = s(x) - s(x-1) = a1 + (2x - 1) a2, its difference 2 a2; d is folded every other point from the fourth
        // on: 2, 4, 6 | 3, 5 | 3, 5 | 3 units
        u64 d = a[0] + a[1];
        const u64 dd = 2 * a[1];
#pragma unroll
        for (int x = 1; x <= M; x++) {
            if (x > m) break;
            if (x > 1) {
                if (x >= 4 && x % 2 == 0) d = ss_fold(d);
                d += dd;
            }
            s = reduce(s + d);
            emit(x - 1, s);
        }
    } else {
        // second differences e = 2 a2 + 6 (x - 1) a3; both are folded every other point: d 3, 2, 4, 2, 4, ... units, e at most 3
        const u64 f = ss_fold(6 * a[2]);
        u64 d = a[0] + a[1] + a[2], e = ss_fold(2 * a[1] + f);
#pragma unroll
        for (int x = 1; x <= M; x++) {
            if (x > m) break;
            if (x > 1) {
                if (x % 2 == 0) {
                    d = ss_fold(d);
                    e = ss_fold(e);
                }
                d += e;
                e += f;
            }
            s = reduce(s + d);
            emit(x - 1, s);
        }
    }
}
