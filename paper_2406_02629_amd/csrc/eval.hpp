// Device-side evaluation of a sharing polynomial at the party IDs 1, 2, ...
#pragma once
#include "field.hpp"

// values a0 + a[0] x + ... at x = 1..M (M <= 5), canonical, handed to emit(x - 1, value); a0, a[] may be unreduced
// sums: a0 < 2 * 2^61 + 2^8, a[] < 2^61 + 2^8 (over the 45-bit prime: below 2^58)
template <int T, int M, typename F>
__device__ __forceinline__ void eval_points(u64 a0, const u64 (&a)[T], F &&emit)
{
    static_assert((T == 1 || T == 2) && M <= 5, "degrees 1 and 2");
    u64 s = a0;
    if constexpr (T == 1) {
#pragma unroll
        for (int x = 1; x <= M; x++) {
            s = ss_reduce(s + a[0]);
            emit(x - 1, s);
        }
    } else {
        // first difference d_x = s(x) - s(x-1) = a1 + (2x - 1) a2, second difference 2 a2
        u64 d = a[0] + a[1];       // < 2 (2^61 + 2^8)
        const u64 dd = 2 * a[1];
#pragma unroll
        for (int x = 1; x <= M; x++) {
            if (x > 1) {
                if (x == 4) d = ss_fold(d);   // d_3 < 6 (2^61 + 2^8)
                d += dd;                      // d_5 < 5 (2^61 + 2^8) + 8
            }
            s = ss_reduce(s + d);   // s_1 + d_1 < 4 (2^61 + 2^8), then s < 2^61
            emit(x - 1, s);
        }
    }
}
