// Balanced radix-2^8 digits of field elements and their byte transposition, shared by the kernels that
// write int8 limb tiles or limb planes.
#pragma once
#include "field.hpp"

// balanced digits of x as 8 signed bytes: x = sum d_i 2^(8i), d_i in [-128, 127]
__device__ __forceinline__ u64 balanced_digits(u64 x) { return (x + 0x8080808080808080ULL) ^ 0x8080808080808080ULL; }

// one dword per limb from the digit words of four consecutive contraction indices (byte c of the result is
// digit `limb` of y[c]); limb may differ from lane to lane
__device__ __forceinline__ u32 limb_dword(const u64 (&y)[4], int limb)
{
    const int i = limb & 3;
    const u32 a = limb < 4 ? (u32)y[0] : (u32)(y[0] >> 32), b = limb < 4 ? (u32)y[1] : (u32)(y[1] >> 32);
    const u32 c = limb < 4 ? (u32)y[2] : (u32)(y[2] >> 32), d = limb < 4 ? (u32)y[3] : (u32)(y[3] >> 32);
    // v_perm_b32: selector byte k picks byte k of {second operand (0..3), first operand (4..7)}; 0x0c = zero
    const u32 sel = (u32)i | ((u32)(4 + i) << 8) | 0x0c0c0000u;
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, sel), __builtin_amdgcn_perm(b, a, sel), 0x05040100u);
}

// the values of v in the four lanes r, r + 16, r + 32, r + 48 of the caller's r, which all four call (register swaps: a
// shuffle by index goes through LDS)
__device__ __forceinline__ void gather_rows(u64 v, u64 (&y)[4])
{
    u32 h[2][4];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const u32 x = (u32)(v >> (32 * i));
        const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);   // rows 0 1 0 1, rows 2 3 2 3
        const auto lo = __builtin_amdgcn_permlane16_swap(a[0], a[0], false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(a[1], a[1], false, false);
        h[i][0] = lo[0], h[i][1] = lo[1], h[i][2] = hi[0], h[i][3] = hi[1];
    }
#pragma unroll
    for (int q = 0; q < 4; q++) y[q] = (u64)h[1][q] << 32 | h[0][q];
}

// Limb dwords of the digit words that the lanes of a 256-thread block hold one per party: lane l of wave w has row (pixel)
// l%16 and contraction index (channel) 4 w + l/16 of the block -> stage[party][limb][row][w].  The four lanes of a row
// swap their digit words, after which each of them owns all four and writes two of the limb dwords.
template <int MAXP>
__device__ __forceinline__ void stage_limbs(const u64 (&dig)[MAXP], u32 (&stage)[MAXP][SS_NLIMB][16][4], int n)
{
    const int lane = threadIdx.x & 63, r16 = lane & 15, j = lane >> 4, w = threadIdx.x >> 6;
#pragma unroll
    for (int p = 0; p < MAXP; p++) {
        if (p < n) {
            u64 y[4];
            gather_rows(dig[p], y);
            if (2 * j < SS_NLIMB) {
                stage[p][2 * j][r16][w] = limb_dword(y, 2 * j);
                stage[p][2 * j + 1][r16][w] = limb_dword(y, 2 * j + 1);
            }
        }
    }
    __syncthreads();
}

// ... and out of LDS: thread t of the 256 takes limb t/16 % SS_NLIMB of row t%16 for the parties t/(16 SS_NLIMB), that
// + 2, ... and writes its 16 bytes to where(party, limb, row) (nullptr: not at all); the 16 rows of a (party, limb) lie
// one after the other, so that 16 threads make 256 bytes in a row (a dword per wave would be a store of 4 of every 16
// bytes).
template <int MAXP, typename F>
__device__ __forceinline__ void store_staged(const u32 (&stage)[MAXP][SS_NLIMB][16][4], int n, F &&where)
{
    constexpr int PSTEP = 256 / (16 * SS_NLIMB);   // parties in flight: 2
    const int t = threadIdx.x, row = t & 15, limb = (t >> 4) % SS_NLIMB, p0 = t / (16 * SS_NLIMB);
    if (p0 >= PSTEP) return;
    for (int p = p0; p < n; p += PSTEP)
        if (signed char *dst = where(p, limb, row)) *reinterpret_cast<int4 *>(dst) = *reinterpret_cast<const int4 *>(&stage[p][limb][row][0]);
}

// to limb planes (per party [limb][channel block of 16][pixel][16 channels], int8): the channels c0..c0+15 of the pixels
// pix0..pix0+15
template <int MAXP>
__device__ __forceinline__ void store_staged_planes(const u32 (&stage)[MAXP][SS_NLIMB][16][4],
                                                    signed char *__restrict__ planes, size_t party_bytes, size_t plane,
                                                    int pix0, int npix, int c0, int n)
{
    store_staged<MAXP>(stage, n, [&](int p, int limb, int px) {
        return pix0 + px < npix ? planes + p * party_bytes + limb * plane + ((size_t)(c0 >> 4) * npix + pix0 + px) * 16 : nullptr;
    });
}
