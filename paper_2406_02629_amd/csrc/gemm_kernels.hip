// Exact modular matrix product on int8 MFMA (SSS-Linear step 1, Sec. VI-A).
//
// A field element x < 2^61 is written in balanced radix 2^8,
//   x = sum_{i<8} d_i 2^(8i),  d_i in [-128, 127],
// which is one add and one xor: the bytes of x + 0x80..80 are d_i + 128.  The
// integer dot product sum_k x_k w_k is then sum_{i,j} 2^(8(i+j)) sum_k d_i(x_k)
// d_j(w_k): 64 int8 dot products.  Only the 15 anti-diagonal sums
//   D_s = sum_{i+j=s} sum_k d_i(x_k) d_j(w_k),   |D_s| <= 8 K 2^14 < 2^31 for K <= 16383,
// are needed, so the 64 MFMA 16x16x64 products of a 16 x 16 tile of field
// outputs accumulate straight into 15 int32 accumulator tiles (the MFMA's own
// C operand does the diagonal sum).  The epilogue turns the 15 sums of each
// output into a 61-bit residue with 2^61 = 1 (mod p) and stores the canonical
// field element.
//
// Built for p = 2^45 - 55 (Sec. VII-A) an element has 6 digits (x < 2^45 leaves
// digits 6 and 7 zero): 36 products, 11 diagonal sums, tiles and limb planes
// three quarters the size, and the epilogue folds with 2^45 = 55 (mod p).
#include "kernels.hpp"
#include "eval.hpp"
#include "digits.hpp"

#include <hip/hip_ext.h>

namespace SS_NS {

typedef int v4i __attribute__((ext_vector_type(4)));

namespace {

// NL digits per field element (8 for p = 2^61 - 1, 6 for p = 2^45 - 55: the digits above are zero), hence
// ND anti-diagonal sums; a packed tile (16 rows x 64 contraction indices) is NL limb slices of 64 lanes x
// 16 bytes = TILE 16-byte words
constexpr int NL = SS_NLIMB, ND = 2 * NL - 1, TILE = NL * 64;

// Lane (r, j) = r + 16 j of a wave holds the digit words y of the contraction indices (or channels) 4 j .. 4 j + 3 of row r,
// that is one dword per limb.  Transposed over j by register swaps, it holds the 16 bytes of limb j and those of limb
// 4 + j of its row, so that a wave stores 256 contiguous bytes per limb, 16 per lane, in two stores.  (As dwords, 8 stores,
// each quarter of a wave met two cache lines in parts and the four quarters the same two: the stores bound the kernels.
// Limb planes of 8 images of 64 x 56 x 56 with their sharing, n = 3: 21.9 -> 15.1 us; limb tiles of 4 shares of 500 x 1201 and
// 1201 x 333: 23.3 -> 14.9 us; of a 7 x 7 stem at 224 x 224, n = 5: 37.7 -> 26.3 us.)  store(limb, 16 bytes); the four
// lanes of a row call together.
template <typename F>
__device__ __forceinline__ void store_limbs(const u64 (&y)[4], int j, F &&store)
{
    u32 w[8];
#pragma unroll
    for (int limb = 0; limb < 8; limb++) w[limb] = limb < NL ? limb_dword(y, limb) : 0;
#pragma unroll
    for (int h = 0; h < 8; h += 4) {
        const auto a = __builtin_amdgcn_permlane32_swap(w[h], w[h + 2], false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(w[h + 1], w[h + 3], false, false);
        const auto lo = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
        if (h + j < NL) store(h + j, (v4i){(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]});
    }
}

// One workgroup per (row block, k block) tile, one thread per (row, 4 contraction indices): thread t -> row t%16, k group
// t/16.  grid (Rb * Kb, n), block 256; the index along which the source is contiguous runs fastest over the workgroups
// (k_first), an XCD's workgroups are neighbours, and elements outside the matrix are loaded from its first one, so that a
// thread's four loads are in flight together (a load per branch waits for each).
// taps > 0: the contraction index of the packed operand runs (tap, channel) while the source runs (channel,
// tap) with `taps` taps per channel (convolution weights for the kernel that reads its other operand from
// limb planes); stride_k is then the stride of the source's own index.  tap_blocks > 0: k blocks of a tap (C a multiple of 64);
// the taps of 64 channels, which share their cache lines, are neighbours then (in the order of the packed operand an XCD's
// workgroups took one tap of all channels and every XCD read all of them; 3 x 3 taps, n = 5, us: 9 x 512 channels 5.1 -> 3.4, 453 x 512
// 65 -> 48).
__global__ __launch_bounds__(256) void pack_matrix_kernel(const u64 *__restrict__ src, v4i *__restrict__ dst,
                                                          int rows, int K, int Rb, int Kb, fdiv dRb, fdiv dKb, bool k_first,
                                                          size_t party_stride, size_t stride_r, size_t stride_k,
                                                          size_t dst_party_stride, int taps, int tap_blocks, fdiv dTaps)
{
    const int b = (int)xcd_slot(blockIdx.x, gridDim.x), q = (int)fd_div((u32)b, k_first ? dKb : dRb);
    const int rb = k_first ? q : b - q * Rb;
    int kb = k_first ? b - q * Kb : q;
    const int r16 = threadIdx.x & 15, kq = threadIdx.x >> 4, row = rb * 16 + r16;
    const u64 *s = src + (size_t)blockIdx.y * party_stride + (row < rows ? (size_t)row * stride_r : 0);
    u64 y[4];
    if (tap_blocks) {   // uniform
        const int channels = (int)fd_div((u32)kb, dTaps), tap = kb - channels * taps;   // block of channels
        kb = tap * tap_blocks + channels;
        s += (size_t)(channels * 64 + 4 * kq) * taps + tap;
#pragma unroll
        for (int c = 0; c < 4; c++) y[c] = s[c * taps];
    } else {
        const int C = taps ? K / taps : 1;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const int k = kb * 64 + 4 * kq + c, ks = k >= K ? 0 : taps ? (k % C) * taps + k / C : k;
            y[c] = s[(size_t)ks * stride_k];
        }
    }
#pragma unroll
    for (int c = 0; c < 4; c++) y[c] = row < rows && kb * 64 + 4 * kq + c < K ? balanced_digits(y[c]) : 0;
    v4i *tile = dst + (size_t)blockIdx.y * dst_party_stride + ((size_t)rb * Kb + kb) * TILE + r16 + 16 * (kq >> 2);
    store_limbs(y, kq & 3, [&](int limb, v4i v) { tile[limb * 64] = v; });
}

// The same for two operands with one contraction in one launch (a dense layer whose operands both change: 500 x 333 x 1201, n = 4, 14.9 us in
// two launches, 12.6 us in one, and no gap): the blocks of `a` come first, in the order of its contraction, then those of `b`, in the order of its rows.
struct pack_job {
    const u64 *src;
    v4i *dst;
    int rows, Rb, blocks;
    fdiv dFast;              // of the blocks along the index that runs fastest
    size_t party_stride, stride_r, stride_k, dst_party_stride;
};
__global__ __launch_bounds__(256) void pack_pair_kernel(pack_job a, pack_job b, int K, int Kb)
{
    const bool first = (int)blockIdx.x < a.blocks;   // uniform
    const pack_job j = first ? a : b;
    const int at = (int)xcd_slot(first ? blockIdx.x : blockIdx.x - a.blocks, j.blocks), q = (int)fd_div((u32)at, j.dFast);
    const int rb = first ? q : at - q * j.Rb, kb = first ? at - q * Kb : q;
    const int r16 = threadIdx.x & 15, kq = threadIdx.x >> 4, row = rb * 16 + r16, k0 = kb * 64 + 4 * kq;
    const u64 *s = j.src + (size_t)blockIdx.y * j.party_stride + (row < j.rows ? (size_t)row * j.stride_r : 0);
    u64 y[4];
#pragma unroll
    for (int c = 0; c < 4; c++) y[c] = s[(size_t)(k0 + c < K ? k0 + c : 0) * j.stride_k];
#pragma unroll
    for (int c = 0; c < 4; c++) y[c] = row < j.rows && k0 + c < K ? balanced_digits(y[c]) : 0;
    v4i *tile = j.dst + (size_t)blockIdx.y * j.dst_party_stride + ((size_t)rb * Kb + kb) * TILE + r16 + 16 * (kq >> 2);
    store_limbs(y, kq & 3, [&](int limb, v4i v) { tile[limb * 64] = v; });
}

// rows = (b, ho, wo), k = (c, r, s) gathered from x [n][B][C][H][W]; zero padding.  An element is gathered once per tap, so
// the index arithmetic is kept short: divisions by constants of the launch, and a thread's four loads unconditional (taps in the
// padding and indices past the matrix load the tensor's first element).
struct im2col_args {
    int H, W, kh, kw, stride, pad, M, K, Kb;
    fdiv dTaps, dKw, dWo, dHoWo;
    int HoWo, Wo;
    size_t image, party;     // elements
};
__global__ __launch_bounds__(256) void pack_im2col_kernel(const u64 *__restrict__ x, v4i *__restrict__ dst, im2col_args g,
                                                          size_t dst_party_stride)
{
    const int rb = blockIdx.x, kb = blockIdx.y, r16 = threadIdx.x & 15, kq = threadIdx.x >> 4;
    const int row = rb * 16 + r16, k0 = kb * 64 + 4 * kq, taps = g.kh * g.kw;
    const int b = (int)fd_div((u32)row, g.dHoWo), hw = row - b * g.HoWo, ho = (int)fd_div((u32)hw, g.dWo), wo = hw - ho * g.Wo;
    int c = (int)fd_div((u32)k0, g.dTaps), rs = k0 - c * taps, r = (int)fd_div((u32)rs, g.dKw), s = rs - r * g.kw;
    const int h0 = ho * g.stride - g.pad, w0 = wo * g.stride - g.pad;
    const u64 *xi = x + blockIdx.z * g.party;
    u64 y[4];
    bool in[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const int hi = h0 + r, wi = w0 + s;
        in[q] = row < g.M && k0 + q < g.K && (unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W;
        y[q] = xi[in[q] ? b * g.image + ((size_t)c * g.H + hi) * g.W + wi : 0];
        if (++s == g.kw) { s = 0; if (++r == g.kh) { r = 0; ++c; } }
    }
#pragma unroll
    for (int q = 0; q < 4; q++) y[q] = in[q] ? balanced_digits(y[q]) : 0;
    v4i *tile = dst + (size_t)blockIdx.z * dst_party_stride + ((size_t)rb * g.Kb + kb) * TILE + r16 + 16 * (kq >> 2);
    store_limbs(y, kq & 3, [&](int limb, v4i v) { tile[limb * 64] = v; });
}

// The two kernels below take one element per thread: lane l of a wave holds row (or pixel) l%16 and the
// contraction index (or channel) 4 g + l/16 of the wave's group g of four, and the limb dwords of the block leave
// through LDS (stage_limbs).  The layers of a batch-1 network are small: one element per thread is what fills the chip.

// shares of element e of the plaintext tensor, as GEN (Eq. 1) draws them (element index = position in the
// tensor, so the values are those of the plain share kernel): stored, and returned as digit words
template <int N, int T>
__device__ __forceinline__ void gen_digits(const u64 *__restrict__ secret, u64 *__restrict__ shares, size_t count,
                                           size_t e, int n, int t, const ss_keys &keys, u64 (&dig)[N ? N : SS_MAXN])
{
    constexpr int MAXP = N ? N : SS_MAXN, MAXD = T ? T : SS_MAXT;
    const u64 a0 = secret[e], counter = ss_counter(e);
    u64 c[MAXD];
#pragma unroll
    for (int j = 0; j < MAXD; j++) c[j] = (j < t) ? ss_draw_field_at(keys.k[j], counter) : 0;
    if constexpr (N != 0) {
        eval_points<T, N>(a0, c, [&](int p, u64 v) {
            shares[(size_t)p * count + e] = v;
            dig[p] = balanced_digits(v);
        });
    } else {
#pragma unroll
        for (int p = 0; p < MAXP; p++) {
            if (p < n) {
                const u64 v = ss_poly_eval<MAXD>(a0, c, t, p + 1);
                shares[(size_t)p * count + e] = v;
                dig[p] = balanced_digits(v);
            }
        }
    }
}

// GEN (Eq. 1) of the input of a dense or 1x1 convolution layer and its limb
// tiles in one pass.  The secret is [B][K][HW] (dense: HW = 1); operand row
// (b, hw), contraction index k.  grid (row blocks, 4 Kb), block 256: wave w of
// block (rb, y) takes the group of four contraction indices 4 y + w of row block
// rb.  N, T > 0 fix the scheme at compile time, 0 takes the run-time values.
template <int N, int T>
__global__ __launch_bounds__(256) void share_pack_kernel(const u64 *__restrict__ secret, u64 *__restrict__ shares,
                                                         v4i *__restrict__ dst, int B, int K, int HW, int Kb,
                                                         size_t dst_party_stride, int n_rt, int t_rt, ss_keys keys)
{
    constexpr int MAXP = N ? N : SS_MAXN;
    const int n = N ? N : n_rt, t = T ? T : t_rt;
    const int lane = threadIdx.x & 63, r16 = lane & 15, j = lane >> 4;
    const int g = blockIdx.y * 4 + (threadIdx.x >> 6), kb = g >> 4, kq = g & 15;
    const int rb = blockIdx.x, row = rb * 16 + r16, k = kb * 64 + 4 * kq + j, rows = B * HW;
    u64 dig[MAXP];
#pragma unroll
    for (int p = 0; p < MAXP; p++) dig[p] = 0;   // digits of padding rows and columns
    if (row < rows && k < K) {
        const int b = row / HW, hw = row - b * HW;
        gen_digits<N, T>(secret, shares, (size_t)B * K * HW, ((size_t)b * K + k) * HW + hw, n, t, keys, dig);
    }
    __shared__ __align__(16) u32 stage[MAXP][NL][16][4];   // [party][limb][row][wave]
    stage_limbs<MAXP>(dig, stage, n);
    signed char *tile = reinterpret_cast<signed char *>(dst + ((size_t)rb * Kb + kb) * TILE + 16 * (kq >> 2));   // kq / 4 is the same for all waves
    store_staged<MAXP>(stage, n, [&](int p, int limb, int r) { return tile + (p * dst_party_stride + limb * 64 + r) * 16; });
}

// Conv input [B][C][H][W] -> limb planes [party][limb][channel block of 16][b][h][w][16 channels] (int8), the form
// the convolution kernel gathers its second operand from: 16 consecutive channels of one tap of one output pixel
// are 16 consecutive bytes, and those of neighbouring pixels follow one another, so that a wave's gather is (all
// but) contiguous.  (With all channels innermost four neighbouring lanes meet four cache lines, and such loads run
// at 16 bytes per clock and CU instead of 64, measured on data in L2; cache accesses of a launch over 8 images of
// 64 x 56 x 56, n = 3: 22.2 million with all channels innermost, 15.0 as it is, 13.2 from packed tiles.)  GEN: the input is the plaintext tensor and the kernel also is GEN (Eq. 1):
// it writes the n shares and their planes; otherwise the input is the share tensor [n][B][C][H][W].
// grid (pixel blocks of 16, C / 16), block 256: wave w of block (x, y) takes channels 16 y + 4 w .. +3.
// Every party's planes end in a pad whose first 16 bytes are zero (the source of taps in the padding).
template <int N, int T, bool GEN>
__global__ __launch_bounds__(256) void planes_kernel(const u64 *__restrict__ in, u64 *__restrict__ shares,
                                                     signed char *__restrict__ planes, int B, int C, int HW,
                                                     size_t party_bytes, int n_rt, int t_rt, ss_keys keys)
{
    constexpr int MAXP = N ? N : SS_MAXN;
    const int n = N ? N : n_rt, t = T ? T : t_rt;
    const int lane = threadIdx.x & 63, r16 = lane & 15, j = lane >> 4;
    const int pix = blockIdx.x * 16 + r16, c0 = blockIdx.y * 16 + 4 * (threadIdx.x >> 6);
    const size_t plane = (size_t)B * HW * C;
    if (blockIdx.x == 0 && blockIdx.y == 0 && (int)threadIdx.x < n)
        *reinterpret_cast<v4i *>(planes + threadIdx.x * party_bytes + NL * plane) = (v4i){0, 0, 0, 0};
    u64 dig[MAXP];
#pragma unroll
    for (int p = 0; p < MAXP; p++) dig[p] = 0;
    const bool live = pix < B * HW;
    if (live) {
        const int b = pix / HW, hw = pix - b * HW;
        const size_t e = ((size_t)b * C + (c0 + j)) * HW + hw;
        if constexpr (GEN) {
            gen_digits<N, T>(in, shares, plane, e, n, t, keys, dig);
        } else {
#pragma unroll
            for (int p = 0; p < MAXP; p++)
                if (p < n) dig[p] = balanced_digits(in[(size_t)p * plane + e]);
        }
    }
    __shared__ __align__(16) u32 stage[MAXP][NL][16][4];   // [party][limb][pixel][wave]
    stage_limbs<MAXP>(dig, stage, n);
    store_staged_planes<MAXP>(stage, planes, party_bytes, plane, blockIdx.x * 16, B * HW, blockIdx.y * 16, n);
}

// The same with four channels per thread (thread t of block (pixel block, channel block of 64): pixel t%16,
// channels from 4 (t/16)): fewer, longer threads, the better shape for large tensors.
template <int N, int T, bool GEN>
__global__ __launch_bounds__(256) void planes4_kernel(const u64 *__restrict__ in, u64 *__restrict__ shares,
                                                     signed char *__restrict__ planes, int B, int C, int HW,
                                                     size_t party_bytes, int n_rt, int t_rt, ss_keys keys)
{
    constexpr int MAXP = N ? N : SS_MAXN, MAXD = T ? T : SS_MAXT;
    const int n = N ? N : n_rt, t = T ? T : t_rt;
    const int pix = blockIdx.x * 16 + (threadIdx.x & 15), c0 = blockIdx.y * 64 + 4 * (threadIdx.x >> 4);
    const size_t plane = (size_t)B * HW * C, count = plane;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < MAXP && (int)threadIdx.x < n)
        *reinterpret_cast<v4i *>(planes + threadIdx.x * party_bytes + NL * plane) = (v4i){0, 0, 0, 0};
    if (pix >= B * HW) return;
    const int b = pix / HW, hw = pix - b * HW;
    u64 y[MAXP][4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const size_t e = ((size_t)b * C + (c0 + q)) * HW + hw;
        if constexpr (GEN) {
            const u64 a0 = in[e], counter = ss_counter(e);
            u64 c[MAXD];
#pragma unroll
            for (int j = 0; j < MAXD; j++) c[j] = (j < t) ? ss_draw_field_at(keys.k[j], counter) : 0;
            if constexpr (N != 0) {
                eval_points<T, N>(a0, c, [&](int p, u64 v) {
                    shares[(size_t)p * count + e] = v;
                    y[p][q] = balanced_digits(v);
                });
            } else {
#pragma unroll
                for (int p = 0; p < MAXP; p++) {
                    if (p < n) {
                        const u64 v = ss_poly_eval<MAXD>(a0, c, t, p + 1);
                        shares[(size_t)p * count + e] = v;
                        y[p][q] = balanced_digits(v);
                    }
                }
            }
        } else {
#pragma unroll
            for (int p = 0; p < MAXP; p++)
                if (p < n) y[p][q] = balanced_digits(in[(size_t)p * count + e]);
        }
    }
#pragma unroll
    for (int p = 0; p < MAXP; p++) {
        if (p < n) {
            v4i *dst = reinterpret_cast<v4i *>(planes + p * party_bytes) + (size_t)(c0 >> 4) * (B * HW) + pix;
            store_limbs(y[p], (c0 >> 2) & 3, [&](int limb, v4i v) { dst[limb * (plane / 16)] = v; });
        }
    }
}

struct gemm_args {
    const v4i *A, *B;          // packed operands, all parties
    u64 *out, *parts;          // the first plane of the product; the others (tiles computed in parts), part_stride elements apart
    size_t part_stride;
    int rows, cols, Rb, Cb, Kb, RT, CT;
    unsigned units;            // tiles * Kb, or 0: whole tiles only
    unsigned whole;            // tiles 0 .. whole - 1 are dealt whole, each workgroup's before its range of units
    unsigned cost0;            // cost position of the first tile dealt by units (number `whole`)
    unsigned wlast;            // cost of one unit of the last column tile (SS_UNIT_COST for the others)
    unsigned tcost, tlast;     // cost of a whole tile, fold included: all column tiles but the last; the last
    unsigned share, rest;      // (cost of all tiles - cost0) / G and % G for the G workgroups of the launch
    int slots;                 // planes: the most workgroups that can share a tile (>= 1)
    fdiv dG, dKb, dCT, dRT, dRowcost, dTilecost, dWlast, dCdiv;
    size_t a_party_stride, b_party_stride, out_party_stride, stride_row, stride_cb;
    int cdiv;
    // second operand read straight from limb planes (convolution without a materialised im2col): planes
    // [party][limb][channel block of 16][b][h][w][16] int8, contraction index (tap, channel), C a multiple of 64
    const v4i *planes, *zero;          // zero: 16 zero bytes, for taps that fall into the padding
    unsigned plane16, party16;         // strides of a limb plane and of a party, in 16-byte units
    int cvH, cvW, cvPixels, cvKw, cvStride, cvPad, cvHoWo, cvWo, cvKbTap;   // Pixels = images * H * W, KbTap = C/64
    fdiv dHoWo, dWo, dKbTap, dKw;
    // second operand read straight from field elements (gemm_ksplit_kernel): the rows of a dense input [party][cols][K], or the taps of a
    // convolution input [party][b][c][h][w] with contraction index (channel, tap)
    const u64 *raw;
    size_t raw_party, raw_image;       // elements
    int K, cvTaps;
    fdiv dTaps;
};

// where one wave's block of a unit comes from: limb slice q is the 64 lanes x 16 bytes at base + q * qs
struct wave_src {
    const v4i *p;    // block pointer (packed operand), or the party's planes (implicit operand)
    int hw, bpix;    // implicit operand: (h0 << 16) | (w0 & 0xffff) of this lane's output pixel, and the
                     // pixel index of its image, -1 if the lane's column is past the matrix
};

// a * b + c, one instruction (the compiler turns a multiplication by a power of two into a sign extension,
// a 64-bit shift and a 64-bit addition)
__device__ __forceinline__ long long mad_i64(int a, int b, long long c)
{
    long long d;
    asm("v_mad_i64_i32 %0, vcc, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c) : "vcc");
    return d;
}

// D_0 + D_1 2^8 + D_2 2^16 (+ D_3 2^24): up to four of the signed 32-bit diagonal sums in one signed 64-bit
// word, |result| < 2^31 (1 + 2^8 + 2^16 + 2^24) < 2^56
__device__ __forceinline__ long long join4(int d0, int d1, int d2, int d3)
{
    return mad_i64(d3, 1 << 24, mad_i64(d2, 1 << 16, mad_i64(d1, 1 << 8, (long long)d0)));
}
__device__ __forceinline__ long long join3(int d0, int d1, int d2)
{
    return mad_i64(d2, 1 << 16, mad_i64(d1, 1 << 8, (long long)d0));
}

// The ND diagonal sums of one output -> canonical field element.  The sums are signed 32-bit numbers and
// stay signed: four of them at a time go into one signed 64-bit word, the words are joined with the field's
// reduction rule, and a multiple of p makes the total positive before it is reduced.
#if defined(SS_FIELD_P45)
__device__ __forceinline__ u64 fold_diagonals(const v4i (&acc)[ND], int r)
{
    const long long off = (long long)(SS_P << 12);   // a multiple of p above 2^56
    const u64 g0 = (u64)(join4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]) + off);
    const u64 g1 = (u64)(join4(acc[4][r], acc[5][r], acc[6][r], acc[7][r]) + off);
    const u64 g2 = (u64)(join3(acc[8][r], acc[9][r], acc[10][r]) + off);
    // g0 + g1 2^32 + g2 2^64.  With g = a 2^13 + b: g 2^32 = a 2^45 + b 2^32 = 55 a + b 2^32, and
    // 2^64 = 55 2^19 (mod p)
    const u64 r1 = ss_reduce(g1), r2 = ss_reduce(g2);
    const u64 t1 = SS_PC * (r1 >> 13) + ((r1 & 0x1FFFull) << 32);   // < 2^38 + 2^45
    const u64 t2 = ss_mul(r2, SS_PC << 19);
    return ss_reduce(ss_fold(g0) + t1 + t2);
}
#else
__device__ __forceinline__ u64 fold_diagonals(const v4i (&acc)[15], int r)
{
    const long long g0 = join4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
    const long long g1 = join4(acc[4][r], acc[5][r], acc[6][r], acc[7][r]);
    const long long g2 = join4(acc[8][r], acc[9][r], acc[10][r], acc[11][r]);
    const long long g3 = join3(acc[12][r], acc[13][r], acc[14][r]);
    // g0 + g1 2^32 + g2 2^64 + g3 2^96 with 2^61 = 1: 2^64 = 2^3, 2^96 = 2^35 = 2^3 2^32
    const long long lo = g0 + (g2 << 3), hi = g1 + (g3 << 3);   // |.| < 2^60
    // hi 2^32 = (hi >> 29) 2^61 + (hi mod 2^29) 2^32 = (hi >> 29) + (hi mod 2^29) 2^32
    const long long tot = lo + (hi >> 29) + (long long)(((u64)hi & ((1ULL << 29) - 1)) << 32) + (long long)(2 * SS_P);
    return ss_reduce((u64)tot);   // 2^61 < tot < 2^63
}
#endif

// The units are dealt to the workgroups by cost, not by count.  A unit of a full tile costs SS_UNIT_COST; a
// unit of the last column tile, where only some of the four column blocks exist and the MFMAs of the others
// are skipped, costs less (see unit_cost); and every tile ends with its fold and stores, which cost about as
// much as a unit (SS_FOLD_COST; a workgroup whose range holds the ends of two tiles really is busy that much
// longer than one whose range lies inside one tile).  On the cost axis a tile is its units followed by its
// fold; with cp(u) the position of unit u, workgroup s of G owns the units with bound(s) <= cp(u) <
// bound(s + 1), bound(s) = cost0 + floor(s (cost - cost0) / G).  (cost - cost0) / G >= SS_UNIT_COST + SS_FOLD_COST, the
// largest step between two unit starts, so no range is empty.
//
// Where there are tiles for several rounds of the chip, the workgroups first take equal runs of whole tiles and the rest is dealt by
// cost: the last 256 to 511 tiles, or one or more rounds besides (all tiles, if it comes to that) where ragged tiles among them would
// leave ranges shorter than a full tile.  The tiles taken whole need no second plane.
__device__ __forceinline__ unsigned range_bound(const gemm_args &g, unsigned s)
{
    return g.cost0 + s * g.share + fd_div(s * g.rest, g.dG);   // s <= G <= 256, rest < G
}

// first unit whose cost position is >= x (x <= cost); positions inside a tile's fold belong to the next tile
__device__ __forceinline__ unsigned unit_at(const gemm_args &g, unsigned x)
{
    const unsigned full = ((unsigned)g.CT - 1) * g.tcost, rowcost = full + g.tlast;
    const unsigned rg = fd_div(x, g.dRowcost), rem = x - rg * rowcost;
    unsigned ct, j;
    if (rem < full) {
        ct = fd_div(rem, g.dTilecost);
        j = (rem - ct * g.tcost + SS_UNIT_COST - 1) / SS_UNIT_COST;
    } else {
        ct = (unsigned)g.CT - 1;
        j = fd_div(rem - full + g.wlast - 1, g.dWlast);
    }
    j = min(j, (unsigned)g.Kb);   // j == Kb: first unit of the next tile
    return (rg * (unsigned)g.CT + ct) * (unsigned)g.Kb + j;
}

// tile -> (column tile, row tile, party)
__device__ __forceinline__ void tile_coords(const gemm_args &g, unsigned tile, int &ct, int &rt, int &party)
{
    const unsigned rem = fd_div(tile, g.dCT);
    ct = (int)(tile - rem * (unsigned)g.CT);
    party = (int)fd_div(rem, g.dRT);
    rt = (int)(rem - (unsigned)party * (unsigned)g.RT);
}

// where column block cb of a party's second operand comes from (blocks past the end are clamped: their products are
// computed and never stored)
template <bool IMPLICIT>
__device__ __forceinline__ wave_src column_source(const gemm_args &g, int party, int cb, int lane)
{
    wave_src ws = {nullptr, 0, 0};
    if (!IMPLICIT) {
        ws.p = g.B + (size_t)party * g.b_party_stride + (size_t)min(cb, g.Cb - 1) * g.Kb * TILE + lane;
    } else {
        // lane l of a block holds column 16 cb + l%16 = output pixel (b, ho, wo)
        const int col = min(cb, g.Cb - 1) * 16 + (lane & 15);
        const int cc = min(col, g.cols - 1), b = (int)fd_div((u32)cc, g.dHoWo), r = cc - b * g.cvHoWo,
                  ho = (int)fd_div((u32)r, g.dWo), wo = r - ho * g.cvWo;
        ws.p = g.planes + (size_t)party * g.party16;
        ws.hw = (int)((unsigned)(ho * g.cvStride - g.cvPad) << 16) | ((wo * g.cvStride - g.cvPad) & 0xffff);
        ws.bpix = col < g.cols ? b * g.cvH * g.cvW : -1;
    }
    return ws;
}

// this wave's source block of tile `tile`: block `wave` of A for waves 0..3, of
// B for waves 4..7
template <bool IMPLICIT>
__device__ __forceinline__ wave_src tile_source(const gemm_args &g, unsigned tile, int wave, int lane)
{
    int ct, rt, party;
    tile_coords(g, tile, ct, rt, party);
    if (wave >= 4) return column_source<IMPLICIT>(g, party, ct * 4 + wave - 4, lane);
    return {g.A + (size_t)party * g.a_party_stride + (size_t)min(rt * 4 + wave, g.Rb - 1) * g.Kb * TILE + lane, 0, 0};
}

// base address and limb stride (16-byte units) of a column block for k block kb
template <bool IMPLICIT>
__device__ __forceinline__ const v4i *column_base(const gemm_args &g, const wave_src &ws, int kb, int lane, unsigned &qs)
{
    if (!IMPLICIT) {
        qs = 64;
        return ws.p + (size_t)kb * TILE;
    }
    // k block kb = channels [64 (kb % KbTap), +64) of tap kb / KbTap; this lane: 16 of them
    const int tap = (int)fd_div((u32)kb, g.dKbTap), c16 = (kb - tap * g.cvKbTap) * 4 + (lane >> 4);
    const int r = (int)fd_div((u32)tap, g.dKw), sx = tap - r * g.cvKw;
    const int hi = (ws.hw >> 16) + r, wi = (int)(short)(ws.hw & 0xffff) + sx;
    const bool ok = ws.bpix >= 0 && (unsigned)hi < (unsigned)g.cvH && (unsigned)wi < (unsigned)g.cvW;
    qs = ok ? g.plane16 : 0;
    return ok ? ws.p + (size_t)c16 * g.cvPixels + (ws.bpix + hi * g.cvW + wi) : g.zero;
}

// the same for the block of a wave of the big kernel
template <bool IMPLICIT>
__device__ __forceinline__ const v4i *unit_base(const gemm_args &g, const wave_src &ws, int kb, int wave, int lane,
                                                unsigned &qs)
{
    if (!IMPLICIT || wave < 4) {
        qs = 64;
        return ws.p + (size_t)kb * TILE;
    }
    return column_base<IMPLICIT>(g, ws, kb, lane, qs);
}

// What the column operand of gemm_ksplit_kernel is.
enum column_operand { IN_TILES, IN_PLANES, IN_ROWS, IN_IMAGES };

// The 16 elements that lane l of a block in MFMA order holds of an operand given as field elements: column 16 cb + l%16, contraction
// indices 64 kb + 16 (l/16) and on; zero outside the matrix and in the padding of an image.  (Places outside are loaded from the
// tensor's first element, so that a lane's loads are in flight together.)
template <column_operand OPERAND>
__device__ __forceinline__ void load_elements(const gemm_args &g, int party, int cb, int kb, int lane, u64 (&y)[16], unsigned &inside)
{
    const int col = cb * 16 + (lane & 15), k0 = kb * 64 + 16 * (lane >> 4);
    const u64 *x = g.raw + (size_t)party * g.raw_party;
    inside = 0;
    if constexpr (OPERAND == IN_ROWS) {
        const size_t row = (size_t)col * g.K;
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const bool in = col < g.cols && k0 + i < g.K;
            inside |= (unsigned)in << i;
            y[i] = x[in ? row + (k0 + i) : 0];
        }
    } else {
        const int b = (int)fd_div((u32)col, g.dHoWo), hw = col - b * g.cvHoWo, ho = (int)fd_div((u32)hw, g.dWo), wo = hw - ho * g.cvWo;
        const int h0 = ho * g.cvStride - g.cvPad, w0 = wo * g.cvStride - g.cvPad;
        int c = (int)fd_div((u32)k0, g.dTaps), rs = k0 - c * g.cvTaps, r = (int)fd_div((u32)rs, g.dKw), q = rs - r * g.cvKw;
        const int kh = g.cvTaps / g.cvKw;
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int hi = h0 + r, wi = w0 + q;
            const bool in = col < g.cols && k0 + i < g.K && (unsigned)hi < (unsigned)g.cvH && (unsigned)wi < (unsigned)g.cvW;
            inside |= (unsigned)in << i;
            y[i] = x[in ? b * g.raw_image + ((size_t)c * g.cvH + hi) * g.cvW + wi : 0];
            if (++q == g.cvKw) { q = 0; if (++r == kh) { r = 0; ++c; } }
        }
    }
}

// ... as the lane's 16 bytes of every limb
__device__ __forceinline__ void limbs_of(const u64 (&y)[16], unsigned inside, v4i (&b)[NL])
{
    u64 d[4][4];
#pragma unroll
    for (int i = 0; i < 16; i++) d[i >> 2][i & 3] = inside >> i & 1 ? balanced_digits(y[i]) : 0;
#pragma unroll
    for (int l = 0; l < NL; l++)
        b[l] = (v4i){(int)limb_dword(d[0], l), (int)limb_dword(d[1], l), (int)limb_dword(d[2], l), (int)limb_dword(d[3], l)};
}

__device__ __forceinline__ u64 *plane_at(const gemm_args &g, unsigned plane)
{
    return plane ? g.parts + (size_t)(plane - 1) * g.part_stride : g.out;
}

// Planes that get zeros from workgroup `slot`, whose range ends at unit u1.  A workgroup that starts a tile
// sees to the planes that no part of the tile goes to.  For a tile it computes whole that is all planes but
// its own; the only tile it can start and not finish is the one its range ends in, which has one more part
// for every following workgroup whose range starts before the tile ends (at most slots parts in all).
__device__ __forceinline__ int zero_planes_of_cut_tile(const gemm_args &g, unsigned u1, unsigned slot, unsigned G)
{
    const unsigned tile_end = (fd_div(u1, g.dKb) + 1) * (unsigned)g.Kb;
    int nc = 1;
    while (slot + nc < G && nc < g.slots && unit_at(g, range_bound(g, slot + nc)) < tile_end) nc++;
    return g.slots - nc;
}

// Persistent kernel, one workgroup of 8 waves (4 x 2) per CU.  The work is the
// flat list of units (output tile of 64 x 64, k block of 64), tile-major; each
// workgroup takes one contiguous range of it, of equal cost, so every CU gets
// the same amount of work whatever the layer shape.  Wave (wr, wc) owns row
// block wr and column blocks 2wc, 2wc+1 of the tile (2 x 15 accumulator tiles);
// the two waves of a SIMD differ in wc.
//
// Per unit the workgroup needs four row blocks of A and four column blocks of
// B, 8 KB each and already in MFMA lane order, so wave w copies block w (A for
// w < 4, B otherwise) straight into LDS with eight 1 KB global->LDS loads; two
// stages, the next unit's loads (also across a tile boundary) in flight during
// the 128 MFMAs per wave of the current one.
//
// A tile whose k range is cut by a range boundary is computed in parts by
// consecutive workgroups, and nothing passes between them: the output is
// `slots` planes, workgroup `slot` stores what it has of a tile (folded to a
// field element) in plane slot % slots -- the workgroups that share a tile are
// consecutive and at most `slots`, so they hit different planes -- and whoever
// reads the product adds the planes mod p.  The workgroup that starts a tile
// gives the planes nobody writes zeros, so every position of every plane is
// written by exactly one workgroup in every launch.  Integer sums are exact, so
// the sum of the planes does not depend on how the units were dealt.
//
template <bool IMPLICIT>
__global__ __launch_bounds__(512) void gemm_limb_kernel(gemm_args g)
{
    extern __shared__ v4i lds[];   // 2 stages x (4 A blocks + 4 B blocks) x TILE
    constexpr int STAGE = 8 * TILE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wr = wave & 3, wc = wave >> 2;
    const unsigned G = gridDim.x;
    const unsigned slot = xcd_slot(blockIdx.x, G);
    const unsigned myplane = g.slots > 1 ? slot % (unsigned)g.slots : 0;
    // its whole tiles w0 .. w1 - 1 and its range of units u0 .. u1 - 1; u counts the units of the one, then of the other
    unsigned w0 = 0, w1 = 0, u0 = 0, u1 = 0;
    if (g.whole) {
        w0 = g.whole == G ? slot : (unsigned)((unsigned long long)slot * g.whole / SS_GEMM_CUS);
        w1 = g.whole == G ? slot + 1 : (unsigned)((unsigned long long)(slot + 1) * g.whole / SS_GEMM_CUS);
    }
    if (g.units) {
        u0 = unit_at(g, range_bound(g, slot));
        u1 = unit_at(g, range_bound(g, slot + 1));
    }
    bool range_ahead = g.whole && u0 < u1;
    unsigned u = g.whole ? 0 : u0, uend = g.whole ? (w1 - w0) * (unsigned)g.Kb : u1;
    if (u >= uend) return;
    unsigned ucopy = uend + (range_ahead ? 1 : 0);   // units below have a copy to send for the next one
    const unsigned range_tile = fd_div(u0, g.dKb);
    const int range_kb = (int)(u0 - range_tile * (unsigned)g.Kb);
    v4i *mine = lds + wave * TILE;   // wave-uniform LDS destination of this wave's block

    unsigned tile = g.whole ? w0 : range_tile;
    int kb = g.whole ? 0 : range_kb;
    wave_src src = tile_source<IMPLICIT>(g, tile, wave, lane);
    {
        unsigned qs;
        const v4i *ub = unit_base<IMPLICIT>(g, src, kb, wave, lane, qs);
#pragma unroll
        for (int q = 0; q < NL; q++) __builtin_amdgcn_global_load_lds(ub + (size_t)q * qs, mine + q * 64, 16, 0, 0);
    }
    int st = 0;
    // (worked out while the first unit is on its way)
    const int zero_cut = g.slots > 1 ? zero_planes_of_cut_tile(g, u1, slot, G) : 0;

    while (u < uend) {
        int ct, rt, party;
        tile_coords(g, tile, ct, rt, party);
        // column blocks of this wave that lie inside the matrix (0 if its row block lies outside): MFMAs of
        // blocks past the edge are skipped, so a ragged last tile costs only its valid part
        const int nblk = rt * 4 + wr >= g.Rb ? 0 : max(0, min(2, g.Cb - (ct * 4 + 2 * wc)));
        const int kb_first = kb;
        v4i acc[2][ND];
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int s = 0; s < ND; s++) acc[h][s] = (v4i){0, 0, 0, 0};

        // units of this tile that belong to this workgroup
        const int kb_end = min(g.Kb, kb + (int)(uend - u));
        wave_src next_src = src;
        for (; kb < kb_end; kb++, u++) {
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's part of the unit is in LDS
            __syncthreads();                      // everyone's part is; stage st^1 is no longer read
            // first the LDS reads of this unit's first half, then the copies of the next unit: right behind
            // the barrier both waves of a SIMD are reading and the MFMA pipe idles, so that stretch is kept short
            const v4i *sa = lds + st * STAGE + wr * TILE + lane;
            const v4i *sb = lds + st * STAGE + 4 * TILE + wc * 2 * TILE + lane;
            v4i a[NL], b[NL];
            if (nblk >= 1) {
#pragma unroll
                for (int i = 0; i < NL; i++) {
                    a[i] = sa[i * 64];
                    b[i] = sb[i * 64];
                }
            }
            // where the next unit's block comes from (nothing is loaded yet)
            const bool more = u + 1 < ucopy;
            const v4i *cp = nullptr;
            unsigned cqs = 64;
            if (more) {
                int nkb = kb + 1;
                if (nkb == g.Kb) {
                    const bool jump = u + 1 == uend;   // to the range: it follows on a whole tile
                    nkb = jump ? range_kb : 0;
                    next_src = tile_source<IMPLICIT>(g, jump ? range_tile : tile + 1, wave, lane);
                }
                cp = unit_base<IMPLICIT>(g, next_src, nkb, wave, lane, cqs);
            }
            v4i *cdst = mine + (st ^ 1) * STAGE;
            if (nblk == 2 && more) {
                // the usual case in one run of instructions: the copies of the next unit go out one by one between
                // the MFMAs of the first column block, so that their issue hides behind matrix work
#pragma unroll
                for (int i = 0; i < NL; i++) {
#pragma unroll
                    for (int j = 0; j < NL; j++)
                        acc[0][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[0][i + j], 0, 0, 0);
                    __builtin_amdgcn_global_load_lds(cp + (size_t)i * cqs, cdst + i * 64, 16, 0, 0);
                }
#pragma unroll
                for (int j = 0; j < NL; j++) b[j] = sb[TILE + j * 64];
#pragma unroll
                for (int i = 0; i < NL; i++)
#pragma unroll
                    for (int j = 0; j < NL; j++)
                        acc[1][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[1][i + j], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < NL; i++) {
                    __builtin_amdgcn_sched_group_barrier(0x008, NL, 0);   // NL MFMAs
                    __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);    // one copy
                }
            } else {
                if (more) {
#pragma unroll
                    for (int q = 0; q < NL; q++) __builtin_amdgcn_global_load_lds(cp + (size_t)q * cqs, cdst + q * 64, 16, 0, 0);
                }
                // MFMAs of column blocks past the matrix edge are skipped (nblk < 2; uniform over the wave)
                if (nblk >= 1) {
#pragma unroll
                    for (int i = 0; i < NL; i++)
#pragma unroll
                        for (int j = 0; j < NL; j++)
                            acc[0][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[0][i + j], 0, 0, 0);
                }
                if (nblk == 2) {
#pragma unroll
                    for (int j = 0; j < NL; j++) b[j] = sb[TILE + j * 64];
#pragma unroll
                    for (int i = 0; i < NL; i++)
#pragma unroll
                        for (int j = 0; j < NL; j++)
                            acc[1][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[1][i + j], 0, 0, 0);
                }
            }
            st ^= 1;
        }

        // The part is done.  Lane holds, per column block h, column lane%16 and rows 4*(lane/16)+r of its
        // wave's 16 x 32 outputs.
        const int lrow = rt * 64 + wr * 16 + 4 * (lane >> 4);
        u64 v[2][4];
        size_t off[2];        // element offset inside a plane of this lane's first row, per column block
        unsigned mask = 0;    // bit 4h + r: value (h, r) lies inside the matrix
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int col = ct * 64 + wc * 32 + (lane & 15) + 16 * h;
            const u32 cq = fd_div((u32)col, g.dCdiv);
            off[h] = (size_t)party * g.out_party_stride + (size_t)cq * g.stride_cb + ((u32)col - cq * (u32)g.cdiv) +
                     (size_t)lrow * g.stride_row;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                if (h < nblk) v[h][r] = fold_diagonals(acc[h], r);
                if (h < nblk && col < g.cols && lrow + r < g.rows) mask |= 1u << (4 * h + r);
            }
        }
        // a tile dealt whole lies in the first plane alone
        const bool in_range = tile >= g.whole;
        const unsigned pl = in_range ? myplane : 0;
        const int nzero = (g.slots > 1 && in_range && kb_first == 0) ? (kb_end == g.Kb ? g.slots - 1 : zero_cut) : 0;
        u64 *o = plane_at(g, pl);
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (mask >> (4 * h + r) & 1) o[off[h] + (size_t)r * g.stride_row] = v[h][r];
        for (int z = 0; z < nzero; z++) {
            unsigned zpl = myplane + (unsigned)(g.slots - nzero + z);
            if (zpl >= (unsigned)g.slots) zpl -= (unsigned)g.slots;
            u64 *zo = plane_at(g, zpl);
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int r = 0; r < 4; r++)
                    if (mask >> (4 * h + r) & 1) zo[off[h] + (size_t)r * g.stride_row] = 0;
        }
        if (kb == g.Kb) {
            kb = 0;
            tile++;
            src = next_src;
            if (u == uend && range_ahead) {
                range_ahead = false;
                u = u0, uend = ucopy = u1, tile = range_tile, kb = range_kb;
            }
        }
    }
}

// The same contraction for products that are too small, or too narrow, for tiles of 64 x 64 and operands shared through LDS:
// there a launch lasts as long as its chain of dependent steps, or as it takes to read the one large operand once.  A wave
// owns a tile of 16 x 16, takes every KS-th of the k blocks and reads both operand blocks straight into registers, the
// next unit's while the MFMAs of the current one run; the KS waves that share a tile add their residues through LDS.  CW
// tiles, neighbours in the list, make a workgroup.  Where that leaves CUs idle the k blocks are also divided into `parts` equal
// runs, each with a plane of its own (every tile has all of them).
// Of the smallest products (element_waves) the column operand may be field elements: a wave takes the digits of its block itself, once per
// row block, which saves the launch that would pack them.
template <column_operand OPERAND, int KS>
__global__ __launch_bounds__(KS == 8 ? 512 : 256, 2) void gemm_ksplit_kernel(gemm_args g, fdiv dParts)
{
    constexpr bool ELEMENTS = OPERAND == IN_ROWS || OPERAND == IN_IMAGES;
    constexpr int NW = KS == 8 ? 8 : 4, CW = NW / KS;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), cw = wave % CW, ks = wave / CW;
    const unsigned slot = xcd_slot(blockIdx.x, gridDim.x);
    const unsigned group = fd_div(slot, dParts), part = slot - group * (unsigned)g.slots;
    // tile `block` of the list: party-major, then the longer side of the product, then the shorter one, so that the tiles
    // that read one block of the longer side are neighbours
    auto coords = [&](unsigned block, int &cb, int &rb, int &party) {
        int minor, major;
        tile_coords(g, block, minor, major, party);
        cb = g.Rb < g.Cb ? major : minor;
        rb = g.Rb < g.Cb ? minor : major;
    };
    const unsigned block = group * CW + cw;
    int cb, rb, party;
    coords(block, cb, rb, party);
    const bool inside = block < g.units;
    const int k0 = (int)fd_div(part * (unsigned)g.Kb, dParts) + ks, k1 = (int)fd_div((part + 1) * (unsigned)g.Kb, dParts);

    v4i acc[ND];
#pragma unroll
    for (int s = 0; s < ND; s++) acc[s] = (v4i){0, 0, 0, 0};
    if (inside) {
        const v4i *const pa = g.A + (size_t)party * g.a_party_stride + (size_t)rb * g.Kb * TILE + lane;
        auto load_row_block = [&](v4i (&a)[NL], int kb) {
#pragma unroll
            for (int q = 0; q < NL; q++) a[q] = pa[(size_t)kb * TILE + q * 64];
        };
        auto multiply = [&](const v4i (&a)[NL], const v4i (&b)[NL]) {
#pragma unroll
            for (int i = 0; i < NL; i++)
#pragma unroll
                for (int j = 0; j < NL; j++)
                    acc[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[i + j], 0, 0, 0);
        };
        if constexpr (ELEMENTS) {
            for (int kb = k0; kb < k1; kb += KS) {   // (one, see element_waves)
                u64 y[16];
                unsigned in = 0;
                v4i a[NL], b[NL];
                load_elements<OPERAND>(g, party, cb, kb, lane, y, in);
                load_row_block(a, kb);
                limbs_of(y, in, b);
                multiply(a, b);
            }
        } else {
            const wave_src src = column_source<OPERAND == IN_PLANES>(g, party, cb, lane);
            auto load = [&](v4i (&a)[NL], v4i (&b)[NL], int kb) {
                unsigned qs;
                const v4i *pb = column_base<OPERAND == IN_PLANES>(g, src, kb, lane, qs);
#pragma unroll
                for (int q = 0; q < NL; q++) {
                    a[q] = pa[(size_t)kb * TILE + q * 64];
                    b[q] = pb[(size_t)q * qs];
                }
            };
            v4i a0[NL], b0[NL], a1[NL], b1[NL];
            if (k0 < k1) load(a0, b0, k0);
            for (int kb = k0; kb < k1; kb += 2 * KS) {
                if (kb + KS < k1) load(a1, b1, kb + KS);
                multiply(a0, b0);
                if (kb + KS < k1) {
                    if (kb + 2 * KS < k1) load(a0, b0, kb + 2 * KS);
                    multiply(a1, b1);
                }
            }
        }
    }

    // lane holds column lane%16 and rows 4*(lane/16)+r of its tile
    u64 v[4];
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = fold_diagonals(acc, r);
    auto store = [&](unsigned which, int r, u64 value) {
        int scb, srb, sparty;
        coords(which, scb, srb, sparty);
        const int row = srb * 16 + 4 * (lane >> 4) + r, col = scb * 16 + (lane & 15);
        if (which >= g.units || row >= g.rows || col >= g.cols) return;
        const u32 cq = fd_div((u32)col, g.dCdiv);
        plane_at(g, part)[(size_t)sparty * g.out_party_stride + (size_t)cq * g.stride_cb + ((u32)col - cq * (u32)g.cdiv) +
                          (size_t)row * g.stride_row] = value;
    };
    if constexpr (KS == 1) {
#pragma unroll
        for (int r = 0; r < 4; r++) store(block, r, v[r]);
    } else {
        __shared__ u64 sums[NW][4][64];
#pragma unroll
        for (int r = 0; r < 4; r++) sums[wave][r][lane] = v[r];
        __syncthreads();
        // wave w adds the KS residues of the (tile, row) pairs w, w + NW, ... of the CW x 4
        for (int i = wave; i < 4 * CW; i += NW) {
            u64 x = sums[i >> 2][i & 3][lane];
#pragma unroll
            for (int k = 1; k < KS; k++) x = ss_add(x, sums[k * CW + (i >> 2)][i & 3][lane]);
            store(group * CW + (i >> 2), i & 3, x);
        }
    }
}

// Products of a few to some tens of units per CU: four waves share two row blocks and two column blocks through LDS, so that the
// caches give 32 KB (24 KB over the 45-bit prime) for four units of 16 x 16, where a wave of the kernel above takes them 64 KB (48 KB)
// by itself.  A workgroup owns a tile of 32 x 32 and one of `runs` equal runs of its k blocks (each run has a plane); wave w
// copies block w.  There is one stage: the operands of a unit go to registers, and the next ones are copied while the MFMAs run; three
// workgroups on a CU (four) fill each other's waits (two stages and two workgroups: 16.6 -> 17.4 us for 1024 x 196 x 256, n = 5, which waves on
// their own take 19.5 for; its matrix work lasts 8.2).  What the first copies need arrives in registers: the rest of the arguments
// is loaded meanwhile.
// (blocks: row blocks | column blocks << 16; ks: k blocks | runs << 16; reciprocals of the tiles along the shorter and the longer side and of
// the runs; G: workgroups, which gridDim would load from memory)
template <bool IMPLICIT>
__global__ __launch_bounds__(256, NL == 8 ? 3 : 4) void gemm_square_kernel(const v4i *A, const v4i *B, u32 blocks, u32 ks, u32 minor_m, u32 minor_s,
                                                                          u32 major_m, u32 major_s, u32 runs_m, u32 runs_s, u32 G, gemm_args g)
{
    __shared__ v4i lds[4 * TILE];   // 2 row blocks + 2 column blocks
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wr = wave & 1, wc = wave >> 1;
    const int Rb = (int)(blocks & 0xffff), Cb = (int)(blocks >> 16), Kb = (int)(ks & 0xffff);
    const unsigned runs = ks >> 16;
    // party, run, longer side of the product, shorter side: workgroups that read the same blocks are neighbours, and those of a run read
    // its share of them only (run by run against run fastest: 512 x 392 x 2048, n = 5, two runs, 103 -> 101 us; 512 x 196 x 1024 29.6 -> 29.0)
    const unsigned place = xcd_slot(blockIdx.x, G), q = fd_div(place, fdiv{minor_m, minor_s}), upper = fd_div(q, fdiv{major_m, major_s});
    const unsigned Rt = (unsigned)(Rb + 1) / 2, Ct = (unsigned)(Cb + 1) / 2, minor = place - q * min(Rt, Ct), major = q - upper * max(Rt, Ct);
    const int party = (int)fd_div(upper, fdiv{runs_m, runs_s}), rt = (int)(Rt < Ct ? minor : major), ct = (int)(Rt < Ct ? major : minor);
    const unsigned run = upper - (unsigned)party * runs;
    const int k0 = (int)fd_div(run * (unsigned)Kb, fdiv{runs_m, runs_s}), k1 = (int)fd_div((run + 1) * (unsigned)Kb, fdiv{runs_m, runs_s});

    const bool row_block = wave < 2;   // this wave copies one of these (else a column block)
    wave_src src = {nullptr, 0, 0};
    if (row_block || !IMPLICIT) {
        const int count = row_block ? Rb : Cb, block = row_block ? rt * 2 + wave : ct * 2 + wave - 2;
        src.p = (row_block ? A : B) + ((size_t)party * count + min(block, count - 1)) * Kb * TILE + lane;
    } else {
        src = column_source<IMPLICIT>(g, party, ct * 2 + wave - 2, lane);
    }
    v4i *mine = lds + wave * TILE;
    auto copy = [&](int kb) {
        unsigned qs = 64;
        const v4i *p = row_block || !IMPLICIT ? src.p + (size_t)kb * TILE : column_base<IMPLICIT>(g, src, kb, lane, qs);
#pragma unroll
        for (int i = 0; i < NL; i++) __builtin_amdgcn_global_load_lds(p + (size_t)i * qs, mine + i * 64, 16, 0, 0);
    };
    copy(k0);
    const int rb = rt * 2 + wr, cb = ct * 2 + wc;
    const bool inside = rb < Rb && cb < Cb;
    v4i acc[ND];
#pragma unroll
    for (int s = 0; s < ND; s++) acc[s] = (v4i){0, 0, 0, 0};
    const v4i *sa = lds + wr * TILE + lane, *sb = lds + (2 + wc) * TILE + lane;
    for (int kb = k0; kb < k1; kb++) {
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's block is in LDS
        __syncthreads();                      // everyone's is
        v4i a[NL], b[NL];
#pragma unroll
        for (int i = 0; i < NL; i++) {
            a[i] = sa[i * 64];
            b[i] = sb[i * 64];
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): they are in registers
        __syncthreads();                      // everyone's are: the blocks may be replaced
        if (kb + 1 < k1) copy(kb + 1);
        if (inside) {
#pragma unroll
            for (int i = 0; i < NL; i++)
#pragma unroll
                for (int j = 0; j < NL; j++)
                    acc[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[i + j], 0, 0, 0);
        }
    }
    if (!inside) return;
    // lane holds column lane%16 and rows 4*(lane/16)+r of its tile
    const int row = rb * 16 + 4 * (lane >> 4), col = cb * 16 + (lane & 15);
    if (col >= g.cols) return;
    const u32 cq = fd_div((u32)col, g.dCdiv);
    u64 *out = plane_at(g, run) + (size_t)party * g.out_party_stride + (size_t)cq * g.stride_cb + ((u32)col - cq * (u32)g.cdiv) +
               (size_t)row * g.stride_row;
#pragma unroll
    for (int r = 0; r < 4; r++)
        if (row + r < g.rows) out[(size_t)r * g.stride_row] = fold_diagonals(acc, r);
}

// The same contraction for a first operand of at most 16 rows and a large second one (dense layers at a small batch).
// There the time goes into reading the second operand once, so a launch is as
// fast as it keeps bytes in flight: a workgroup's tile is 16 rows x 128 columns, one row block and eight
// column blocks per unit, twice the column blocks of the square tile in the same LDS, and no MFMA is spent on
// row blocks that do not exist.  Wave w copies column block w and limb slice w of the row block, and owns
// the 16 x 16 outputs of column block w.  Units, ranges, planes and fold are those of the kernel above.
// (Four units of half the width in the same LDS, three on their way: 0.81 to 0.98 of the rate, n = 5.)
// STREAM: the second operand is read past the caches, see streams_operand.
template <bool STREAM>
__global__ __launch_bounds__(512) void gemm_skinny_kernel(gemm_args g)
{
    extern __shared__ v4i lds[];   // 2 stages x (1 row block + 8 column blocks) x TILE
    constexpr int STAGE = 9 * TILE;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned G = gridDim.x;
    const unsigned slot = xcd_slot(blockIdx.x, G);
    unsigned u0, u1;
    if (g.units) {
        u0 = unit_at(g, range_bound(g, slot));
        u1 = unit_at(g, range_bound(g, slot + 1));
    } else {
        u0 = 0;
        u1 = (unsigned)g.Kb;
    }
    if (u0 >= u1) return;
    const int zero_cut = g.slots > 1 ? zero_planes_of_cut_tile(g, u1, slot, G) : 0;

    // this wave's column block of tile t (clamped past the edge: computed, never stored) and its limb slice
    // of the party's row block
    auto b_source = [&](unsigned t) {
        const unsigned party = fd_div(t, g.dCT), ct = t - party * (unsigned)g.CT;
        return g.B + (size_t)party * g.b_party_stride + (size_t)min((int)ct * 8 + wave, g.Cb - 1) * g.Kb * TILE + lane;
    };
    auto a_source = [&](unsigned t) {
        const unsigned party = fd_div(t, g.dCT);
        return g.A + (size_t)party * g.a_party_stride + min(wave, NL - 1) * 64 + lane;
    };
    auto copy_unit = [&](const v4i *as, const v4i *bs, int k, int stage) {
        v4i *dst = lds + stage * STAGE;
#pragma unroll
        for (int q = 0; q < NL; q++)
            __builtin_amdgcn_global_load_lds(bs + (size_t)k * TILE + q * 64, dst + (1 + wave) * TILE + q * 64, 16, 0, STREAM ? 2 : 0);   // 2: nt
        if (wave < NL) __builtin_amdgcn_global_load_lds(as + (size_t)k * TILE, dst + wave * 64, 16, 0, 0);
    };

    unsigned tile = g.units ? fd_div(u0, g.dKb) : slot;
    int kb = (int)(u0 - (g.units ? tile * (unsigned)g.Kb : 0));
    const v4i *as = a_source(tile), *bs = b_source(tile);
    copy_unit(as, bs, kb, 0);
    int st = 0;

    unsigned u = u0;
    while (u < u1) {
        const int party = (int)fd_div(tile, g.dCT), ct = (int)(tile - (unsigned)party * (unsigned)g.CT);
        const bool inside = ct * 8 + wave < g.Cb;   // this wave's column block lies inside the matrix
        const int kb_first = kb;
        v4i acc[ND];
#pragma unroll
        for (int s = 0; s < ND; s++) acc[s] = (v4i){0, 0, 0, 0};

        const int kb_end = min(g.Kb, kb + (int)(u1 - u));
        const v4i *next_as = as, *next_bs = bs;
        for (; kb < kb_end; kb++, u++) {
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's part of the unit is in LDS
            __syncthreads();                      // everyone's part is; stage st^1 is no longer read
            if (u + 1 < u1) {
                int nkb = kb + 1;
                if (nkb == g.Kb) {
                    nkb = 0;
                    next_as = a_source(tile + 1);
                    next_bs = b_source(tile + 1);
                }
                copy_unit(next_as, next_bs, nkb, st ^ 1);
            }
            if (inside) {
                const v4i *sa = lds + st * STAGE + lane, *sb = lds + st * STAGE + (1 + wave) * TILE + lane;
                v4i a[NL], b[NL];
#pragma unroll
                for (int i = 0; i < NL; i++) {
                    a[i] = sa[i * 64];
                    b[i] = sb[i * 64];
                }
#pragma unroll
                for (int i = 0; i < NL; i++)
#pragma unroll
                    for (int j = 0; j < NL; j++)
                        acc[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[i + j], 0, 0, 0);
            }
            st ^= 1;
        }

        // lane holds column lane%16 of its block and rows 4*(lane/16)+r
        const int lrow = 4 * (lane >> 4), col = ct * SKINNY_COLS + wave * 16 + (lane & 15);
        const u32 cq = fd_div((u32)col, g.dCdiv);
        const size_t opos = (size_t)party * g.out_party_stride + (size_t)cq * g.stride_cb + ((u32)col - cq * (u32)g.cdiv);
        const unsigned plane = g.slots > 1 ? slot % (unsigned)g.slots : 0;
        u64 *outp = plane_at(g, plane);
#pragma unroll
        for (int r = 0; r < 4; r++)
            if (inside && lrow + r < g.rows && col < g.cols)
                outp[opos + (size_t)(lrow + r) * g.stride_row] = fold_diagonals(acc, r);
        const int nzero = (g.slots > 1 && kb_first == 0) ? (kb_end == g.Kb ? g.slots - 1 : zero_cut) : 0;
        for (int z = 0; z < nzero; z++) {
            unsigned zpl = plane + (unsigned)(g.slots - nzero + z);
            if (zpl >= (unsigned)g.slots) zpl -= (unsigned)g.slots;
            u64 *zp = plane_at(g, zpl);
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (inside && lrow + r < g.rows && col < g.cols) zp[opos + (size_t)(lrow + r) * g.stride_row] = 0;
        }
        if (kb == g.Kb) {
            kb = 0;
            tile++;
            as = next_as;
            bs = next_bs;
        }
    }
}

// The planes of a product added up into the first one, for callers that want it as a tensor: four planes requested at a time.
__device__ __forceinline__ void sum_planes(u64 *out, const u64 *part, size_t part_stride, int slots, size_t off)
{
    part += off;
    u64 v = out[off];
    int s = 1;
    for (; s + 3 < slots; s += 4, part += 4 * part_stride) {
        const u64 x0 = part[0], x1 = part[part_stride], x2 = part[2 * part_stride], x3 = part[3 * part_stride];
        v = ss_add(ss_add(v, x0), ss_add(ss_add(x1, x2), x3));
    }
    for (; s < slots; s++, part += part_stride) v = ss_add(v, *part);
    out[off] = v;
}

// Every tile has parts: one thread per element, in the order of memory, and no argument that has to be loaded (these few
// arrive in registers).  A tile per workgroup with the arguments of the product took longer, product and sum, us (rows x columns x
// contraction): n = 5 512 x 196 x 1024 35.1 -> 32.8, 256 x 784 x 512 34.9 -> 33.4; n = 3 249 x 648 x 1152 37.2 -> 34.9.
__global__ __launch_bounds__(256) void add_planes_kernel(u64 *out, const u64 *parts, size_t part_stride, size_t count, int slots)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) sum_planes(out, parts, part_stride, slots, i);
}

// Only the tiles of 64 x 64 from first_tile on have parts: one thread per element, 256 of a tile per workgroup.
__global__ __launch_bounds__(256) void add_cut_tiles_kernel(gemm_args g, unsigned first_tile)
{
    int ct, rt, party;
    tile_coords(g, first_tile + blockIdx.x, ct, rt, party);
    const int i = blockIdx.y * 256 + threadIdx.x, row = rt * 64 + (i >> 6), col = ct * 64 + (i & 63);
    if (row >= g.rows || col >= g.cols) return;
    const u32 cq = fd_div((u32)col, g.dCdiv);
    sum_planes(g.out, g.parts, g.part_stride, g.slots, (size_t)party * g.out_party_stride + (size_t)cq * g.stride_cb +
                                                           ((u32)col - cq * (u32)g.cdiv) + (size_t)row * g.stride_row);
}

}  // namespace

ss_part_src ss_gemm_parts(const product_plan &r, int n, int rows, int cols, int hw)
{
    ss_part_src ps = {};
    ps.planes = r.planes();
    ps.stride = (size_t)n * rows * cols;
    ps.first_cut = r.sq.runs ? 0 : r.p.whole;
    ps.party_tiles = (unsigned)r.p.RT * (unsigned)r.p.CT;
    ps.row_tiles = (unsigned)r.p.CT;
    ps.hw = (unsigned)hw;
    ps.rows = (unsigned)rows;
    ps.dHw = make_fdiv(ps.hw);
    ps.dRows = make_fdiv(ps.rows);
    return ps;
}

int ss_gemm_planes(int n, int rows, int cols, int K, int gather)
{
    const product_plan r = plan_product(n, rows, cols, K, gather, false, SQUARE_RUNS);
    return r.planes() > r.p.slots ? r.planes() : r.p.slots;
}

size_t ss_gemm_scratch_bytes(int n, int rows, int cols, int K, int gather)
{
    // room for either form of the second operand (tiles may take the 16-row kernel, limb planes never do)
    const int a = plan_gemm(n, rows, cols, K, gather).slots, b = gather ? plan_gemm(n, rows, cols, K, 0).slots : a;
    return (size_t)((a > b ? a : b) - 1) * n * rows * cols * sizeof(u64);   // the first plane is the product itself
}

size_t ss_packed_bytes(int rows, int K)
{
    return (size_t)((rows + 15) / 16) * (size_t)((K + 63) / 64) * (TILE * 16);
}

hipError_t ss_launch_pack_matrix(const u64 *src, void *dst, int n, int rows, int K, size_t party_stride,
                                 size_t stride_r, size_t stride_k, int taps, hipStream_t stream)
{
    const int Rb = (rows + 15) / 16, Kb = (K + 63) / 64;
    if (!fits_grid((long)Rb * Kb, 256)) return hipErrorInvalidConfiguration;   // (103 GB and more of tiles per party)
    hipLaunchKernelGGL(pack_matrix_kernel, dim3((unsigned)Rb * (unsigned)Kb, n), dim3(256), 0, stream, src, (v4i *)dst, rows, K, Rb,
                       Kb, make_fdiv((u32)Rb), make_fdiv((u32)Kb), stride_k == 1, party_stride, stride_r, stride_k,
                       ss_packed_bytes(rows, K) / 16, taps, taps && K / taps % 64 == 0 ? K / taps / 64 : 0, make_fdiv(taps ? (u32)taps : 1));
    return hipGetLastError();
}

hipError_t ss_launch_pack_operands(const u64 *x, void *packedX, const u64 *w, void *packedW, int n, int M, int K, int N, hipStream_t stream)
{
    const int Kb = (K + 63) / 64;
    const long xblocks = (long)((M + 15) / 16) * Kb, wblocks = (long)((N + 15) / 16) * Kb;
    if (!fits_grid(xblocks + wblocks, 256)) {
        const hipError_t e = ss_launch_pack_matrix(w, packedW, n, N, K, (size_t)K * N, 1, (size_t)N, 0, stream);
        return e == hipSuccess ? ss_launch_pack_matrix(x, packedX, n, M, K, (size_t)M * K, (size_t)K, 1, 0, stream) : e;
    }
    const pack_job a = {x, (v4i *)packedX, M, (M + 15) / 16, (int)xblocks, make_fdiv((u32)Kb), (size_t)M * K, (size_t)K, 1, ss_packed_bytes(M, K) / 16};
    const int Nb = (N + 15) / 16;
    const pack_job b = {w, (v4i *)packedW, N, Nb, (int)wblocks, make_fdiv((u32)Nb), (size_t)K * N, 1, (size_t)N, ss_packed_bytes(N, K) / 16};
    hipLaunchKernelGGL(pack_pair_kernel, dim3((unsigned)(xblocks + wblocks), n), dim3(256), 0, stream, a, b, K, Kb);
    return hipGetLastError();
}

hipError_t ss_launch_share_pack(const u64 *secret, u64 *shares, void *dst, int n, int t, int B, int K, int HW,
                                const ss_keys &keys, hipStream_t stream)
{
    const int rows = B * HW, Rb = (rows + 15) / 16, Kb = (K + 63) / 64;
    const dim3 grid(Rb, Kb * 4), block(256);
    const size_t stride = ss_packed_bytes(rows, K) / 16;
#define SS_SHARE_PACK(NC, TC) \
    hipLaunchKernelGGL((share_pack_kernel<NC, TC>), grid, block, 0, stream, secret, shares, (v4i *)dst, B, K, HW, Kb, stride, n, t, keys)
    if (n == 5 && t == 2)
        SS_SHARE_PACK(5, 2);
    else if (n == 3 && t == 1)
        SS_SHARE_PACK(3, 1);
    else
        SS_SHARE_PACK(0, 0);
#undef SS_SHARE_PACK
    return hipGetLastError();
}

hipError_t ss_launch_planes(const u64 *in, u64 *shares, void *planes, int n, int t, int B, int C, int HW, bool gen,
                            const ss_keys &keys, hipStream_t stream)
{
    // one element per thread fills the chip for the small tensors of a batch-1 network; from about half a
    // million elements on, four per thread move the data with fewer instructions
    const bool big = (size_t)B * HW * C >= ((size_t)1 << 19);
    const dim3 grid((B * HW + 15) / 16, big ? C / 64 : C / 16), block(256);
    const size_t party_bytes = ss_planes_bytes(B, C, HW, 1);
#define SS_PLANES(NC, TC, G)                                                                                        \
    do {                                                                                                            \
        if (big)                                                                                                    \
            hipLaunchKernelGGL((planes4_kernel<NC, TC, G>), grid, block, 0, stream, in, shares, (signed char *)planes, B, \
                               C, HW, party_bytes, n, t, keys);                                                     \
        else                                                                                                        \
            hipLaunchKernelGGL((planes_kernel<NC, TC, G>), grid, block, 0, stream, in, shares, (signed char *)planes, B,  \
                               C, HW, party_bytes, n, t, keys);                                                     \
    } while (0)
    if (!gen)
        SS_PLANES(0, 0, false);
    else if (n == 5 && t == 2)
        SS_PLANES(5, 2, true);
    else if (n == 3 && t == 1)
        SS_PLANES(3, 1, true);
    else
        SS_PLANES(0, 0, true);
#undef SS_PLANES
    return hipGetLastError();
}

hipError_t ss_launch_pack_im2col(const u64 *x, void *dst, int n, int B, int C, int H, int W, int kh, int kw,
                                 int stride, int pad, int Ho, int Wo, hipStream_t stream)
{
    const int M = B * Ho * Wo, K = C * kh * kw;
    const int Rb = (M + 15) / 16, Kb = (K + 63) / 64;
    im2col_args g;
    g.H = H, g.W = W, g.kh = kh, g.kw = kw, g.stride = stride, g.pad = pad, g.M = M, g.K = K, g.Kb = Kb;
    g.dTaps = make_fdiv((u32)(kh * kw)), g.dKw = make_fdiv((u32)kw), g.dWo = make_fdiv((u32)Wo), g.dHoWo = make_fdiv((u32)(Ho * Wo));
    g.HoWo = Ho * Wo, g.Wo = Wo;
    g.image = (size_t)C * H * W, g.party = B * g.image;
    hipLaunchKernelGGL(pack_im2col_kernel, dim3(Rb, Kb, n), dim3(256), 0, stream, x, (v4i *)dst, g, ss_packed_bytes(M, K) / 16);
    return hipGetLastError();
}

namespace {

struct conv_planes {   // geometry of an operand given as limb planes or (elements) as field elements
    const void *planes;
    int B, C, H, W, kh, kw, stride, pad, Ho, Wo;
    const u64 *elements;
};

hipError_t launch_gemm(const product_plan &plan, const void *packedA, const void *packedB, const u64 *rowsB, const conv_planes *cv, u64 *out,
                       u64 *parts, bool add_parts, int n, int rows, int cols, int K, size_t out_party_stride, size_t stride_row, int cdiv,
                       size_t stride_cb, hipStream_t stream, hipEvent_t started, hipEvent_t stopped)
{
    static bool lds_opt_in = false;
    constexpr int LDS_BYTES = 2 * 8 * TILE * 16, LDS_BYTES_SKINNY = 2 * 9 * TILE * 16;
    if (!lds_opt_in) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_limb_kernel<false>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)gemm_limb_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    LDS_BYTES);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)gemm_skinny_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    LDS_BYTES_SKINNY);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)gemm_skinny_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    LDS_BYTES_SKINNY);
        if (e != hipSuccess) return e;
        lds_opt_in = true;
    }
    const gemm_plan &p = plan.p;
    if (p.G <= 0) return hipErrorInvalidValue;
    gemm_args g = {};
    g.A = (const v4i *)packedA;
    g.B = (const v4i *)packedB;
    g.out = out;
    g.parts = parts;
    g.part_stride = (size_t)n * rows * cols;
    g.rows = rows;
    g.cols = cols;
    g.Rb = (rows + 15) / 16;
    g.Cb = (cols + 15) / 16;
    g.Kb = p.Kb;
    g.RT = p.RT;
    g.CT = p.CT;
    g.units = (unsigned)p.units;   // (gemm_ksplit_kernel: its tiles)
    g.whole = p.whole;
    g.cost0 = p.cost0;
    g.wlast = p.wlast;
    g.tcost = p.tcost;
    g.tlast = p.tlast;
    g.share = (p.cost - p.cost0) / (unsigned)p.G;
    g.rest = (p.cost - p.cost0) % (unsigned)p.G;
    g.slots = p.slots;
    auto fdz = [](unsigned long long d) { return make_fdiv(d >= 1 && d < (1ull << 32) ? (u32)d : 1u); };
    g.dG = fdz((unsigned)p.G);
    g.dKb = fdz((unsigned)g.Kb);
    g.dCT = fdz((unsigned)g.CT);
    g.dRT = fdz((unsigned)g.RT);
    g.dRowcost = fdz((unsigned long long)(g.CT - 1) * g.tcost + g.tlast);
    g.dTilecost = fdz(g.tcost);
    g.dWlast = fdz(g.wlast);
    g.dCdiv = fdz((unsigned)cdiv);
    g.a_party_stride = ss_packed_bytes(rows, K) / 16;
    g.b_party_stride = ss_packed_bytes(cols, K) / 16;
    g.out_party_stride = out_party_stride;
    g.stride_row = stride_row;
    g.stride_cb = stride_cb;
    g.cdiv = cdiv;
    g.K = K;
    g.raw = rowsB;
    g.raw_party = (size_t)cols * K;
    if (cv && cv->elements) {
        g.raw = cv->elements;
        g.raw_image = (size_t)cv->C * cv->H * cv->W;
        g.raw_party = cv->B * g.raw_image;
        g.cvTaps = cv->kh * cv->kw;
        g.dTaps = fdz((unsigned)g.cvTaps);
    }
    if (cv) {
        const size_t plane = (size_t)cv->B * cv->H * cv->W * cv->C;   // bytes
        g.planes = (const v4i *)cv->planes;
        g.plane16 = (unsigned)(plane / 16);
        g.party16 = (unsigned)(ss_planes_bytes(cv->B, cv->C, cv->H, cv->W) / 16);
        g.zero = g.planes + (size_t)NL * g.plane16;   // the pad behind the first party's planes
        g.cvH = cv->H, g.cvW = cv->W, g.cvPixels = cv->B * cv->H * cv->W, g.cvKw = cv->kw, g.cvStride = cv->stride, g.cvPad = cv->pad;
        g.cvHoWo = cv->Ho * cv->Wo, g.cvWo = cv->Wo, g.cvKbTap = cv->C / 64;
        g.dHoWo = fdz((unsigned)g.cvHoWo);
        g.dWo = fdz((unsigned)g.cvWo);
        g.dKbTap = fdz((unsigned)g.cvKbTap);   // (elements: not used)
        g.dKw = fdz((unsigned)g.cvKw);
    }
    // with an event pair the launch goes through the entry point that stamps the events with the kernel's own
    // start and end (profiling only)
#define SS_LAUNCH_PRODUCT_AS(KERNEL, GRID, THREADS, LDS, ...)                                                          \
    do {                                                                                                              \
        if (started && stopped)                                                                                       \
            hipExtLaunchKernelGGL(KERNEL, dim3((unsigned)(GRID)), dim3(THREADS), LDS, stream, started, stopped, 0, __VA_ARGS__); \
        else                                                                                                          \
            hipLaunchKernelGGL(KERNEL, dim3((unsigned)(GRID)), dim3(THREADS), LDS, stream, __VA_ARGS__);              \
    } while (0)
#define SS_LAUNCH_PRODUCT(KERNEL, LDS, ...) SS_LAUNCH_PRODUCT_AS(KERNEL, p.G, p.threads, LDS, __VA_ARGS__)
#define SS_LAUNCH_KSPLIT(KS)                                                                                          \
    SS_LAUNCH_PRODUCT((g.raw ? cv ? gemm_ksplit_kernel<IN_IMAGES, KS> : gemm_ksplit_kernel<IN_ROWS, KS>                 \
                       : cv  ? gemm_ksplit_kernel<IN_PLANES, KS> : gemm_ksplit_kernel<IN_TILES, KS>),                   \
                      0, g, make_fdiv((u32)p.slots))
    if (const int runs = plan.sq.runs) {
        const fdiv minors = make_fdiv(plan.sq.minors), majors = make_fdiv(plan.sq.majors), dRuns = make_fdiv((u32)runs);
        SS_LAUNCH_PRODUCT_AS((cv ? gemm_square_kernel<true> : gemm_square_kernel<false>), plan.sq.G, 256, 0, g.A, g.B,
                             (u32)g.Rb | (u32)g.Cb << 16, (u32)g.Kb | (u32)runs << 16, minors.m, minors.s, majors.m, majors.s, dRuns.m,
                             dRuns.s, plan.sq.G, g);
    } else switch (p.ksplit) {
        case 0:
            if (p.skinny)
                SS_LAUNCH_PRODUCT((streams_operand(n * ss_packed_bytes(cols, K)) ? gemm_skinny_kernel<true> : gemm_skinny_kernel<false>),
                                  LDS_BYTES_SKINNY, g);
            else
                SS_LAUNCH_PRODUCT((cv ? gemm_limb_kernel<true> : gemm_limb_kernel<false>), LDS_BYTES, g);
            break;
        case 1: SS_LAUNCH_KSPLIT(1); break;
        case 2: SS_LAUNCH_KSPLIT(2); break;
        case 4: SS_LAUNCH_KSPLIT(4); break;
        default: SS_LAUNCH_KSPLIT(8);
    }
#undef SS_LAUNCH_KSPLIT
#undef SS_LAUNCH_PRODUCT
#undef SS_LAUNCH_PRODUCT_AS
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !add_parts || plan.planes() == 1) return e;
    if (!plan.sq.runs && p.whole) {
        hipLaunchKernelGGL(add_cut_tiles_kernel, dim3((unsigned)p.tiles - p.whole, 16), dim3(256), 0, stream, g, p.whole);
        return hipGetLastError();
    }
    for (size_t first = 0; first < g.part_stride; first += (size_t)1 << 31) {   // one thread per element: see fits_grid
        const size_t count = g.part_stride - first < ((size_t)1 << 31) ? g.part_stride - first : (size_t)1 << 31;
        hipLaunchKernelGGL(add_planes_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, out + first,
                           parts + first, g.part_stride, count, plan.planes());
    }
    return hipGetLastError();
}

}  // namespace

size_t ss_planes_bytes(int B, int C, int H, int W)
{
    return (size_t)NL * B * H * W * C + 256;   // the limb planes and a pad that starts with 16 zero bytes
}

hipError_t ss_launch_gemm(const product_plan &plan, const void *packedA, const void *packedB, u64 *out, u64 *parts, bool add_parts, int n, int rows,
                          int cols, int K, size_t out_party_stride, size_t stride_row, int cdiv, size_t stride_cb,
                          hipStream_t stream, hipEvent_t started, hipEvent_t stopped)
{
    return launch_gemm(plan, packedA, packedB, nullptr, nullptr, out, parts, add_parts, n, rows, cols, K, out_party_stride, stride_row, cdiv,
                       stride_cb, stream, started, stopped);
}

hipError_t ss_launch_gemm_conv(const product_plan &plan, const void *packedW, const void *planes, u64 *out, u64 *parts, bool add_parts, int n, int B,
                               int C, int H, int W, int Co, int kh, int kw, int stride, int pad, int Ho, int Wo,
                               hipStream_t stream, hipEvent_t started, hipEvent_t stopped)
{
    const conv_planes cv = {planes, B, C, H, W, kh, kw, stride, pad, Ho, Wo, nullptr};
    const size_t HW = (size_t)Ho * Wo;
    // rows = output channel, cols = (b, ho, wo): y[b][co][hw]
    return launch_gemm(plan, packedW, nullptr, nullptr, &cv, out, parts, add_parts, n, Co, (int)(B * HW), C * kh * kw, (size_t)B * Co * HW, HW,
                       (int)HW, (size_t)Co * HW, stream, started, stopped);
}

hipError_t ss_launch_gemm_rows(const product_plan &plan, const u64 *x, const void *packedW, u64 *out, u64 *parts, int n, int M, int K, int N,
                               hipStream_t stream, hipEvent_t started, hipEvent_t stopped)
{
    // rows = output column, cols = row of x: y[col][row]
    return launch_gemm(plan, packedW, nullptr, x, nullptr, out, parts, true, n, N, M, K, (size_t)M * N, 1, 1, (size_t)N, stream, started,
                       stopped);
}

hipError_t ss_launch_gemm_images(const product_plan &plan, const void *packedW, const u64 *x, u64 *out, u64 *parts, int n, int B, int C, int H,
                                 int W, int Co, int kh, int kw, int stride, int pad, int Ho, int Wo, hipStream_t stream,
                                 hipEvent_t started, hipEvent_t stopped)
{
    const conv_planes cv = {nullptr, B, C, H, W, kh, kw, stride, pad, Ho, Wo, x};
    const size_t HW = (size_t)Ho * Wo;
    return launch_gemm(plan, packedW, nullptr, nullptr, &cv, out, parts, true, n, Co, (int)(B * HW), C * kh * kw, (size_t)B * Co * HW, HW,
                       (int)HW, (size_t)Co * HW, stream, started, stopped);
}

}  // namespace SS_NS
