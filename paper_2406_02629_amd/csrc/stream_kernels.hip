// Element-wise kernels: GEN (Eq. 1), REC (Eq. 2), reshare degree reduction with
// RERAND (Sec. IV-B, IV-C) and masked truncation (Sec. VI-B).
//
// One thread owns VEC consecutive elements and walks over all parties, so every
// plane is read and written with unit stride across a wave and the random
// coefficients of an element are drawn once, not once per party.
#include "kernels.hpp"
#include "eval.hpp"
#include "digits.hpp"
#include "pool_plan.hpp"

namespace SS_NS {

namespace {

constexpr int BLOCK = 256;
constexpr size_t LAUNCH_ELEMENTS = (size_t)1 << 31;   // of a tensor that goes in several launches, one thread each

// Block of elements that a workgroup of an element-wise kernel takes.  Where the planes of a tensor do not start on a cache
// line (starts_lines, which goes by the plane's size: a tensor whose first word is off a line counts by its planes alone) the blocks
// share lines, and workgroups are dealt round-robin to the 8 XCDs, so that neighbours write their parts of a line from two L2s.
// There 64 consecutive blocks go to one XCD (8 are as good for most, all of a plane's eighth is worse for the larger tensors):
// n = 7, t = 3 reduce + truncate of 640003 elements 123 -> 100 us with operands that change from call to call (300001: 45.0 -> 44.7,
// where only the same call repeated gains, 53 -> 48), sharing among three of 2^24 + 3 118 -> 95 us, reconstruction from two 88 -> 78 us.
// PER elements of a launch's `count` per workgroup; planes of `plane` elements.  (The grid is worked out from the count, which arrives
// in registers: read from the launch it puts a memory access in front of a small kernel's first load.)
__host__ __device__ __forceinline__ bool starts_lines(size_t count) { return count % 16 == 0; }
__host__ __device__ __forceinline__ bool starts_halves(size_t count) { return count % 8 == 0; }   // of cache lines
template <int PER>
__device__ __forceinline__ size_t element_block(size_t count, size_t plane)
{
    constexpr unsigned RUN = 64;
    const unsigned b = blockIdx.x, base = b / (8 * RUN) * (8 * RUN);
    if (starts_lines(plane) || (size_t)(base + 8 * RUN) * PER >= count + PER) return b;   // past the last whole 8 * RUN workgroups
    return base + (b % 8) * RUN + (b - base) / 8;
}

template <int VEC>
struct pack_t;
template <>
struct pack_t<1> {
    u64 v[1];
    __device__ __forceinline__ void load(const u64 *p) { v[0] = *p; }
    __device__ __forceinline__ void load_streaming(const u64 *p) { v[0] = __builtin_nontemporal_load(p); }
    __device__ __forceinline__ void store(u64 *p) const { *p = v[0]; }
    __device__ __forceinline__ void store_streaming(u64 *p) const { __builtin_nontemporal_store(v[0], p); }
    template <bool STREAM>
    __device__ __forceinline__ void send(u64 *p) const { STREAM ? store_streaming(p) : store(p); }
};
template <>
struct pack_t<2> {
    u64 v[2];
    __device__ __forceinline__ void load(const u64 *p)
    {
        const ulonglong2 q = *reinterpret_cast<const ulonglong2 *>(p);
        v[0] = q.x;
        v[1] = q.y;
    }
    __device__ __forceinline__ void load_streaming(const u64 *p)
    {
        typedef unsigned long long v2u __attribute__((ext_vector_type(2)));
        const v2u q = __builtin_nontemporal_load(reinterpret_cast<const v2u *>(p));
        v[0] = q.x;
        v[1] = q.y;
    }
    __device__ __forceinline__ void store(u64 *p) const
    {
        ulonglong2 q;
        q.x = v[0];
        q.y = v[1];
        *reinterpret_cast<ulonglong2 *>(p) = q;
    }
    // for output that nothing in the same launch reads again
    __device__ __forceinline__ void store_streaming(u64 *p) const
    {
        typedef unsigned long long v2u __attribute__((ext_vector_type(2)));
        v2u q = {v[0], v[1]};
        __builtin_nontemporal_store(q, reinterpret_cast<v2u *>(p));
    }
    template <bool STREAM>
    __device__ __forceinline__ void send(u64 *p) const { STREAM ? store_streaming(p) : store(p); }
};

// A message that nothing in the launch reads again.  STREAM: past the caches, see streams_messages.
template <bool STREAM>
__device__ __forceinline__ void send(u64 *p, u64 v)
{
    if constexpr (STREAM)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// First party whose share of element e has more than one plane of the incoming product: the tiles of the last parties are
// the ones dealt in parts (ss_part_src).
__device__ __forceinline__ int first_cut_party(const ss_part_src &ps, size_t e)
{
    if (ps.first_cut == 0) return 0;   // uniform
    const u32 q = fd_div((u32)e, ps.dHw), b = fd_div(q, ps.dRows), row = q - b * ps.rows, col = b * ps.hw + ((u32)e - q * ps.hw);
    const u32 tile = (row >> 6) * ps.row_tiles + (col >> 6);
    int i = 0;
    for (u32 t = tile; t < ps.first_cut; t += ps.party_tiles) i++;
    return i;
}

// the further planes of the first NR shares of element e, added to v[]: two planes requested at a time; LEAN: every tile has all
// planes, which come one by one.  (For three shares the last plane is a loop as well, though it runs once: written straight the kernels
// are slower on tensors too, reduce + truncate of 802816 elements, n = 4, 31.7 -> 34.1 us.  For five it makes no difference, for
// seven the loop spills eight more scalar registers: over the 45-bit prime 43565 elements, n = 7, 11.6 -> 11.9 us.)
template <int NR, bool LEAN = false>
__device__ __forceinline__ void add_planes(u64 (&v)[NR], const u64 *c, size_t count, size_t e, const ss_part_src &ps)
{
    c += e;
    if (LEAN || ps.first_cut == 0) {   // uniform: every tile has all planes
        int s = 1;
        for (; !LEAN && s + 1 < ps.planes; s += 2) {
            u64 x[NR], y[NR];
#pragma unroll
            for (int i = 0; i < NR; i++) {
                x[i] = c[(size_t)s * ps.stride + (size_t)i * count];
                y[i] = c[(size_t)(s + 1) * ps.stride + (size_t)i * count];
            }
#pragma unroll
            for (int i = 0; i < NR; i++) v[i] = ss_add(v[i], ss_add(x[i], y[i]));
        }
        for (; s < ps.planes; s++) {
            u64 x[NR];
#pragma unroll
            for (int i = 0; i < NR; i++) x[i] = c[(size_t)s * ps.stride + (size_t)i * count];
#pragma unroll
            for (int i = 0; i < NR; i++) v[i] = ss_add(v[i], x[i]);
            if (!LEAN && NR > 3) break;
        }
        return;
    }
    const int cut = first_cut_party(ps, e);
    if (cut >= NR) return;
    for (int s = 1; s < ps.planes; s++) {
        u64 x[NR];
#pragma unroll
        for (int i = 0; i < NR; i++) x[i] = i >= cut ? c[(size_t)s * ps.stride + (size_t)i * count] : 0;
#pragma unroll
        for (int i = 0; i < NR; i++) v[i] = ss_add(v[i], x[i]);
    }
}

// v, share i of element e in the first plane, and what the further planes hold of it: two planes requested at a time
__device__ __forceinline__ u64 add_planes_of(u64 v, const u64 *c, int i, size_t count, size_t e, const ss_part_src &ps, int first_cut)
{
    if (i < first_cut) return v;
    const u64 *q = c + (size_t)i * count + e + ps.stride;
    int s = 1;
    for (; s + 1 < ps.planes; s += 2, q += 2 * ps.stride) {
        const u64 x = q[0], y = q[ps.stride];
        v = ss_add(v, ss_add(x, y));
    }
    return s < ps.planes ? ss_add(v, *q) : v;
}

template <int MAXD>
__device__ __forceinline__ void draw_coeffs(u64 (&c)[MAXD], const u64 *keys, int d, u64 e)
{
    const u64 counter = ss_counter(e);
#pragma unroll
    for (int j = 0; j < MAXD; j++) c[j] = (j < d) ? ss_draw_field_at(keys[j], counter) : 0;
}

// ------------------------------------------------------------------ GEN
// NC, DC > 0 fix the party count and the degree at compile time (the schemes
// the paper evaluates: (k,n) = (2,3) and (3,5)), so that the evaluation points
// become immediates; 0 means "take the run-time value".
// Bound by the writes of its n planes.  Five of them leave a wave at a time: workgroups of one wave write 5 % faster
// than those of four, and so does the longer reduction (PACED) against the short one (n = 5, 2^28 elements: 2.15 ms
// against 2.32 ms with four waves and 2.40 ms with the short reduction too; 2^26: 514, 548 and 570 us; 2^20: 7.6, 8.4
// and 8.5 us).  With three planes four waves are the better ones (2^24 elements: 75.6 against 76.5 us), and the form of
// the reduction makes no difference beyond that of two runs (long and short, 2^20: 6.3 and 6.2, 2^24: 75.5 and 75.4, 2^26:
// 362 and 366, 2^28: 1444 and 1453 us).  Five planes that do not start on halves of cache lines go through the caches, which put the
// parts of a line together (2^24 + 3 elements 185 -> 148 us, 2^22 + 2 40 -> 37 us; on halves past them and in the order of the
// launch: 438888 elements 5.5 -> 4.7 us, 5.8 M 43.5 -> 41.1; three planes 95 and 92, 21 and 25 us: past them).  That choice, a branch
// before each of the five stores, also keeps them where their plane is ready; without it the compiler gathers four at the end, and planes
// on the lines are written slower (2^28 elements 2160 -> 2076 us, 2^25 271 -> 260, 2^24 equal).
// Odd counts, one element per thread, have the schemes fixed too (2^20-odd elements, n = 3: 11 -> 7 us).
template <int VEC, int NC>
constexpr int SHARE_BLOCK = VEC == 2 && NC == 5 ? 64 : BLOCK;
template <int VEC, int NC, int DC>
__global__ __launch_bounds__((SHARE_BLOCK<VEC, NC>)) void share_kernel(const u64 *__restrict__ secret, u64 *__restrict__ shares,
                                                      size_t count, int n_rt, int degree_rt, ss_keys keys)
{
    constexpr int MAXD = DC ? DC : SS_MAXDEG;
    constexpr int MAXP = NC ? NC : SS_MAXN;
    const int n = NC ? NC : n_rt, degree = DC ? DC : degree_rt;
    const size_t e0 = (element_block<SHARE_BLOCK<VEC, NC> * VEC>(count, starts_halves(count) ? 0 : count) * SHARE_BLOCK<VEC, NC> +
                       threadIdx.x) * VEC;
    if (e0 >= count) return;
    pack_t<VEC> a0;
    a0.load(secret + e0);
    u64 c[VEC][MAXD];
#pragma unroll
    for (int u = 0; u < VEC; u++) draw_coeffs<MAXD>(c[u], keys.k, degree, e0 + u);
    if constexpr (NC != 0 && (DC == 1 || DC == 2)) {
        // consecutive party IDs: forward differences, two additions per point instead of Horner's multiplications
        pack_t<VEC> s[NC];
#pragma unroll
        for (int u = 0; u < VEC; u++) eval_points<DC, NC, true>(a0.v[u], c[u], [&](int p, u64 v) { s[p].v[u] = v; });
#pragma unroll
        for (int p = 0; p < NC; p++) {   // written, not read again
            u64 *to = shares + (size_t)p * count + e0;
            NC == 5 && !starts_halves(count) ? s[p].store(to) : s[p].store_streaming(to);
        }
    } else {
#pragma unroll
        for (int i = 1; i <= MAXP; i++) {
            if (i <= n) {
                pack_t<VEC> s;
#pragma unroll
                for (int u = 0; u < VEC; u++) s.v[u] = ss_poly_eval<MAXD>(a0.v[u], c[u], degree, i);
                s.store_streaming(shares + (size_t)(i - 1) * count + e0);
            }
        }
    }
}

// ------------------------------------------------------------------ REC
// Bound by reading m planes.  STREAM (streams_messages): shares and secret go past the caches, which hold neither for a
// later reader at such sizes: m = 3, 2^28 elements 1.37 -> 1.30 ms (6.6 TB/s), 2^26 349 -> 330 us; m = 2, 2^24 elements
// 67.8 -> 63.5 us.  Requesting all planes before the first sum is slower (2^28: 1.44 to 1.48 ms).
template <int VEC, bool STREAM>
__global__ __launch_bounds__(BLOCK) void reconstruct_kernel(const u64 *__restrict__ shares,
                                                            u64 *__restrict__ secret, size_t count,
                                                            ss_rec_params rp)
{
    const size_t e0 = (element_block<BLOCK * VEC>(count, count) * BLOCK + threadIdx.x) * VEC;
    if (e0 >= count) return;
    pack_t<VEC> out;
    ss_sacc acc[VEC];
#pragma unroll
    for (int u = 0; u < VEC; u++) acc[u].clear();
#pragma unroll
    for (int i = 0; i < SS_MAXN; i++) {
        if (i < rp.m) {
            pack_t<VEC> s;
            const u64 *from = shares + (size_t)rp.plane[i] * count + e0;
            STREAM ? s.load_streaming(from) : s.load(from);
#pragma unroll
            for (int u = 0; u < VEC; u++) acc[u].mac(s.v[u], rp.ilambda[i]);
        }
    }
#pragma unroll
    for (int u = 0; u < VEC; u++) out.v[u] = rp.dinv == 1 ? acc[u].value() : ss_mul(acc[u].value(), rp.dinv);
    out.template send<STREAM>(secret + e0);
}

// e of the truncation mask alpha = e * 2^f: uniform in [1, 2^(32-f)]
__device__ __forceinline__ u64 mask_e(u64 key, u64 e, int f)
{
    return 1 + ((ss_draw(key, e) >> 3) & ((1ULL << (32 - f)) - 1));
}

// the same before a division by kh*kw: the sample space of e shrinks to [1, floor(2^(32-f) / kdiv)], which keeps
// alpha = e * 2^f * kdiv within (0, 2^32] (Sec. VII-B); range = 2^(32-f) gives mask_e
__device__ __forceinline__ u64 mask_e_below(u64 key, u64 e, unsigned range)
{
    return 1 + (ss_draw(key, e) >> 3) % range;
}

// what the elite party does with the reconstructed x + alpha: floor division of the signed value by 2^f
__device__ __forceinline__ u64 shift_signed(u64 v, int f)
{
    const int64_t sv = (v <= (SS_P - 1) / 2) ? (int64_t)v : (int64_t)v - (int64_t)SS_P;
    const int64_t qv = sv >> f;
    return qv >= 0 ? (u64)qv : SS_P - (u64)(-qv);
}

// The same followed by the rounding division that average pooling moves into the truncation (Sec. VI-C):
// [q / kdiv] = floor((q + floor(kdiv/2)) / kdiv) on the signed quotient q, so that a remainder of
// ceil(kdiv/2) or more goes up (the worst case of App. C) and [(q + e*kdiv) / kdiv] = [q / kdiv] + e.
__device__ __forceinline__ u64 shift_round_div(u64 v, int f, int kdiv)
{
    const int64_t sv = (v <= (SS_P - 1) / 2) ? (int64_t)v : (int64_t)v - (int64_t)SS_P;
    const int64_t a = (sv >> f) + kdiv / 2;
    const u64 d = (u64)kdiv;
    return a >= 0 ? (u64)a / d : SS_P - ((u64)(-a) + d - 1) / d;
}

// ------------------------------------------------------------------ RED + RERAND, truncation
// The protocol steps for the element a thread owns.  All parties are simulated by that one thread, so a message is
// written to the workspace (the "send") and what follows from it is computed in registers (the "receive"); messages and
// results are exactly those of the per-party steps:
//   RED   1. party i = 1..2t+1: sub-shares of c_i for parties q = 1..k                   -> msg1[i][q]
//         2. party q: received row vector times R, in factored form R = B^-1[:, :k] * V (V[j][m] = m^j): first the
//            k low coefficients of the polynomial through the received values, then its value at every party ID
//            -- same residues as the (2t+1) x n product                                  -> msg2[q][m]
//         3. party m: REC of the k received values, plus its share of zero (RERAND)
//   trunc 1. parties q = 1..k add their share of alpha = e * 2^f (e * 2^f * kdiv with the rounding division) -> umsg[q]
//         2. the elite party reconstructs x + alpha, divides by 2^f with floor on the signed value (then by kdiv with
//            rounding) and shares the quotient                                           -> wsh[m]
//         3. every party m adds its share of alpha~ = -e
// At the sizes of a network's layers this code is bound by its instructions (all of them issue at the same rate on
// this machine, 64-bit multiply-adds included), so it carries the polynomials behind the messages along and works on
// coefficients where the protocol works on values:
//  * a party evaluates its polynomial at the consecutive points 1, 2, ... by forward differences (eval_points);
//  * what the parties reconstruct in step 3 of RED is the combination of the k polynomials of step 2 with the Lagrange
//    multipliers, so the coefficients are combined, not their values at every ID; the sharings of zero and of the mask
//    are added coefficient by coefficient too, and the sum is evaluated once;
//  * REC of a sharing whose polynomial is at hand is its constant term, whichever IDs are asked for;
//  * sums of value * small signed constant keep the value in two pieces of 31 and 30 bits and accumulate in signed
//    64-bit words (one multiply-add per piece), with no case split on the sign of the constant;
//  * sums stay unreduced (any word of the right residue within the bounds noted) until a value is stored.
// n = 5, t = 2, reduce + truncate + open on MI355X: 24.0 -> 15.4 us at 200 K elements, where writing the same words
// without any arithmetic takes 13.9 us.
// n = 7, t = 3: 50.4 -> 27.1 us; n = 4, t = 1: 18.9 -> 10.1 us (against values at every ID and loops over n and t).
// N: parties fixed at compile time, or 0 for the run-time value n; T: degree.

// sum of v * c over at most 8 terms, v canonical given as v = w0 + w1 2^31 (w0 < 2^31), |c| < 2^26
struct ss_sacc2 {
    long long lo, hi;
    __device__ __forceinline__ void clear() { lo = 0; hi = 0; }
    __device__ __forceinline__ void mac(u32 w0, u32 w1, int c)
    {
        lo += (long long)(int)w0 * c;   // |sum| < 8 * 2^31 * 2^26 = 2^60
        hi += (long long)(int)w1 * c;
    }
    // the sum, below 2^61 + 2^3 (2^45 + 2^25)
    __device__ __forceinline__ u64 lazy() const
    {
#if defined(SS_FIELD_P45)
        // here |hi| < 2^43 (w1 < 2^14).  Offsets that are multiples of p make both words positive;
        // h 2^31 with h = a 2^14 + b: a 2^45 + b 2^31 = 55 a + b 2^31
        const u64 l = (u64)(lo + (long long)(SS_P << 16)), h = (u64)(hi + (long long)SS_P);   // < 2^62, < 2^46
        return ss_fold(l + SS_PC * (h >> 14) + ((h & 0x3FFFull) << 31));
#else
        const u64 l = (u64)(lo + (long long)SS_P), h = (u64)(hi + (long long)SS_P);   // in (2^60, 2^62)
        // h 2^31 with 2^61 = 1: low 30 bits of h shifted, the rest wraps to weight 1
        return ss_fold(l + ((h & 0x3FFFFFFFull) << 31) + (h >> 30));
#endif
    }
    __device__ __forceinline__ u64 value() const { return ss_canon(lazy()); }
};
#define SS_SPLIT31(v, w0, w1) const u32 w0 = (u32)(v)&0x7FFFFFFFu, w1 = (u32)((v) >> 31)


template <int N>
constexpr int MAXP = N ? N : SS_MAXN;

template <int T>
__device__ __forceinline__ u64 mask_of(const ss_tr_params &tp, size_t e, u64 &alpha)
{
    const u64 ev = tp.kdiv > 1 ? mask_e_below(tp.e_key, e, tp.e_range) : mask_e(tp.e_key, e, tp.f);
    alpha = tp.kdiv > 1 ? (ev * (u64)tp.kdiv) << tp.f : ev << tp.f;   // <= 2^32
    return ev;
}

// truncation steps 2 and 3 from the opened x + alpha (canonical): the new shares in o[], their secret in `secret`; the
// messages of step 2 go to wsh unless it is nullptr
template <int N, int T, bool STREAM>
__device__ __forceinline__ void shift_and_unmask(u64 opened, u64 ev, u64 counter, size_t em, size_t mcount,
                                                 u64 *__restrict__ wsh, const ss_tr_params &tp, int n, u64 (&o)[MAXP<N>],
                                                 u64 &secret)
{
    const u64 w = tp.kdiv > 1 ? shift_round_div(opened, tp.f, tp.kdiv) : shift_signed(opened, tp.f);
    u64 cw[T], co[T];
#pragma unroll
    for (int j = 0; j < T; j++) {
        cw[j] = ss_draw_lazy_at(tp.gen_key[j], counter);
        co[j] = ss_fold(cw[j] + ss_draw_lazy_at(tp.alphat_key[j], counter));
    }
    if (wsh) eval_points<T, MAXP<N>>(w, cw, [&](int m, u64 v) { send<STREAM>(wsh + (size_t)m * mcount + em, v); }, n);
    secret = ss_canon(w + SS_P - ev);
    eval_points<T, MAXP<N>>(secret, co, [&](int m, u64 v) { o[m] = v; }, n);
}

// RED + RERAND and, with TRUNC, truncation of element e: the new shares come back in o[], their secret (what any k of
// them reconstruct to) in `secret`
// (em, mcount: position and plane size of this element in the message buffers, which need not be e, count)
template <int N, int T, bool TRUNC, bool STREAM, bool LEAN>
__device__ __forceinline__ void reduce_truncate(size_t e, size_t count, size_t em, size_t mcount, const u64 *c,
                                                u64 *__restrict__ msg1, u64 *__restrict__ msg2, u64 *__restrict__ umsg,
                                                u64 *__restrict__ wsh, const ss_dr_params &dp, const ss_tr_params &tp,
                                                const ss_part_src &ps, u64 (&o)[MAXP<N>], u64 &secret)
{
    constexpr int K = T + 1, NR = 2 * T + 1;
    const int n = N ? N : dp.n;
    const u64 counter = ss_counter(e);

    // all incoming shares are requested at once
    u64 cin[NR];
#pragma unroll
    for (int i = 0; i < NR; i++) cin[i] = c[(size_t)i * count + e];
    // (t = 3 has no registers to spare: with the sum of planes out of its straight path the compiler spills elsewhere, n = 7 reduce +
    // truncate of 4629 elements 9.0 -> 8.6 us, over the 45-bit prime 10.2 -> 9.3)
    const bool several = ps.planes > 1;
    if (T == 3 ? __builtin_expect(several, 0) : several) add_planes<NR, LEAN>(cin, c, count, e, ps);

    // step 1, and of step 2 the sums coef[q][j] = sum_i msg1[i][q] * D binv[i][j] (j = 0: without D, see ilambda0)
    ss_sacc2 coef[K][K];
#pragma unroll
    for (int q = 0; q < K; q++)
#pragma unroll
        for (int j = 0; j < K; j++) coef[q][j].clear();
#pragma unroll
    for (int i = 0; i < NR; i++) {
        u64 r[T];
#pragma unroll
        for (int j = 0; j < T; j++) r[j] = ss_draw_lazy_at(dp.reshare_key[i][j], counter);
        eval_points<T, K>(cin[i], r, [&](int q, u64 v) {
            send<STREAM>(msg1 + ((size_t)i * K + q) * mcount + em, v);
            SS_SPLIT31(v, w0, w1);
            coef[q][0].mac(w0, w1, dp.ilambda0[i]);
#pragma unroll
            for (int j = 1; j < K; j++) coef[q][j].mac(w0, w1, dp.ibinv[i][j]);
        });
    }

    // rest of step 2: party q evaluates its polynomial at every party ID
    u64 poly[K][K];   // [coefficient][q], < 2^61 + 2^3
#pragma unroll
    for (int q = 0; q < K; q++) {
        u64 cf[T];
        poly[0][q] = coef[q][0].lazy();
#pragma unroll
        for (int j = 1; j < K; j++) cf[j - 1] = poly[j][q] = ss_fold(ss_mul_lazy(coef[q][j].lazy(), dp.dinv));
        eval_points<T, MAXP<N>>(poly[0][q], cf,
                                [&](int m, u64 v) { send<STREAM>(msg2 + ((size_t)q * n + m) * mcount + em, v); }, n);
    }
    // step 3: sum_q lambda_q poly[.][q], lambda = (2, -1), (3, -3, 1) or (4, -6, 4, -1), then RERAND and the mask of
    // truncation step 1
    u64 u[K], ev = 0, alpha = 0;
    if (TRUNC) ev = mask_of<T>(tp, e, alpha);
#pragma unroll
    for (int j = 0; j < K; j++) {
        auto minus = [](u64 a, u64 b) { return ss_fold(a + 2 * SS_P - b); };   // a, b and the result < 2^61 + 2^3
        const u64 d = minus(poly[j][0], poly[j][1]);
        u64 v;   // < 5 (2^61 + 2^3)
        if constexpr (T == 1)
            v = d + poly[j][0];
        else if constexpr (T == 2)
            v = 2 * d + d + poly[j][2];
        else
            v = poly[j][0] + 3 * minus(d, minus(poly[j][1], poly[j][2])) + minus(poly[j][2], poly[j][3]);
        if (j > 0) {
            v += ss_draw_lazy_at(dp.zero_key[j - 1], counter);
            if (TRUNC) v += ss_draw_lazy_at(tp.alpha_key[j - 1], counter);
        } else if (TRUNC) {
            v += alpha;
        }
        u[j] = ss_fold(v);
    }
    u64 uc[T];
#pragma unroll
    for (int j = 0; j < T; j++) uc[j] = u[j + 1];
    if constexpr (!TRUNC) {
        eval_points<T, MAXP<N>>(u[0], uc, [&](int m, u64 v) { o[m] = v; }, n);
        secret = ss_canon(u[0]);
    } else {
        // the masked shares of parties 1..k; the elite party's REC of x + alpha is the constant term
        eval_points<T, K>(u[0], uc, [&](int q, u64 v) { send<STREAM>(umsg + (size_t)q * mcount + em, v); });
        shift_and_unmask<N, T, STREAM>(ss_canon(u[0]), ev, counter, em, mcount, wsh, tp, n, o, secret);
    }
}

// Most elements of a reduction that asks for its arguments together (request_arguments): further on the time is the same, or longer by 2 %
// (n = 3, 200704 elements 8.1 -> 8.3, 802816 23.1 -> 23.6; n = 5, 802816 47.2 -> 47.5).  Reduction and truncation, back to back on operands
// that change, us: n = 3, 2000 elements 4.6 -> 4.1, 50176 4.35 -> 3.95; n = 5 5.1 -> 4.6 (5.05 where the host is slower), 6.9 -> 6.6, 120000
// 9.6 -> 9.2; n = 7 8.0 -> 7.7, 10.5 -> 9.9, 16.2 -> 15.5, 200704 25.9 -> 24.7, 400000 49.4 -> 49.4.
template <int T>
constexpr size_t REQUEST_MAX_COUNT = (size_t)1 << (T == 3 ? 18 : 17);

// One thread per element.  `count` stands among the arguments that arrive in registers: whether a launch is short enough to ask for the others together is
// known without a load.
// (t = 3: without the second bound the compiler takes 157 registers, three waves per SIMD, to no gain)
// LEAN: without the code for products of which only a part of the tiles is cut, see HAS_LEAN.
template <int N, int T, bool TRUNC, bool STREAM, bool LEAN>
__global__ __launch_bounds__(BLOCK, T == 3 ? 4 : 1) void degree_reduce_kernel(const u64 *c, u64 *__restrict__ msg1, u64 *__restrict__ msg2,
                                                              u64 *__restrict__ umsg, u64 *__restrict__ wsh, u64 *out,
                                                              size_t count, u64 *__restrict__ rec, ss_dr_params dp,
                                                              ss_tr_params tp, ss_part_src ps)
{
    if (count <= REQUEST_MAX_COUNT<T>) request_arguments<8 * 8 + sizeof(ss_dr_params) + sizeof(ss_tr_params) + sizeof(ss_part_src)>();
    const size_t e = element_block<BLOCK>(count, count) * BLOCK + threadIdx.x;
    if (e >= count) return;
    u64 o[MAXP<N>], secret;
    reduce_truncate<N, T, TRUNC, STREAM, LEAN>(e, count, e, count, c, msg1, msg2, umsg, wsh, dp, tp, ps, o, secret);
#pragma unroll
    for (int m = 0; m < MAXP<N>; m++)
        if (N != 0 || m < dp.n) out[(size_t)m * count + e] = o[m];
    if (TRUNC && rec) rec[e] = secret;   // if asked for, REC of the result
}

// RED + RERAND of small tensors with t = 3, where the serial work of one thread per element leaves most of the chip idle: a
// workgroup takes 32 elements and eight party lanes per element.  Lane p = 0..6 first plays reducing party p+1 (step 1)
// while lane 7 draws the sharing of zero; then, after these went through LDS, lane p plays receiving party p+1: it forms
// the four values that parties 1..4 would send it (step 2, with the full matrix R instead of its factors, so that the
// lanes do not wait on each other) and reconstructs from them (step 3).  Same messages and results.
// 4 K elements, n = 8: 7.0 us against 8.2 us of the kernel above.
__global__ __launch_bounds__(BLOCK) void degree_reduce_lanes_kernel(const u64 *c, u64 *__restrict__ msg1,
                                                                    u64 *__restrict__ msg2, u64 *out, size_t count,
                                                                    ss_dr_params dp, ss_part_src ps)
{
    constexpr int T = 3, K = T + 1, NR = 2 * T + 1;
    __shared__ u64 sub[NR][K][32];
    __shared__ u64 zero[T][32];
    const int el = threadIdx.x & 31, p = threadIdx.x >> 5;
    const size_t e = (size_t)blockIdx.x * 32 + el;
    const bool live = e < count;
    if (live && p < NR) {
        u64 ci = c[(size_t)p * count + e];
        if (ps.planes > 1) ci = add_planes_of(ci, c, p, count, e, ps, first_cut_party(ps, e));
        u64 r[T];
        draw_coeffs<T>(r, dp.reshare_key[p], T, e);
        eval_points<T, K>(ci, r, [&](int q, u64 v) {
            sub[p][q][el] = v;
            msg1[((size_t)p * K + q) * count + e] = v;
        });
    } else if (live) {
        u64 z[T];
        draw_coeffs<T>(z, dp.zero_key, T, e);
#pragma unroll
        for (int j = 0; j < T; j++) zero[j][el] = z[j];
    }
    __syncthreads();
    if (!live || p >= dp.n) return;
    ss_sacc red;
    red.clear();
#pragma unroll
    for (int q = 0; q < K; q++) {
        ss_sacc acc;
        acc.clear();
#pragma unroll
        for (int i = 0; i < NR; i++) acc.mac(sub[i][q][el], dp.irmat[i][p]);
        const u64 v = ss_mul(acc.value(), dp.dinv);
        msg2[((size_t)q * dp.n + p) * count + e] = v;
        red.mac(v, dp.ilambda[q]);
    }
    u64 z[T];
#pragma unroll
    for (int j = 0; j < T; j++) z[j] = zero[j][el];
    out[(size_t)p * count + e] = ss_add(red.value(), ss_poly_eval<T>(0, z, T, p + 1));
}

// truncation of given shares (parties 1..k are read) from element `first` on
template <int N, int T, bool STREAM>
__global__ __launch_bounds__(BLOCK) void truncate_kernel(const u64 *x, u64 *__restrict__ umsg, u64 *__restrict__ wsh,
                                                         u64 *out, size_t count, size_t first, ss_tr_params tp)
{
    const size_t e = first + element_block<BLOCK>(min(count - first, LAUNCH_ELEMENTS), count) * BLOCK + threadIdx.x;
    if (e >= count) return;
    constexpr int K = T + 1;
    const u64 counter = ss_counter(e);
    u64 xs[K];
#pragma unroll
    for (int q = 0; q < K; q++) xs[q] = x[(size_t)q * count + e];
    u64 alpha, ca[T];
    const u64 ev = mask_of<T>(tp, e, alpha);
#pragma unroll
    for (int j = 0; j < T; j++) ca[j] = ss_draw_lazy_at(tp.alpha_key[j], counter);
    ss_sacc2 acc;
    acc.clear();
    eval_points<T, K>(alpha, ca, [&](int q, u64 v) {
        const u64 um = ss_add(xs[q], v);
        send<STREAM>(umsg + (size_t)q * count + e, um);
        SS_SPLIT31(um, w0, w1);
        acc.mac(w0, w1, tp.ilambda[q]);
    });
    u64 o[MAXP<N>], secret;
    shift_and_unmask<N, T, STREAM>(acc.value(), ev, counter, e, count, wsh, tp, N ? N : tp.n, o, secret);
#pragma unroll
    for (int m = 0; m < MAXP<N>; m++)
        if (N != 0 || m < tp.n) out[(size_t)m * count + e] = o[m];
}

// ReLU under the multiplicative mask for one element (the three steps of relu_kernel below), n and t
// fixed: x[] the n shares, r[] the n output shares
template <int N, int T, bool STREAM>
__device__ __forceinline__ void relu_fixed(const u64 (&x)[N], size_t em, size_t mcount, const u64 (&b)[2 * T + 1],
                                           const u64 (&bi)[N], u64 *__restrict__ msg, u64 *__restrict__ yplain,
                                           const ss_nl_params &np, u64 (&r)[N])
{
    constexpr int NR = 2 * T + 1;
    ss_sacc2 acc;
    acc.clear();
#pragma unroll
    for (int i = 0; i < NR; i++) {
        const u64 m = ss_mul(x[i], b[i]);
        send<STREAM>(msg + (size_t)i * mcount + em, m);
        SS_SPLIT31(m, w0, w1);
        acc.mac(w0, w1, np.ilambda[i]);
    }
    const u64 v = acc.value();   // the multipliers of IDs 1..2t+1 are integers
    const u64 y = v <= (SS_P - 1) / 2 ? v : 0;
    send<STREAM>(yplain + em, y);
#pragma unroll
    for (int m = 0; m < N; m++) r[m] = ss_mul(y, bi[m]);
}

// Linear - Truncation - NonLinear tail of a convolution layer in one launch (the order of Sec. VII-A):
// reduction + RERAND + truncation of the product shares c [n][B][C][HW], then ReLU under the mask, the
// result stored as shares and, if planes != nullptr, as limb planes for the next
// convolution.  One element per thread, lanes arranged as in the share + planes kernel (lane l: pixel l%16,
// channel 4 g + l/16 of the wave's group g).  The messages hold the values of the separate kernels, in the
// order of this kernel's threads (so that a wave writes 512 consecutive bytes of every message plane): the
// element of thread t of block (x, y) is at position (y gridDim.x + x) 256 + t of a plane of gridDim.x
// gridDim.y 256 positions.
template <int N, int T, bool STREAM, bool LEAN>
__global__ __launch_bounds__(BLOCK) void layer_tail_kernel(const u64 *c, u64 *__restrict__ msg1, u64 *__restrict__ msg2,
                                                           u64 *__restrict__ umsg, u64 *__restrict__ wsh,
                                                           u64 *__restrict__ rmsg, u64 *__restrict__ yplain,
                                                           const u64 *__restrict__ sh_b, const u64 *__restrict__ sh_bi,
                                                           u64 *out, signed char *__restrict__ planes, int B, int C, int HW,
                                                           size_t party_bytes, ss_dr_params dp, ss_tr_params tp,
                                                           ss_nl_params np, ss_part_src ps)
{
    const int lane = threadIdx.x & 63, r16 = lane & 15, j = lane >> 4;
    const int pix = blockIdx.x * 16 + r16, c0 = blockIdx.y * 16 + 4 * (threadIdx.x >> 6);
    const size_t count = (size_t)B * HW * C;
    if (planes && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < N)
        *reinterpret_cast<int4 *>(planes + threadIdx.x * party_bytes + SS_NLIMB * count) = make_int4(0, 0, 0, 0);
    u64 dig[N];
#pragma unroll
    for (int p = 0; p < N; p++) dig[p] = 0;
    // A lane past the last pixel repeats the last pixel of its channel: it loads, computes and stores the very
    // values of that element's own lane, which sits in the same wave (so also in place nothing is read after
    // it was overwritten), and its messages go to its own, otherwise unused position.  Without this a block
    // of one or two pixels leaves its waves with four or eight active lanes, and waves with so few lanes run
    // their 64-bit integer arithmetic almost twice as slowly as full ones (measured on MI355X).
    if (c0 + j < C) {
        const int px = min(pix, B * HW - 1);
        const int b = px / HW, hw = px - b * HW;
        const size_t e = ((size_t)b * C + (c0 + j)) * HW + hw;
        const size_t mcount = (size_t)gridDim.x * gridDim.y * BLOCK;
        const size_t em = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * BLOCK + threadIdx.x;
        u64 o[N], r[N];
        // the mask shares are requested before the reduction starts, so that they arrive while it computes
        u64 mb[2 * T + 1], mbi[N];
#pragma unroll
        for (int i = 0; i < 2 * T + 1; i++) mb[i] = sh_b[(size_t)i * count + e];
#pragma unroll
        for (int m = 0; m < N; m++) mbi[m] = sh_bi[(size_t)m * count + e];
        u64 secret;
        reduce_truncate<N, T, true, STREAM, LEAN>(e, count, em, mcount, c, msg1, msg2, umsg, wsh, dp, tp, ps, o, secret);
        relu_fixed<N, T, STREAM>(o, em, mcount, mb, mbi, rmsg, yplain, np, r);
#pragma unroll
        for (int p = 0; p < N; p++) {
            out[(size_t)p * count + e] = r[p];
            dig[p] = balanced_digits(r[p]);
        }
    }
    if (!planes) return;   // uniform
    __shared__ __align__(16) u32 stage[N][SS_NLIMB][16][4];   // [party][limb][pixel][wave]
    stage_limbs<N>(dig, stage, N);
    store_staged_planes<N>(stage, planes, party_bytes, count, blockIdx.x * 16, B * HW, blockIdx.y * 16, N);
}

// The outputs of the layer tail without the protocol (all parties on one device): as for
// reduce_truncate_direct_kernel, what the parties end up with follows from the secret of the incoming
// degree-2t sharing.  x = REC of the 2t+1 product shares; the truncated value is floor(x / 2^f) on the signed
// value whatever the mask was; the elite party of the ReLU sees floor(x / 2^f) * beta, beta = REC of its k
// shares; every party's output is max(., 0) times its share of beta^-1.  Same residues in `out` and in the limb
// planes as layer_tail_kernel; no message is formed.  Lanes as in that kernel (pixel l%16, channel 4 g + l/16),
// so that the planes leave through the same staged 16-byte stores.
__global__ __launch_bounds__(BLOCK) void tail_direct_kernel(const u64 *c, const u64 *__restrict__ sh_b,
                                                            const u64 *__restrict__ sh_bi, u64 *out,
                                                            signed char *__restrict__ planes, int B, int C, int HW,
                                                            size_t party_bytes, ss_nl_params open_all, ss_tr_params tp,
                                                            ss_part_src ps)
{
    const int lane = threadIdx.x & 63, r16 = lane & 15, j = lane >> 4;
    const int pix = blockIdx.x * 16 + r16, c0 = blockIdx.y * 16 + 4 * (threadIdx.x >> 6);
    const size_t count = (size_t)B * HW * C;
    const int n = tp.n, k = tp.t + 1, nr = 2 * tp.t + 1;
    if (planes && blockIdx.x == 0 && blockIdx.y == 0 && (int)threadIdx.x < n)
        *reinterpret_cast<int4 *>(planes + threadIdx.x * party_bytes + SS_NLIMB * count) = make_int4(0, 0, 0, 0);
    u64 dig[SS_MAXN];
#pragma unroll
    for (int p = 0; p < SS_MAXN; p++) dig[p] = 0;
    if (pix < B * HW && c0 + j < C) {
        const int b = pix / HW, hw = pix - b * HW;
        const size_t e = ((size_t)b * C + (c0 + j)) * HW + hw;
        u64 cin[2 * SS_MAXT + 1];
#pragma unroll
        for (int i = 0; i < 2 * SS_MAXT + 1; i++)
            if (i < nr) cin[i] = c[(size_t)i * count + e];
        if (ps.planes > 1) {
            const int cut = first_cut_party(ps, e);
#pragma unroll
            for (int i = 0; i < 2 * SS_MAXT + 1; i++)
                if (i < nr) cin[i] = add_planes_of(cin[i], c, i, count, e, ps, cut);
        }
        ss_sacc acc, bacc;
        acc.clear();
        bacc.clear();
#pragma unroll
        for (int i = 0; i < 2 * SS_MAXT + 1; i++)
            if (i < nr) acc.mac(cin[i], open_all.ilambda[i]);
#pragma unroll
        for (int q = 0; q < SS_MAXK; q++)
            if (q < k) bacc.mac(sh_b[(size_t)q * count + e], tp.ilambda[q]);
        // the multipliers of IDs 1..2t+1 and of IDs 1..k are integers
        const u64 v = ss_mul(shift_signed(acc.value(), tp.f), bacc.value());
        const u64 y = v <= (SS_P - 1) / 2 ? v : 0;
#pragma unroll
        for (int m = 0; m < SS_MAXN; m++) {
            if (m < n) {
                const u64 r = ss_mul(y, sh_bi[(size_t)m * count + e]);
                out[(size_t)m * count + e] = r;
                dig[m] = balanced_digits(r);
            }
        }
    }
    if (!planes) return;   // uniform
    __shared__ __align__(16) u32 stage[SS_MAXN][SS_NLIMB][16][4];   // [party][limb][pixel][wave]
    stage_limbs<SS_MAXN>(dig, stage, n);
    store_staged_planes<SS_MAXN>(stage, planes, party_bytes, count, blockIdx.x * 16, B * HW, blockIdx.y * 16, n);
}

// ------------------------------------------------------------------ reduction + truncation, all parties at once
// The outputs of RED + RERAND + truncation do not depend on the reshare or zero
// randomness: the elite party of the truncation reconstructs x + alpha, where x
// is the secret of the incoming degree-2t sharing, whatever the reduced shares
// look like.  With every party's share in one thread that secret can be taken
// directly (REC from the 2t+1 incoming shares), and the output shares follow from
// it as in truncation steps 2 and 3.  Same residues in `out` (and `rec`) as the
// protocol kernels; no message is formed, so this is not what the parties of the
// protocol compute, only what they end up with.
// SEVERAL: the product is in several planes.  Tensors and products of one plane take the instance without the code that adds them up:
// it holds no registers for it and does not wait for the launch's arguments to know (300000 elements, n = 3 5.10 -> 4.60 us, n = 5 over
// the 45-bit prime 7.42 -> 6.72; the reductions with messages gain nothing by it, t = 3 loses up to 15 %).
template <int N, int T, bool SEVERAL>
__global__ __launch_bounds__(BLOCK) void reduce_truncate_direct_kernel(const u64 *c, u64 *out, u64 *__restrict__ rec,
                                                                       size_t count, size_t first,
                                                                       ss_nl_params open_all, ss_tr_params tp,
                                                                       ss_part_src ps)
{
    const size_t e = first + element_block<BLOCK>(min(count - first, LAUNCH_ELEMENTS), count) * BLOCK + threadIdx.x;   // from element `first` on
    if (e >= count) return;
    // (the shares are requested ahead of the planes' bounds: after a product in eight planes, 512 x 49 x 4608, 49 -> 43 us)
    u64 cin[2 * T + 1];
#pragma unroll
    for (int i = 0; i < 2 * T + 1; i++) cin[i] = c[(size_t)i * count + e];
    if constexpr (SEVERAL) add_planes(cin, c, count, e, ps);
    ss_sacc2 acc;
    acc.clear();
#pragma unroll
    for (int i = 0; i < 2 * T + 1; i++) {
        SS_SPLIT31(cin[i], w0, w1);
        acc.mac(w0, w1, open_all.ilambda[i]);
    }
    u64 alpha, o[MAXP<N>], secret;
    const u64 ev = mask_of<T>(tp, e, alpha);
    shift_and_unmask<N, T, false>(ss_canon(ss_fold(acc.lazy() + alpha)), ev, ss_counter(e), e, count, nullptr, tp,
                                  N ? N : tp.n, o, secret);
#pragma unroll
    for (int m = 0; m < MAXP<N>; m++)
        if (N != 0 || m < tp.n) out[(size_t)m * count + e] = o[m];
    if (rec) rec[e] = secret;
}

// ------------------------------------------------------------------ SSS-NonLinear (Sec. VI-C)
// What the trusted source prepares ahead of the inference (Sec. VII-B): a positive
// mask beta per element, its inverse in F_p (Fermat: beta^(p-2), p - 2 = 2^61 - 3)
// and a degree-t sharing of each.  One thread per element.
__device__ __forceinline__ u64 mask_beta(const ss_nl_params &np, u64 counter)
{
    return 1 + ((ss_draw(np.beta_key, counter) >> 3) & ((1ULL << np.bbits) - 1));
}

__device__ __forceinline__ u64 field_inverse(u64 beta)
{
#if defined(SS_FIELD_P45)
    // beta^(p - 2), p - 2 = 2^45 - 57: square and multiply from the top bit down
    u64 inv = beta;
    for (int bit = SS_PBITS - 2; bit >= 0; bit--) {
        inv = ss_mul(inv, inv);
        if (((SS_P - 2) >> bit) & 1) inv = ss_mul(inv, beta);
    }
    return inv;
#else
    // beta^(2^61 - 3): the exponent is 59 one bits, then 0, then 1
    u64 inv = beta;
    for (int i = 0; i < 58; i++) inv = ss_mul(ss_mul(inv, inv), beta);   // beta^(2^59 - 1)
    inv = ss_mul(inv, inv);                                              // bit 1 of the exponent is 0
    return ss_mul(ss_mul(inv, inv), beta);                               // bit 0 is 1
#endif
}

__global__ __launch_bounds__(BLOCK) void nonlinear_masks_kernel(u64 *__restrict__ sh_b, u64 *__restrict__ sh_bi,
                                                                size_t count, ss_nl_params np)
{
    const size_t e = (size_t)blockIdx.x * BLOCK + threadIdx.x;
    if (e >= count) return;
    const u64 beta = mask_beta(np, e);
    const u64 inv = field_inverse(beta);
    u64 cb[SS_MAXT], cbi[SS_MAXT];
    draw_coeffs<SS_MAXT>(cb, np.bgen_key, np.t, e);
    draw_coeffs<SS_MAXT>(cbi, np.bigen_key, np.t, e);
#pragma unroll
    for (int m = 0; m < SS_MAXN; m++) {
        if (m < np.n) {
            sh_b[(size_t)m * count + e] = ss_poly_eval<SS_MAXT>(beta, cb, np.t, m + 1);
            sh_bi[(size_t)m * count + e] = ss_poly_eval<SS_MAXT>(inv, cbi, np.t, m + 1);
        }
    }
}

// ReLU on shares, the three steps for the elements a thread owns (send = store
// to the workspace, receive = from registers, as in the kernels above):
//   1. parties 1..2t+1: m_i = x_i * beta_i                          -> msg[i]
//   2. elite party: REC of the 2t+1 products = x * beta; ReLU on the
//      signed value, in the clear                                   -> yplain
//   3. every party: out_i = y * betainv_i                            -> out[i]
// MASKOFF = false stops after step 2 (the pooled form continues from yplain in another kernel).
template <int VEC, bool MASKOFF, bool STREAM>
__global__ __launch_bounds__(BLOCK) void relu_kernel(const u64 *x, const u64 *__restrict__ sh_b,
                                                     const u64 *__restrict__ sh_bi, u64 *__restrict__ msg,
                                                     u64 *__restrict__ yplain, u64 *out, size_t count,
                                                     ss_nl_params np)
{
    const size_t e0 = (element_block<BLOCK * VEC>(count, count) * BLOCK + threadIdx.x) * VEC;
    if (e0 >= count) return;
    const int nr = 2 * np.t + 1;
    // all operands are requested up front, so that the three steps wait for memory once
    pack_t<VEC> xi[2 * SS_MAXT + 1], bi[2 * SS_MAXT + 1], binv[SS_MAXN];
#pragma unroll
    for (int i = 0; i < 2 * SS_MAXT + 1; i++) {
        if (i < nr) {
            xi[i].load(x + (size_t)i * count + e0);
            bi[i].load(sh_b + (size_t)i * count + e0);
        }
    }
#pragma unroll
    for (int m = 0; m < SS_MAXN; m++)
        if (MASKOFF && m < np.n) binv[m].load(sh_bi + (size_t)m * count + e0);
    ss_sacc acc[VEC];
#pragma unroll
    for (int u = 0; u < VEC; u++) acc[u].clear();
#pragma unroll
    for (int i = 0; i < 2 * SS_MAXT + 1; i++) {
        if (i < nr) {
            pack_t<VEC> m;
#pragma unroll
            for (int u = 0; u < VEC; u++) {
                m.v[u] = ss_mul(xi[i].v[u], bi[i].v[u]);
                acc[u].mac(m.v[u], np.ilambda[i]);
            }
            m.template send<STREAM>(msg + (size_t)i * count + e0);
        }
    }
    pack_t<VEC> y;
#pragma unroll
    for (int u = 0; u < VEC; u++) {
        const u64 v = acc[u].value();   // the multipliers of IDs 1..2t+1 are integers
        y.v[u] = v <= (SS_P - 1) / 2 ? v : 0;   // negative values are the upper half of the field
    }
    if constexpr (MASKOFF)
        y.template send<STREAM>(yplain + e0);
    else
        y.store(yplain + e0);   // read by the pooling launch
#pragma unroll
    for (int m = 0; m < SS_MAXN; m++) {
        if (MASKOFF && m < np.n) {
            pack_t<VEC> o;
#pragma unroll
            for (int u = 0; u < VEC; u++) o.v[u] = ss_mul(y.v[u], binv[m].v[u]);
            o.store(out + (size_t)m * count + e0);
        }
    }
}

// Masks for ReLU followed by pooling: beta has to be equal inside one pooling kernel.  Where the kernels
// partition the plane a group is a kernel position (elements beyond the last full kernel join the last
// one), otherwise the whole plane; beta is drawn at counter = group index.  The sharing coefficients are
// drawn per element.  INV = false: one thread per input element, shares of beta; INV = true: one thread per
// pooled element, shares of beta^-1 of its kernel's group.
template <bool INV>
__global__ __launch_bounds__(BLOCK) void pool_masks_kernel(u64 *__restrict__ sh, size_t count, ss_pool_geom g,
                                                           ss_nl_params np)
{
    const size_t e = (size_t)blockIdx.x * BLOCK + threadIdx.x;
    if (e >= count) return;
    const int w = INV ? g.Wo : g.W, h = INV ? g.Ho : g.H;
    const size_t plane = e / ((size_t)h * w);
    const int r = (int)(e - plane * (size_t)h * w), row = r / w, col = r - row * w;
    u64 group = plane;
    if (g.tiled) {
        const int oh = INV ? row : min(row / g.kh, g.Ho - 1), ow = INV ? col : min(col / g.kw, g.Wo - 1);
        group = (plane * g.Ho + oh) * g.Wo + ow;
    }
    u64 secret = mask_beta(np, group);
    if (INV) secret = field_inverse(secret);
    u64 cf[SS_MAXT];
    draw_coeffs<SS_MAXT>(cf, INV ? np.bigen_key : np.bgen_key, np.t, e);
#pragma unroll
    for (int m = 0; m < SS_MAXN; m++)
        if (m < np.n) sh[(size_t)m * count + e] = ss_poly_eval<SS_MAXT>(secret, cf, np.t, m + 1);
}

// ReLU and pooling in one launch: a workgroup opens a run of input elements (steps 1 and 2 of relu_kernel), keeps the
// rectified values in LDS, pools them there and takes the mask off.  Bound by memory: 2 (2t+1) words read and 2t+2 written
// per input element, and the pooled values never make the way through memory between two launches.  A run is `P` whole
// planes or, for larger ones, the input rows of `R` output rows of one plane (`strips` runs per plane, ss_pool_cut): both
// are contiguous.  Rows that the next run's kernels share with this one's are opened by both and their messages are written
// by the later run, so a run owns the rows from its first kernel's to the next run's first.
// n = 5, on inputs that change from call to call: 3 x 3 / 2 on 192 planes of 112 x 112 74.9 us, in two launches 75.8 (the
// same call repeated: 59.8 and 60.7 us); on 64 of them 28.2 and 30.0 us; 7 x 7 on 2048 planes of 7 x 7 11.0 and 22.7 us.
template <int T, bool STREAM>
__global__ __launch_bounds__(512) void relu_pool_kernel(const u64 *__restrict__ x, const u64 *__restrict__ sh_b,
                                                          const u64 *__restrict__ sh_bi, u64 *__restrict__ msg,
                                                          u64 *__restrict__ rplain, u64 *__restrict__ yplain,
                                                          u64 *__restrict__ out, int planes, int P, int R, int strips,
                                                          ss_pool_geom g, ss_nl_params np)
{
    extern __shared__ u64 pooled[];   // max(x * beta, 0) of the run's rows that its kernels cover
    constexpr int NR = 2 * T + 1;
    const size_t cin = (size_t)planes * g.H * g.W, cout = (size_t)planes * g.Ho * g.Wo;
    const int plane = strips == 1 ? blockIdx.x * P : blockIdx.x / strips, s = strips == 1 ? 0 : blockIdx.x - plane * strips;
    const int many = min(P, planes - plane);
    const auto [oh0, oh1, row0, own1, need1] = ss_pool_cut(s, strips, R, g.H, g.kh, g.sh, g.ph, g.Ho);
    const bool whole = strips == 1;
    const int open = whole ? many * g.H * g.W : (max(own1, need1) - row0) * g.W, own = whole ? open : (own1 - row0) * g.W,
              keep = whole ? open : (need1 - row0) * g.W;
    const size_t e0 = (size_t)plane * g.H * g.W + (size_t)row0 * g.W;
    for (int i = threadIdx.x; i < open; i += (int)blockDim.x) {
        const size_t e = e0 + i;
        u64 xs[NR], b[NR];
#pragma unroll
        for (int q = 0; q < NR; q++) {
            xs[q] = x[(size_t)q * cin + e];
            b[q] = sh_b[(size_t)q * cin + e];
        }
        ss_sacc2 acc;
        acc.clear();
#pragma unroll
        for (int q = 0; q < NR; q++) {
            const u64 m = ss_mul(xs[q], b[q]);
            if (i < own) send<STREAM>(msg + (size_t)q * cin + e, m);
            SS_SPLIT31(m, w0, w1);
            acc.mac(w0, w1, np.ilambda[q]);
        }
        const u64 v = acc.value();   // the multipliers of IDs 1..2t+1 are integers
        const u64 r = v <= (SS_P - 1) / 2 ? v : 0;
        if (i < own) send<STREAM>(rplain + e, r);
        if (i < keep) pooled[i] = r;
    }
    __syncthreads();
    const int outs = whole ? many * g.Ho * g.Wo : (oh1 - oh0) * g.Wo;
    const size_t o0 = ((size_t)plane * g.Ho + oh0) * g.Wo;
    for (int i = threadIdx.x; i < outs; i += (int)blockDim.x) {
        const unsigned row = (unsigned)i / (unsigned)g.Wo, ow = i - row * g.Wo;   // row: over all planes of the run
        const unsigned pl = whole ? row / (unsigned)g.Ho : 0, oh = whole ? row - pl * g.Ho : oh0 + row;
        const int h0 = (int)oh * g.sh - g.ph, w0 = (int)ow * g.sw - g.pw;
        const u64 *src = pooled + (size_t)pl * g.H * g.W;
        u64 acc = 0;
        for (int a = max(0, h0); a < min(g.H, h0 + g.kh); a++)
            for (int c = max(0, w0); c < min(g.W, w0 + g.kw); c++) {
                const u64 v = src[(a - row0) * g.W + c];
                acc = g.mode == 0 ? (v > acc ? v : acc) : ss_add(acc, v);
            }
        const size_t o = o0 + i;
        send<STREAM>(yplain + o, acc);
#pragma unroll
        for (int m = 0; m < SS_MAXN; m++)
            if (m < np.n) out[(size_t)m * cout + o] = ss_mul(acc, sh_bi[(size_t)m * cout + o]);
    }
}

// The same from the rectified values in memory, where a kernel's rows do not fit into LDS or the output lies in the
// mask (ss_plan_pool).  One thread per pooled element: the maximum or the sum of the opened, rectified products
// r = max(x*beta, 0) over the kernel's elements inside the plane (padding adds nothing to a sum and cannot win a maximum of
// non-negative values), then y * betainv_m for every party.
__global__ __launch_bounds__(BLOCK) void pool_maskoff_kernel(const u64 *__restrict__ rplain,
                                                             const u64 *__restrict__ sh_bi, u64 *__restrict__ yplain,
                                                             u64 *__restrict__ out, size_t count, ss_pool_geom g, int n)
{
    const size_t o = (size_t)blockIdx.x * BLOCK + threadIdx.x;
    if (o >= count) return;
    const size_t plane = o / ((size_t)g.Ho * g.Wo);
    const int r = (int)(o - plane * (size_t)g.Ho * g.Wo), oh = r / g.Wo, ow = r - oh * g.Wo;
    const u64 *src = rplain + plane * (size_t)g.H * g.W;
    const int h0 = oh * g.sh - g.ph, w0 = ow * g.sw - g.pw;
    u64 acc = 0;
    for (int i = max(0, -h0); i < min(g.kh, g.H - h0); i++)
        for (int j = max(0, -w0); j < min(g.kw, g.W - w0); j++) {
            const u64 v = src[(size_t)(h0 + i) * g.W + (w0 + j)];
            acc = g.mode == 0 ? (v > acc ? v : acc) : ss_add(acc, v);
        }
    yplain[o] = acc;
#pragma unroll
    for (int m = 0; m < SS_MAXN; m++)
        if (m < n) out[(size_t)m * count + o] = ss_mul(acc, sh_bi[(size_t)m * count + o]);
}

// below this many elements one element per thread gives more waves to hide latency
constexpr size_t VEC2_MIN_COUNT = (size_t)1 << 20;
// Below this many elements RED + RERAND alone with t = 3 spreads an element over party lanes: the one-thread kernel takes
// 1.2 times as long at 1 K elements and as long at 16 K.  For t = 1 and 2, and with the truncation in the same launch, it
// is the faster one at every size (n = 5, 64 elements: 4.2 against 6.5 us).
constexpr size_t LANES_MAX_COUNT = 16 * 1024;

// Messages are written once and not read by the library again.  Left to the caches they cost nothing while a call's
// traffic fits the 256 MB of the last level (the next call overwrites them there); beyond, writing them past the
// caches is faster.  44 planes written per 5 read, no arithmetic, the same call repeated, MI355X: 24.4 / 26.7 us (cached /
// streamed) at 157 MB, 56.2 / 53.1 us at 315 MB, 324 / 273 us at 1.65 GB.  With inputs that change from call to call the line
// lies there too (at 64, 128, 600 MB stacks and single calls are 0 to 8 % slower).  The reductions' many planes only where they
// start on halves of cache lines: smaller parts past the caches cost more, whole halves do not.  Reduce + truncate, us, streamed /
// cached, with planes 1, 2 or 4 elements off a line, then 8: n = 5, 1.2 M elements 125 / 108, 91 / 99; n = 7, 2.6 M 430 / 390, 355 / 388;
// n = 4, 2.4 M 124 / 114, 100 / 103.  The reduction alone of t = 1 sends the fewest planes and off the halves is faster past
// the caches from 300 MB on: n = 4, 2.3 M elements 2 off 80 / 93, n = 3, 2.7 M 78 / 82, 1.9 M (269 MB) 56 / 50.
// The other kernels go by the size alone.  Streamed / cached with planes 1 or 2 off a line and operands that change: reconstruction, m = 3,
// 349 MB 55 / 60, 670 MB 103 / 114; truncation, n = 5, 349 MB 63 / 73, 670 MB 145 / 136; ReLU, n = 5, 349 MB 84 / 88, 670 MB 163 / 160: past
// 600 MB the last two are 0 to 15 % faster cached there.
inline bool streams_messages(size_t words) { return words * sizeof(u64) > ((size_t)256 << 20); }

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

inline unsigned blocks_for(size_t count, int vec, int block = BLOCK)
{
    const size_t per_block = (size_t)block * vec;
    return (unsigned)((count + per_block - 1) / per_block);
}

// A launch holds less than 2^32 threads in each direction.  The runtime takes a larger grid without an error and runs a
// part of it, so that no launcher may reach it: a tensor goes in several launches or is refused.
inline bool fits_launch(size_t blocks, int block = BLOCK) { return blocks * block < ((size_t)1 << 32); }
template <typename F>
inline void for_each_launch(size_t count, F &&launch)
{
    for (size_t first = 0; first < count; first += LAUNCH_ELEMENTS)
        launch(first, dim3(blocks_for(count - first < LAUNCH_ELEMENTS ? count - first : LAUNCH_ELEMENTS, 1)));
}

}  // namespace

// The two-element path needs every plane start 16-byte aligned: aligned bases
// and an even element count.
hipError_t ss_launch_share(const u64 *secret, u64 *shares, size_t count, int n, int degree, const ss_keys &keys,
                           hipStream_t stream)
{
    const bool v2 = (count % 2 == 0) && aligned16(secret) && aligned16(shares);
    if (!fits_launch(blocks_for(count, v2 ? 2 : 1))) return hipErrorInvalidConfiguration;
#define SS_SHARE(VEC, NC, DC)                                                                                       \
    hipLaunchKernelGGL((share_kernel<VEC, NC, DC>), dim3(blocks_for(count, VEC, (SHARE_BLOCK<VEC, NC>))), \
                       dim3((SHARE_BLOCK<VEC, NC>)), \
                       0, stream, secret, shares, count, n, degree, keys)
    if (v2 && n == 5 && degree == 2)
        SS_SHARE(2, 5, 2);
    else if (v2 && n == 3 && degree == 1)
        SS_SHARE(2, 3, 1);
    else if (v2)
        SS_SHARE(2, 0, 0);
    else if (n == 5 && degree == 2)
        SS_SHARE(1, 5, 2);
    else if (n == 3 && degree == 1)
        SS_SHARE(1, 3, 1);
    else
        SS_SHARE(1, 0, 0);
#undef SS_SHARE
    return hipGetLastError();
}

hipError_t ss_launch_reconstruct(const u64 *shares, u64 *secret, size_t count, const ss_rec_params &rp,
                                 hipStream_t stream)
{
    const bool v2 = (count % 2 == 0) && aligned16(secret) && aligned16(shares);
    if (!fits_launch(blocks_for(count, v2 ? 2 : 1))) return hipErrorInvalidConfiguration;
    const bool streams = streams_messages((size_t)(rp.m + 1) * count);
#define SS_REC(VEC)                                                                                              \
    hipLaunchKernelGGL((streams ? reconstruct_kernel<VEC, true> : reconstruct_kernel<VEC, false>), dim3(blocks_for(count, VEC)), \
                       dim3(BLOCK), 0, stream, shares, secret, count, rp)
    if (v2)
        SS_REC(2);
    else
        SS_REC(1);
#undef SS_REC
    return hipGetLastError();
}

// (3,1) and (5,2), and the two counts of t = 3, have their party count fixed at compile time; the other counts of t = 1 and
// 2 take theirs at run time.  SS_SCHEME(n, t, LAUNCH) runs LAUNCH(N, T).
#define SS_SCHEME(n_, t_, LAUNCH)               \
    do {                                        \
        if ((n_) == 5 && (t_) == 2) LAUNCH(5, 2); \
        else if ((n_) == 3 && (t_) == 1) LAUNCH(3, 1); \
        else if ((t_) == 1) LAUNCH(0, 1);       \
        else if ((t_) == 2) LAUNCH(0, 2);       \
        else if ((n_) == 7) LAUNCH(7, 3);       \
        else LAUNCH(8, 3);                      \
    } while (0)

// Reductions with an instance without the code for cut tiles, which costs registers (n = 6: seven waves per SIMD instead of eight): what
// tensors and products of at most two planes per tile take where it is the faster one.  Reduce + truncate + open, us, with -> without:
// messages past the caches, 1605632 elements n = 4 66.2 -> 64.7, layer tail of eight images of 64 x 56 x 56, n = 3, 98.0 -> 93.9;
// n = 6, 50176 elements 8.55 -> 8.08; small tensors of t = 1, 10000 elements n = 3 3.62 -> 3.50.  Between those t = 1 is faster with it (n = 3,
// 200704 elements 9.6 -> 9.0), as are (5,2) and t = 3 at most sizes.
template <int N, int T>
constexpr bool HAS_LEAN = T == 1 || (N == 0 && T == 2);
inline bool takes_lean(const ss_part_src &ps, int t, bool streams, size_t count)
{
    return (ps.planes <= 1 || (ps.planes == 2 && ps.first_cut == 0)) && (t != 1 || streams || count < 65536);
}

hipError_t ss_launch_degree_reduce(const u64 *c, u64 *msg1, u64 *msg2, u64 *out, size_t count,
                                   const ss_dr_params &dp, const ss_part_src &ps, hipStream_t stream)
{
    const ss_tr_params none = {};
    if (!fits_launch(blocks_for(count, 1))) return hipErrorInvalidConfiguration;
    if (dp.t == 3 && count < LANES_MAX_COUNT) {
        hipLaunchKernelGGL(degree_reduce_lanes_kernel, dim3((unsigned)((count + 31) / 32)), dim3(BLOCK), 0, stream, c, msg1,
                           msg2, out, count, dp, ps);
        return hipGetLastError();
    }
    const size_t k = dp.t + 1, nr = 2 * dp.t + 1, n = dp.n;
    const size_t words = (nr + n + nr * k + k * n) * count;
    const bool streams = starts_halves(count) ? streams_messages(words) : dp.t == 1 && streams_messages(words - words / 8);
    const bool lean = takes_lean(ps, dp.t, streams, count);
#define SS_LAUNCH(NC, TC)                                                                                               \
    hipLaunchKernelGGL((streams ? lean ? degree_reduce_kernel<NC, TC, false, true, HAS_LEAN<NC, TC>>                        \
                                      : degree_reduce_kernel<NC, TC, false, true, false>                                          \
                               : lean ? degree_reduce_kernel<NC, TC, false, false, HAS_LEAN<NC, TC>>                       \
                                      : degree_reduce_kernel<NC, TC, false, false, false>),                                       \
                       dim3(blocks_for(count, 1)), dim3(BLOCK), 0, stream, c, msg1, msg2, (u64 *)nullptr, (u64 *)nullptr, \
                       out, count, (u64 *)nullptr, dp, none, ps)
    SS_SCHEME(dp.n, dp.t, SS_LAUNCH);
#undef SS_LAUNCH
    return hipGetLastError();
}

hipError_t ss_launch_degree_reduce_truncate(const u64 *c, u64 *msg1, u64 *msg2, u64 *u, u64 *wsh, u64 *out,
                                            u64 *rec, size_t count, const ss_dr_params &dp, const ss_tr_params &tp,
                                            const ss_part_src &ps, hipStream_t stream)
{
    if (!fits_launch(blocks_for(count, 1))) return hipErrorInvalidConfiguration;
    const size_t k = dp.t + 1, nr = 2 * dp.t + 1, n = dp.n;
    const bool streams = starts_halves(count) && streams_messages((nr + n + nr * k + k * n + k + n) * count);
    const bool lean = takes_lean(ps, dp.t, streams, count);
#define SS_LAUNCH(NC, TC)                                                                                               \
    hipLaunchKernelGGL((streams ? lean ? degree_reduce_kernel<NC, TC, true, true, HAS_LEAN<NC, TC>>                        \
                                      : degree_reduce_kernel<NC, TC, true, true, false>                                          \
                               : lean ? degree_reduce_kernel<NC, TC, true, false, HAS_LEAN<NC, TC>>                       \
                                      : degree_reduce_kernel<NC, TC, true, false, false>),                                       \
                       dim3(blocks_for(count, 1)), dim3(BLOCK), 0, stream, c, msg1, msg2, u, wsh, out, count, rec, dp, tp, ps)
    SS_SCHEME(dp.n, dp.t, SS_LAUNCH);
#undef SS_LAUNCH
    return hipGetLastError();
}

hipError_t ss_launch_truncate(const u64 *x, u64 *u, u64 *wsh, u64 *out, size_t count, const ss_tr_params &tp,
                              hipStream_t stream)
{
    const bool streams = streams_messages((size_t)(2 * (tp.t + 1) + 2 * tp.n) * count);
#define SS_LAUNCH(NC, TC)                                                                                           \
    hipLaunchKernelGGL((streams ? truncate_kernel<NC, TC, true> : truncate_kernel<NC, TC, false>), grid, dim3(BLOCK), 0, \
                       stream, x, u, wsh, out, count, first, tp)
    for_each_launch(count, [&](size_t first, dim3 grid) { SS_SCHEME(tp.n, tp.t, SS_LAUNCH); });
#undef SS_LAUNCH
    return hipGetLastError();
}

hipError_t ss_launch_nonlinear_masks(u64 *sh_b, u64 *sh_bi, size_t count, const ss_nl_params &np, hipStream_t stream)
{
    if (!fits_launch(blocks_for(count, 1))) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(nonlinear_masks_kernel, dim3(blocks_for(count, 1)), dim3(BLOCK), 0, stream, sh_b, sh_bi, count,
                       np);
    return hipGetLastError();
}

hipError_t ss_launch_relu(const u64 *x, const u64 *sh_b, const u64 *sh_bi, u64 *msg, u64 *yplain, u64 *out,
                          size_t count, const ss_nl_params &np, hipStream_t stream)
{
    const bool v2 = (count % 2 == 0) && aligned16(x) && aligned16(sh_b) && aligned16(sh_bi) && aligned16(msg) &&
                    aligned16(yplain) && aligned16(out) && count >= VEC2_MIN_COUNT;
    if (!fits_launch(blocks_for(count, v2 ? 2 : 1))) return hipErrorInvalidConfiguration;
    const size_t nr = 2 * np.t + 1, n = np.n;
    const bool streams = streams_messages((2 * n + nr + n + nr + 1) * count);
#define SS_RELU(VEC)                                                                                                       \
    hipLaunchKernelGGL((streams ? relu_kernel<VEC, true, true> : relu_kernel<VEC, true, false>), dim3(blocks_for(count, VEC)), \
                       dim3(BLOCK), 0, stream, x, sh_b, sh_bi, msg, yplain, out, count, np)
    if (v2)
        SS_RELU(2);
    else
        SS_RELU(1);
#undef SS_RELU
    return hipGetLastError();
}

hipError_t ss_launch_pool_masks(u64 *sh_b, u64 *sh_bi, size_t planes, const ss_pool_geom &g, const ss_nl_params &np,
                                hipStream_t stream)
{
    const size_t cin = planes * g.H * g.W, cout = planes * g.Ho * g.Wo;
    if (!fits_launch(blocks_for(cin, 1)) || !fits_launch(blocks_for(cout, 1))) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(pool_masks_kernel<false>, dim3(blocks_for(cin, 1)), dim3(BLOCK), 0, stream, sh_b, cin, g, np);
    hipLaunchKernelGGL(pool_masks_kernel<true>, dim3(blocks_for(cout, 1)), dim3(BLOCK), 0, stream, sh_bi, cout, g, np);
    return hipGetLastError();
}

hipError_t ss_launch_relu_pool(const u64 *x, const u64 *sh_b, const u64 *sh_bi, u64 *msg, u64 *rplain, u64 *yplain,
                               u64 *out, size_t planes, const ss_pool_geom &g, const ss_nl_params &np,
                               hipStream_t stream)
{
    const size_t cin = planes * g.H * g.W, cout = planes * g.Ho * g.Wo;
    const bool streams = streams_messages((size_t)(3 * (2 * np.t + 1) + 1) * cin);
    // the shares of parties 1..2t+1 are what a call reads of the mask
    const bool out_in_mask = out < sh_b + (2 * np.t + 1) * cin && sh_b < out + (size_t)np.n * cout;
    const ss_pool_plan p = ss_plan_pool(planes, g.H, g.W, g.kh, g.sh, g.Ho, out_in_mask);
    if (p.one_launch) {
#define SS_POOL(T)                                                                                                    \
    hipLaunchKernelGGL((streams ? relu_pool_kernel<T, true> : relu_pool_kernel<T, false>), dim3((unsigned)p.blocks), \
                       dim3(p.threads), p.lds, stream, x, sh_b, sh_bi, msg, rplain, yplain, out, (int)planes, p.P, p.R, \
                       p.strips, g, np)
        if (np.t == 1)
            SS_POOL(1);
        else if (np.t == 2)
            SS_POOL(2);
        else
            SS_POOL(3);
#undef SS_POOL
        return hipGetLastError();
    }
    if (!fits_launch(blocks_for(cin, 1)) || !fits_launch(blocks_for(cout, 1))) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((streams ? relu_kernel<1, false, true> : relu_kernel<1, false, false>), dim3(blocks_for(cin, 1)),
                       dim3(BLOCK), 0, stream, x, sh_b, (const u64 *)nullptr, msg, rplain, (u64 *)nullptr, cin, np);
    hipLaunchKernelGGL(pool_maskoff_kernel, dim3(blocks_for(cout, 1)), dim3(BLOCK), 0, stream, rplain, sh_bi, yplain, out,
                       cout, g, np.n);
    return hipGetLastError();
}

hipError_t ss_launch_reduce_truncate_direct(const u64 *c, u64 *out, u64 *rec, size_t count, const ss_nl_params &open_all,
                                            const ss_tr_params &tp, const ss_part_src &ps, hipStream_t stream)
{
#define SS_LAUNCH(NC, TC)                                                                                       \
    hipLaunchKernelGGL((ps.planes > 1 ? reduce_truncate_direct_kernel<NC, TC, true> : reduce_truncate_direct_kernel<NC, TC, false>), \
                       grid, dim3(BLOCK), 0, stream, c, out, rec, count, first, \
                       open_all, tp, ps)
    for_each_launch(count, [&](size_t first, dim3 grid) { SS_SCHEME(tp.n, tp.t, SS_LAUNCH); });
#undef SS_LAUNCH
    return hipGetLastError();
}

hipError_t ss_launch_tail_direct(const u64 *c, const u64 *sh_b, const u64 *sh_bi, u64 *out, void *planes, int B, int C,
                                 int HW, const ss_nl_params &open_all, const ss_tr_params &tp, const ss_part_src &ps,
                                 hipStream_t stream)
{
    if (tp.kdiv != 1) return hipErrorInvalidValue;   // no rounding division in this kernel
    const dim3 grid((B * HW + 15) / 16, (C + 15) / 16), block(BLOCK);
    if (!fits_launch(grid.x)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(tail_direct_kernel, grid, block, 0, stream, c, sh_b, sh_bi, out, (signed char *)planes, B, C, HW,
                       ss_planes_bytes(B, C, HW, 1), open_all, tp, ps);
    return hipGetLastError();
}

hipError_t ss_launch_layer_tail(const u64 *c, u64 *msg1, u64 *msg2, u64 *umsg, u64 *wsh, u64 *rmsg, u64 *yplain,
                                const u64 *sh_b, const u64 *sh_bi, u64 *out, void *planes, int B, int C, int HW,
                                const ss_dr_params &dp, const ss_tr_params &tp, const ss_nl_params &np,
                                const ss_part_src &ps, hipStream_t stream)
{
    if (tp.kdiv != 1) return hipErrorInvalidValue;   // no rounding division in this kernel
    const dim3 grid((B * HW + 15) / 16, (C + 15) / 16), block(BLOCK);
    if (!fits_launch(grid.x)) return hipErrorInvalidConfiguration;
    const size_t party_bytes = ss_planes_bytes(B, C, HW, 1);
    const size_t k = dp.t + 1, nr = 2 * dp.t + 1, n = dp.n;
    // shares in and out, mask shares, messages
    const bool streams = streams_messages((2 * n + nr + n + nr * k + k * n + k + n + nr + 1) * (size_t)B * C * HW);
    const bool lean = streams && takes_lean(ps, dp.t, streams, (size_t)B * C * HW);
#define SS_TAIL(NC, TC)                                                                                                \
    hipLaunchKernelGGL((!streams ? layer_tail_kernel<NC, TC, false, false>                                             \
                        : lean  ? layer_tail_kernel<NC, TC, true, HAS_LEAN<NC, TC>>                                     \
                                : layer_tail_kernel<NC, TC, true, false>),                                              \
                       grid, block, 0,                                                                                 \
                       stream, c, msg1, msg2, umsg, wsh, rmsg, yplain, sh_b, sh_bi, out, (signed char *)planes, B, C, HW, \
                       party_bytes, dp, tp, np, ps)
    if (dp.n == 5 && dp.t == 2)
        SS_TAIL(5, 2);
    else if (dp.n == 3 && dp.t == 1)
        SS_TAIL(3, 1);
    else
        return hipErrorInvalidValue;   // the caller runs the separate kernels for other schemes
#undef SS_TAIL
    return hipGetLastError();
}

}  // namespace SS_NS
