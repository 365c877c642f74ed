// How a product is given to the kernels of gemm_kernels.hip and cut into work for their workgroups.  Plain C++, so that the
// rules can be checked without a GPU.  SS_NLIMB: limbs of a field element (8, or 6 over the 45-bit prime).
#pragma once
#include <math.h>
#include <stddef.h>

namespace SS_NS {

#define SS_GEMM_CUS 256

// cost of a unit (64 x 64 outputs, one k block) and of a tile's fold and stores
constexpr unsigned SS_UNIT_COST = 18;
constexpr unsigned SS_FOLD_COST = 16;

// A launch holds less than 2^32 threads: the runtime takes a larger grid without an error and runs a part of it.
constexpr bool fits_grid(long workgroups, int threads) { return workgroups * threads < (1L << 32); }

constexpr int SKINNY_COLS = 128;   // columns of a tile of gemm_skinny_kernel

struct gemm_plan {
    bool skinny;               // first operand of at most 16 rows: tiles of 16 x 128 (gemm_skinny_kernel)
    int ksplit;                // waves that share a tile of 16 x 16 in gemm_ksplit_kernel; 0: gemm_limb_kernel
    long tiles, units;         // units == 0: whole tiles only
    int Kb, G, slots, RT, CT;   // G: workgroups, 0 if the launch would be too large
    int threads;               // of a workgroup
    unsigned whole;            // tiles dealt whole, ahead of the ranges
    unsigned wlast, tcost, tlast, cost, cost0;
};

// Relative duration of a unit in which `vb` of the four column blocks exist: a fixed part (copy, barrier,
// LDS reads) plus one part per column block.  Measured on MI355X: 3.1 us for a full unit, 1.55 us with one
// column block.
inline unsigned unit_cost(int vb)
{
    static const unsigned w[5] = {0, 9, 12, 15, SS_UNIT_COST};
    return w[vb];
}

// A further plane of the output is written here and read by whoever takes the product: bytes that take as long as a cost
// of one (0.15 us, over the 45-bit prime 0.085 us, at 5 TB/s, what many streams at a time reach).  Over the 45-bit prime, at 750 KB ->
// at 425 KB, product and reduction, us: n = 5, 269 x 579 x 3245 107.9 -> 96.4; n = 3, 320 x 1800 x 576 56.6 -> 52.9 (as a tensor 43.7 ->
// 33.0); n = 4, 52 x 3468 x 1152 45.4 -> 40.2; of 60 drawn shapes whose plan differs all but nine gain, these lose up to 4 %.
constexpr unsigned long long SS_BYTES_PER_COST = SS_NLIMB == 8 ? 750 * 1000 : 425 * 1000;

// Plan for gemm_ksplit_kernel and what it takes, in units (16 x 16, one k block, four side by side on a CU): a CU's waves get
// their operand blocks out of the caches, 64 KB (48 KB over the 45-bit prime) per unit in about 0.83 us (0.46 us), so a launch lasts as
// long as the fullest CU has units.
inline gemm_plan plan_ksplit(int n, int rows, int cols, int Kb, double *busy, double *spread)
{
    gemm_plan best = {};
    const long Rb = (rows + 15) / 16, Cb = (cols + 15) / 16, blocks = n * Rb * Cb;
    best.Kb = Kb;
    best.RT = (int)(Rb < Cb ? Cb : Rb);
    best.CT = (int)(Rb < Cb ? Rb : Cb);
    best.tiles = best.units = blocks;
    if (blocks >= (1L << 28)) return best;   // (refused by the caller: busy stays)
    for (int ks = 1; ks <= 8 && (ks == 1 || ks <= Kb); ks *= 2) {
        const int cw = ks == 8 ? 1 : 4 / ks, fours = ks == 8 ? 2 : 1;   // tiles, and groups of four waves, of a workgroup
        const long groups = (blocks + cw - 1) / cw;
        int parts = 1;
        // CUs left over: k blocks in parts, as long as every wave keeps two units
        while (ks == 8 && (parts + 1) * groups <= SS_GEMM_CUS && Kb >= 16 * (parts + 1)) parts++;
        const long wgs = groups * parts, units = (Kb + ks * parts - 1) / (ks * parts);
        const int threads = ks == 8 ? 512 : 256;
        // (a convolution of a few channels with a wide padding has that many tiles of 16 x 16 in a few gigabytes)
        if (!fits_grid(wgs, threads)) continue;
        // workgroups of four that the fullest CU runs; over many rounds they even out
        const double fullest = wgs <= 2 * SS_GEMM_CUS ? (double)((wgs + SS_GEMM_CUS - 1) / SS_GEMM_CUS * fours)
                                                      : (double)wgs / SS_GEMM_CUS * fours + 0.3 * fours;
        // (a lone wave on a SIMD waits for its operands a little; half a unit for a wave's fold and start)
        const double cost = fullest * ((fullest == 1 ? 1.15 : 1.0) * units + 0.5);
        if (best.G == 0 || cost < *busy) {
            *busy = cost;
            *spread = (double)wgs / SS_GEMM_CUS * fours * (units + 0.5);   // a CU's share of the whole launch
            best.ksplit = ks;
            best.slots = parts;
            best.threads = threads;
            best.G = (int)wgs;
        }
    }
    return best;
}

// gemm_ksplit_kernel (plan k; busy, spread: see plan_ksplit) takes over from gemm_limb_kernel (plan p; big: the cost of its busiest
// workgroup) where it is the faster one both with operands that repeat and with weights that come from memory.
//
// The same call repeated: 3.4 us and 0.88 us (0.53 us over the 45-bit prime) for each unit of its fullest CU; the big kernel 5.3 us and
// 0.15 us (8.5 and 0.085 us) for a cost of one of its busiest workgroup.  With a single k block the stores decide from some 2560
// tiles on.  Against the 16-row kernel, n = 5 / n = 3 / n = 3 over the 45-bit prime, us (rows x columns x contraction): 4 x 4096 x 512
// 16.7 -> 17.2 / 12.2 -> 11.4 / 9.3 -> 9.8; 1 x 1000 x 2048 17.3 -> 21.7 / 13.1 -> 13.2 / 10.0 -> 9.6.
//
// Weights from memory, product and reduction together, fitted to 1680 timings of both kernels (n = 3 to 7, both fields): 1 us per 20 MB
// of packed operands; a last row tile that is not full makes the big kernel's units shorter; 0.6 us and the loads of the consumer
// for every plane it leaves.  A convolution that reads limb planes with a stride finds the 16 pixels of a block in twice the
// cache lines or more, whose other halves belong to the next taps, all channels later: every tile of 16 x 16 pays for that by itself, the
// more the more channels, and the CUs together then wait for the caches (`spread`); a tile of 64 x 64 pays once for its four row
// blocks.
// Big kernel -> this one with weights from memory, product + reduction + truncation + opening, us, n = 5 / n = 3 / n = 3 over the 45-bit
// prime: taken, 64 x 128 x 256 (repeated, product alone) 9.3 -> 4.7 / 8.8 -> 4.5 / 8.1 -> 4.3; 128 x 784 x 512 30.3 -> 26.7 / 24.6 ->
// 20.7 / 24.8 -> 16.3; 1024 x 196 x 256 41.0 -> 39.0 / 31.0 -> 25.6 / 28.5 -> 20.2 (the product alone of five parties 20.0 -> 21.4: the
// reduction has one plane instead of two).  Left, 39 x 1800 x 4608, n = 5, 111 -> 118; 94 x 1352 x 2304, n = 3, 60.7 -> 68.5; with stride
// 2, 43 x 578 x 4608, n = 5, 51 -> 65; 270 x 80 x 4608, n = 5, 46 -> 56; 27 x 1152 x 4608, n = 4 over the 45-bit prime, 46 -> 51.
// (Timed before gemm_square_kernel, which takes products from both of them now, see plan_square: of the shapes here 128 x 784 x 512 but over the
// 45-bit prime, 1024 x 196 x 256 and 27 x 1152 x 4608.)
// us: the estimate for the kernel that is taken.
inline bool ksplit_is_faster(const gemm_plan &k, const gemm_plan &p, double busy, double spread, double big, bool all_whole, int n,
                             int rows, int cols, int gather, double *us)
{
    const long Rb = (rows + 15) / 16, packed = Rb + (gather ? 0 : (cols + 15) / 16);   // blocks of the packed operands
    const double operand_us = (double)n * packed * p.Kb * (SS_NLIMB << 10) / 20e6;
    const double plane_us = 0.62 + (double)n * rows * cols / p.tiles * (p.tiles - p.whole) * 8 / 5e6;
    const double unit = Rb == 4 * p.RT ? 1.0 : 0.86;
    const double big_us = (SS_NLIMB == 8 ? 6.0 + 0.145 * unit * big : 5.4 + 0.095 * unit * big) + (all_whole ? 0 : (p.slots - 1) * plane_us);
    *us = big_us;
    if (k.G <= 0 || k.tiles * k.Kb >= (1L << 31)) return false;
    if (p.skinny) return k.tiles * k.Kb <= 6144;
    if (k.Kb == 1 && k.tiles > (SS_NLIMB == 8 ? 2560 : 10240)) return false;
    if (SS_NLIMB == 8 ? busy * 5.87 >= big + 12.7 : busy * 6.2 >= big + 62) return false;
    double units = busy;
    if (gather > 1) {
        const double far = SS_NLIMB == 8 ? 0.05 + 0.20 * log2(gather / 64.0) : 0.10 + 0.20 * log2(gather / 64.0);
        // (four waves on neighbouring tiles share what they read of the pixels)
        const double held = (1 + (k.ksplit == 1 ? 0.25 : 1.0) * far) * spread;
        if (held > units) units = held;
    }
    // (waves of one tile share no operand)
    const double ksplit_us = operand_us + (k.ksplit >= 4 ? 1.13 : 1.0) * (SS_NLIMB == 8 ? 1.6 + 0.83 * units : 3.9 + 0.46 * units);
    if (ksplit_us < big_us) *us = ksplit_us;
    return ksplit_us < big_us;
}

// A second operand that gemm_skinny_kernel reads once and that the 256 MB of the last level cannot hold is read past it; one that
// they hold may be there from its last use.  The same call repeated, n = 5 / n = 3 / n = 3 over the 45-bit prime, us, through the
// caches -> past them (rows x columns x contraction): 2 x 12000 x 800 72.6 -> 63.9 (384 MB) / 36.2 -> 39.1 (230 MB) / 27.4 -> 29.9;
// 4 x 4096 x 4096 121 -> 116 / 72.6 -> 65.7 (402 MB) / 49.0 -> 48.8 (302 MB); 5 x 1200 x 4800 37.9 -> 39.7 (230 MB) / - / -.
inline bool streams_operand(size_t bytes) { return bytes > ((size_t)256 << 20); }

// How the units are dealt: one workgroup per CU unless there is too little work for that; slots = the most
// workgroups that can share one tile.
// Whole tiles first and the price of the planes, against every tile dealt by cost with two planes, MI355X: layers of eight
// images of ResNet-50 (n = 5) 16.12 -> 15.30 ms with their tails, 64 channels of 56 x 56 (3 x 3, n = 3, eight images) as a
// tensor 238 -> 227 us; whole tiles as workgroups of their own instead of runs of one workgroup per CU: 16 rounds of two
// units 125 us, in runs 107.
// gather: 0 for a second operand in tiles, 1 for one in limb planes; its channels if the convolution reads them with a stride.
// us: what the product, its operands from memory, and its further planes take.
inline gemm_plan plan_gemm(int n, int rows, int cols, int K, int gather, double *us = nullptr)
{
    typedef unsigned long long ull;
    gemm_plan p = {};
    p.Kb = (K + 63) / 64;
    p.threads = 512;
    p.skinny = gather == 0 && rows <= 16;
    p.CT = p.skinny ? (cols + SKINNY_COLS - 1) / SKINNY_COLS : (cols + 63) / 64;
    p.RT = p.skinny ? 1 : (rows + 63) / 64;
    p.tiles = (long)n * p.RT * p.CT;
    p.units = p.tiles * p.Kb;
    const int vb_last = p.skinny ? 4 : (cols + 15) / 16 - 4 * (p.CT - 1);
    p.wlast = unit_cost(vb_last);   // (every unit of the 16-row kernel copies the same nine blocks: one cost for all)
    p.tcost = (unsigned)p.Kb * SS_UNIT_COST + SS_FOLD_COST;
    p.tlast = (unsigned)p.Kb * p.wlast + (vb_last == 1 ? SS_FOLD_COST / 2 : SS_FOLD_COST);   // one block per wave to fold
    const ull rowcost = (ull)(p.CT - 1) * p.tcost + p.tlast, cost = (ull)(p.tiles / p.CT) * rowcost;
    // With one whole tile per workgroup the launch lasts as many tiles as the fullest CU gets.  Dealt by cost, a workgroup
    // is busy for its share plus the fold of the tile its range ends in, and the tiles that are dealt so have `slots`
    // planes.  With a single k block tiles are never cut, so there is nothing to choose; launches too large for the
    // 32-bit range arithmetic (and that of the consumers, ss_part_src) have tiles enough for every CU many times over.
    const unsigned step = SS_UNIT_COST + SS_FOLD_COST;   // largest distance between two unit starts
    ull busy = ~0ull;   // cost of the busiest workgroup
    bool all_whole = cost >= (1ull << 31) || p.units >= (1L << 31) || (ull)rows * cols >= (1ull << 31);
    if (!all_whole) {
        p.cost = (unsigned)cost;
        // every range must hold at least one unit start
        const unsigned most = p.cost / step;
        p.G = (int)(most < SS_GEMM_CUS ? (most ? most : 1) : SS_GEMM_CUS);
        // Tiles for two rounds and more: all but the last 256 to 511 of them whole, as long as that leaves the ranges longer than
        // a full tile and so two planes, as without; where ragged tiles leave them shorter, whole tiles are given up a round at a
        // time, all of them if need be.  (A workgroup whose whole tiles are ragged ones idles a little: rows of tiles are long
        // where there are that many.)
        if (!p.skinny && p.Kb > 1 && p.tiles >= 2 * SS_GEMM_CUS) {
            p.whole = (unsigned)(p.tiles / SS_GEMM_CUS) * SS_GEMM_CUS;
            do {
                p.whole -= SS_GEMM_CUS;
                p.cost0 = (unsigned)(p.whole / p.CT * rowcost + p.whole % p.CT * p.tcost);
            } while (p.whole && (p.cost - p.cost0) / p.G < p.tcost);
        }
        // a tile of cost <= tcost meets at most this many ranges of length >= share; ranges are cut between
        // units, so a tile of Kb units has at most Kb parts
        const unsigned share = (p.cost - p.cost0) / p.G;
        p.slots = (int)((p.tcost + share - 1) / share) + 1;
        if (p.slots > p.Kb) p.slots = p.Kb;
        busy = (ull)(p.whole / SS_GEMM_CUS) * p.tcost + share + SS_FOLD_COST;
        if (p.Kb > 1) {
            const ull plane_bytes = 16ull * n * rows * cols / p.tiles * (p.tiles - p.whole) * (p.slots - 1);
            const ull rounds = ((ull)p.tiles + SS_GEMM_CUS - 1) / SS_GEMM_CUS;
            all_whole = rounds * p.tcost <= busy + plane_bytes / SS_BYTES_PER_COST;
            if (all_whole) busy = rounds * p.tcost - SS_FOLD_COST;   // (5.3 us hold a fold)
        }
        double kbusy = 0, kspread = 0;
        const gemm_plan k = plan_ksplit(n, rows, cols, p.Kb, &kbusy, &kspread);
        if (p.CT == 1 && vb_last == 2) busy = busy * 7 / 8;   // (units of two column blocks cost less than dealt with)
        double estimate = 0;
        const bool ksplit = ksplit_is_faster(k, p, kbusy, kspread, (double)busy, all_whole, n, rows, cols, gather, &estimate);
        if (us) *us = estimate;
        if (ksplit) return k;
    }
    if (all_whole) {
        const long wgs = p.skinny || p.tiles < SS_GEMM_CUS ? p.tiles : SS_GEMM_CUS;
        const bool launchable = p.tiles < (1L << 30) && fits_grid(wgs, p.threads);   // else G = 0, rejected by the caller
        p.G = (int)(launchable ? wgs : 0);
        p.slots = 1;
        p.units = 0;
        p.whole = launchable ? (unsigned)p.tiles : 0;
        p.cost = p.cost0 = 0;
    }
    return p;
}

// gemm_square_kernel: a workgroup per tile of 32 x 32 and run of k blocks, `runs` runs of equal length with a plane each.  runs == 0: the
// product is left to the plan's kernels.
struct square_plan {
    int runs;
    unsigned minors, majors, G;   // tiles along the shorter and the longer side; workgroups
};
constexpr int SQUARE_RUNS = 8;

// Which products take it (p, p_us: what plan_gemm gives them to otherwise), and how many runs: where it is estimated 3 % faster than that.
// Over the 61-bit prime more is asked where tiles of 64 x 64 fill the matrix and the chip and are as fast or faster with half the reads: from
// tiles 15 % from 60 us on, from limb planes a margin that grows to 22 % between 40 and 60 us (128 x 6272 x 1152 from planes, n = 5, 191 -> 206 us,
// estimated 10 % faster; 256 x 1568 x 1024 89 -> 95; 384 x 338 x 2304, n = 3, 55.3 -> 58.6).  One round of whole tiles of 64 x 64 takes 15 % less than
// plan_gemm estimates, and here it leaves a second round of a few workgroups (64 x 3136 x 576 from planes, n = 5, 44.0 against 44.8; 690 x 441 x 576,
// n = 3, 36.8 against 38.9; 203 x 576 x 500 from tiles, n = 7, 62.6 against 64.0).  Eight waves on a long contraction from planes are
// faster than estimated too (66 x 256 x 6400, n = 3, 27.0 against 30.0).  Below 7 us (8.5 us) launches decide and nothing is gained (4000 shapes: 0.7 %
// slower on average).
// most: planes that there is room for; tensor: the planes are added up by one more launch, where there are several.
// A unit (32 x 32, one k block) keeps a CU busy for 0.605 us (0.365 us over the 45-bit prime), however many workgroups share the CU, down
// to two; less where blocks of the tile lie outside the matrix, more where it is gathered from limb planes.  Three (four)
// workgroups are on a CU at a time.
// Fitted to 10000 shapes, 62000 timings of product + reduction, operands from memory, n = 3 to 7, both fields, 10 us to 6 ms; the lines above set by
// 8000 others of up to 80 us of matrix work and 541 layers of ResNet, VGG and AlexNet at batch 1 to 8, weights from memory: 6 % faster on average over all of
// them, 3 % of those that are taken more than 3 % slower.  Before -> after, us, product + reduction + truncation (rows x columns x contraction, runs):
// n = 5, 128 x 784 x 1152 43.6 -> 37.4 (1), 256 x 196 x 1024 26.8 -> 25.1 (4), 512 x 49 x 2048 30.2 -> 25.6 (3), from planes 256 x 196 x 2304 42.7 -> 40.8
// (4) and 512 x 49 x 4608 46.6 -> 44.2 (3); product + layer tail, n = 3, 128 x 1024 x 1152 35.8 -> 30.5 (2); over the 45-bit prime 512 x 49 x 4608 30.1 -> 25.1
// (5), 256 x 196 x 2304 25.7 -> 21.9 (3).  Taken and slower: from planes read with stride 2, n = 5, 512 x 49 x 4608 45.1 -> 46.8 (3), 256 x 392 x 1152 44.8 -> 47.4 (3);
// n = 3, 196 x 196 x 1600 19.1 -> 21.6 (5); over the 45-bit prime, n = 3, 256 x 676 x 3456 63.7 -> 66.8 (3).  Large convolutions whose weights no L2 holds
// are left: there a tile of 64 x 64 reads them half as often (895 x 8712 x 3200, n = 3, 3.20 -> 3.55 ms).
inline square_plan plan_square(const gemm_plan &p, double p_us, int n, int rows, int cols, int K, int gather, bool tensor, int most)
{
    constexpr bool P61 = SS_NLIMB == 8;
    square_plan best = {};
    const long Rb = (rows + 15) / 16, Cb = ((long)cols + 15) / 16, Rt = (Rb + 1) / 2, Ct = (Cb + 1) / 2;
    const int Kb = (K + 63) / 64;
    if (p_us < (P61 ? 7.0 : 8.5) || p.G <= 0 || p.skinny || Rb < 2 || Cb < 2 || Rb > 0xffff || Cb > 0xffff || !fits_grid(n * Rt * Ct, 256)) return best;
    const double elements = (double)n * rows * cols, far = gather > 1 ? 1 + log2(gather / 64.0) : 0;
    if (gather && elements > 10e6 && (double)rows * K * SS_NLIMB > 12e6) return best;
    const double valid = (double)(Rb * Cb) / (4 * Rt * Ct);
    const double unit = (P61 ? 0.605 * (0.84 + 0.16 * valid) * (1 + 0.043 * far) : 0.365 * (0.86 + 0.14 * valid) * (1 + 0.054 * far)) *
                        (gather == 1 ? 1.06 : 1.0);
    const double plane = P61 ? 0.30 + elements * 3.5e-6 : 0.30 + elements * 4.7e-6;
    const double operands = (double)n * (Rb + (gather ? 0 : Cb)) * Kb * (SS_NLIMB << 10) * (P61 ? 0.032e-6 : 0.035e-6);
    const double add = tensor ? 3.5 + elements * 3.5e-6 : 0;   // (a launch, the first plane once more)
    const bool one_round = !p.ksplit && p.slots == 1 && p.tiles <= SS_GEMM_CUS;   // of whole tiles of 64 x 64
    const double other = p_us * (P61 && one_round ? 0.85 : 1) + (p.slots > 1 ? add * (p.tiles - p.whole) / p.tiles : 0);
    double margin = 1.03;
    if (P61 && gather) margin += 0.19 * fmin(fmax((p_us - 40) / 20, 0.0), 1.0);
    else if (P61 && p_us > 60) margin = 1.15;
    if (P61 && gather && p.ksplit == 8 && Kb >= 64) margin *= 1.15;
    double best_us = other / margin;
    for (int runs = 1; runs <= SQUARE_RUNS && runs <= Kb && runs <= most; runs++) {
        const long G = n * Rt * Ct * runs;
        if (!fits_grid(G, 256)) break;
        const double at_a_time = P61 ? 3 : 4, per_cu = (double)G / SS_GEMM_CUS, rounds = per_cu / at_a_time;
        const double share = per_cu > at_a_time ? per_cu + 0.58 : per_cu > 3 ? 3.8 : per_cu > 2 ? 2.95 : per_cu > 1 ? 2 : P61 ? 1.27 : 1.62;
        // (from the second round on a workgroup's start hides behind the others)
        const double us = (P61 ? 2.4 : 3.7) + (Kb + runs - 1) / runs * unit * share - (P61 ? 1.45 : 2.1) * fmin(fmax(rounds - 1, 0.0), 6.5) +
                          (runs - 1) * plane + operands + (runs > 1 ? add : 0);
        if (us < best_us) {
            best_us = us;
            best = {runs, (unsigned)(Rt < Ct ? Rt : Ct), (unsigned)(Rt < Ct ? Ct : Rt), (unsigned)G};
        }
    }
    return best;
}

// What a product is launched with: gemm_square_kernel where sq.runs > 0, else the plan's kernel.  room: planes that there is memory for,
// plan_gemm's or more; 0: as many as plan_gemm has.
struct product_plan {
    gemm_plan p;
    square_plan sq;
    int planes() const { return sq.runs ? sq.runs : p.slots; }
    // Waves that share a tile where gemm_ksplit_kernel takes its column operand as field elements, without the launch that would pack them; 0:
    // it does not.  The digits of a unit take a wave longer than its products, so that a wave has one unit and the launch few enough waves for
    // all to run at once.  Both kernels -> this one, us, without the 1.5 to 2 us between the two (n = 3): 1 x 120 x 400 7.6 -> 6.1, 16 x 120 x 100 6.9 ->
    // 5.5, 64 x 300 x 180 7.9 -> 6.9, 64 channels of 32 x 32 from three 7.1 -> 6.8; left, with two units and more, 16 x 500 x 1000 9.2 -> 11.1,
    // 200 channels of 14 x 14 from twenty, four images, 13.7 -> 16.3.  input_rows: of a dense input (0: images), whose loads meet a cache line per
    // row: 16 x 1000 x 512 8.5 -> 11.7 us, 16 x 120 x 400 8.0 -> 7.9.
    int element_waves(int input_rows) const
    {
        if (sq.runs || !p.ksplit || p.Kb > 8) return 0;
        const int ks = p.Kb > 4 ? 8 : p.Kb > 2 ? 4 : p.Kb;
        return p.tiles * ks * (ks == 8 && input_rows > 8 ? 3 : 1) <= 8 * SS_GEMM_CUS ? ks : 0;
    }
    product_plan for_elements(int waves) const
    {
        product_plan e = *this;
        e.p.ksplit = waves;
        e.p.slots = 1;
        e.p.threads = e.p.ksplit == 8 ? 512 : 256;
        const int cw = e.p.ksplit == 8 ? 1 : 4 / e.p.ksplit;
        e.p.G = (int)((p.tiles + cw - 1) / cw);
        return e;
    }
};

inline product_plan plan_product(int n, int rows, int cols, int K, int gather, bool tensor, int room)
{
    product_plan r = {};
    double us = 0;
    r.p = plan_gemm(n, rows, cols, K, gather, &us);
    if (us > 0) r.sq = plan_square(r.p, us, n, rows, cols, K, gather, tensor, room > r.p.slots ? room : r.p.slots);
    return r;
}

}  // namespace
