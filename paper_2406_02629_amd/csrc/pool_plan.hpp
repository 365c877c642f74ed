// How ReLU with pooling is cut into runs for its one-launch kernel, or given to the two launches.  Plain C++, so that
// the rule and the cut can be checked without a GPU; constexpr functions may be called from kernels.
#pragma once
#include <stddef.h>

// Output rows oh0..oh1-1 of one plane, pooled by one workgroup from the input rows row0..need1-1; the workgroup writes
// the messages of the rows row0..own1-1.  Rows that the next run's kernels share with this one's are opened by both.
struct ss_pool_rows {
    int oh0, oh1, row0, own1, need1;
};

constexpr ss_pool_rows ss_pool_cut(int s, int strips, int R, int H, int kh, int sh, int ph, int Ho)
{
    const int oh0 = s * R, oh1 = oh0 + R < Ho ? oh0 + R : Ho;
    const int first = oh0 * sh - ph, end = (oh1 - 1) * sh - ph + kh;
    const int next = s == strips - 1 ? H : oh1 * sh - ph;   // first row of the next run
    return {oh0, oh1, s == 0 || first < 0 ? 0 : first, next < 0 ? 0 : next, end < H ? end : H};
}

// Most LDS that a run may take (what a launch gets without asking for more): kernels of up to 8192 elements in all
// their full rows.
constexpr size_t SS_POOL_LDS_BYTES = 64 * 1024;

struct ss_pool_plan {
    bool one_launch;
    int P;               // whole planes per run (strips == 1)
    int R, strips;       // output rows per run, runs per plane
    int threads;
    size_t blocks, lds;  // lds: bytes of a run's rectified values
};

// out_in_mask: the output lies in memory of d_beta that the call reads.  The workgroups of the one-launch kernel write
// their output while others still read the mask; of the two launches the second writes after the first has read it.
inline ss_pool_plan ss_plan_pool(size_t planes, int H, int W, int kh, int sh, int Ho, bool out_in_mask)
{
    // A run is about as many elements as the workgroup has threads: longer ones are slower (2 x 2 on 1024 planes of 64 x 64,
    // n = 5: 115 us with runs of 256, 147 us with 1024; 118 us in two launches).  Kernels that overlap make it longer, until
    // at most one row in eight is opened twice, as far as there are enough output rows for four workgroups per CU.  (These
    // lines and the next ones stand on the shapes named, all n = 5, the same call repeated.)
    const size_t target = 256, enough = 1024, plane = (size_t)H * W, cin = planes * plane;
    ss_pool_plan p = {true, 1, Ho, 1, 256, 0, 0};
    if (plane <= target) {
        p.P = (int)(target / plane);
    } else {
        const size_t rows = target / W;   // input rows of a run
        p.R = rows > (size_t)kh ? (int)((rows - kh) / sh + 1) : 1;
        if (kh > sh) {
            const size_t most = planes * Ho / enough, eighth = (8 * (kh - sh) + sh - 1) / sh;
            const int longer = (int)(eighth < most ? eighth : most);
            if (longer > p.R) p.R = longer;
        }
        if (p.R > Ho) p.R = Ho;
        p.strips = (Ho + p.R - 1) / p.R;
        if (p.strips == 1) p.R = Ho;
    }
    const size_t run = p.strips == 1 ? p.P * plane : (size_t)((p.R - 1) * sh + kh) * W;
    p.lds = run * 8;
    p.blocks = p.strips == 1 ? (planes + p.P - 1) / p.P : planes * p.strips;
    p.threads = run > 256 && run <= 512 ? 512 : 256;   // one pass over the run if it takes twice the threads
    // few wide planes under overlapping kernels would open half their rows twice (4 planes of 400 x 400, 3 x 3 / 2: 23.8
    // against 21.5 us in two launches); below 256 K elements the launch saved is worth more (16 of 112 x 112: 9.6, 10.6 us)
    const bool twice = p.strips > 1 && 3 * (kh - sh) > p.R * sh && cin >= ((size_t)1 << 18);
    // a launch holds less than 2^32 threads (a larger grid runs in part only), which runs shorter than their workgroup
    // reach before cin does
    p.one_launch = p.lds <= SS_POOL_LDS_BYTES && !twice && !out_in_mask && planes < ((size_t)1 << 31) &&
                   p.blocks * p.threads < ((size_t)1 << 32);
    return p;
}
