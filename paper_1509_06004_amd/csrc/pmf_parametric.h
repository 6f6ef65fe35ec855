// Kernels of the breakpoint searches (pmf_parametric, pmf_breakpoints): set
// statistics and exit maps of the integer search; for the real-lambda search,
// graph contraction of the pixels that leave the minimal source set inside
// one unit lambda interval, scaling of a contracted problem to a rational
// lambda, and the per-pixel exit bookkeeping.
#pragma once

#include <stdint.h>

namespace pmf {

constexpr int kProbeMasks = 64;  // masks or probes of one launch (tables passed by value)

// The nested sets of ascending lambdas, row-major masks of n pixels.
struct MaskTable {
    const uint8_t *mask[kProbeMasks];
    int32_t lam[kProbeMasks];
    int32_t count;
};

// out[2 (l - 1)] += the pixels that exactly the first l sets hold and
// out[2 (l - 1) + 1] += the sink slopes of the free ones, l = 1 .. count (out
// zeroed by the caller): set i has the sums of the levels above i.
// exit (may be null): exit[p] = min(exit[p], the first lambda whose set lacks p).
int launch_level_stats(const MaskTable &t, int n, const int32_t *slope, const uint8_t *seed, int64_t *out,
                       int32_t *exit, void *stream);

// out[p] = v (n pixels).
int launch_fill_i32(int32_t *out, int n, int32_t v, void *stream);

// One unit lambda interval (c - 1, c] with changing pixels and their box.
struct Interval {
    int32_t *planes, *ep, *eq;
    int32_t c, x0, y0, w, h;
    int32_t first, count;  // launch_exit_place: its breakpoints
};

// The intervals of one launch.
struct IntervalTable {
    Interval iv[kProbeMasks];
};

// Per-interval statistics written by launch_contract (int64 each).
enum ContractStat : int {
    kCsD = 0,    // pixels of D
    kCsSumCs,    // sum over D of the contracted source capacity
    kCsSumC0,    // sum over D of the contracted sink capacity at lambda 0
    kCsSumSl,    // sum over D of the sink slope
    kCsMaxCs,    // largest contracted source capacity in D
    kCsMaxC0,    // largest contracted sink capacity at lambda 0 in D
    kCsMaxNl,    // largest n-link between two pixels of D
    kCsMaxSl,    // largest sink slope in D
    kCsSeeds,    // seed pixels in D (0 unless capacities reach INF)
    kCsCount
};
constexpr int kCsStride = 32;  // int64 from interval to interval

// boxes[4 i .. 4 i + 3] = {x_min, y_min, x_max, y_max} of the pixels p with
// exit[p] == changes[i] (changes: k ascending values; W x H exit map).
int launch_change_boxes(const int32_t *exit, int W, int H, const int32_t *changes, int k, int32_t *boxes,
                        void *stream);

// Contract the problem (nlink, cap_src, cap_snk0, slope, seed: a W x H
// instance with K-connectivity) to each interval's D = {p : exit[p] == c},
// cropped to the box (x0, y0, w, h, at most n_max pixels) that holds D.  With
// S1 = {exit >= c} and S2 = {exit > c} the pixels of S2 are merged into the
// source and those outside S1 into the sink: a pixel of D gets source capacity
// cs + the n-links into it from S2 and sink capacity at lambda 0 c0 + its
// n-links into pixels outside S1; the n-links between pixels of D stay, every
// other capacity of the box is 0.
// planes: int32 [K + 3][h][w] = n-links (K planes), cs, c0, slope; ep / eq:
// int32 [h][w] exit value c / 1 on D, -1 / 1 elsewhere; stats: int64
// [count][kCsStride], zeroed here before the kernel adds to it.
int launch_contract(const IntervalTable &t, int count, int n_max, const int32_t *nlink, const int32_t *cap_src,
                    const int32_t *cap_snk0, const int32_t *slope, const uint8_t *seed, int W, int H, int K,
                    const int32_t *exit, int64_t *stats, void *stream);

// One probe of a contracted problem: lambda = p / q, n pixels of its box.
struct Probe {
    const int32_t *planes;  // launch_contract's
    int32_t *ep, *eq;
    const uint8_t *mask;  // its minimal source set once solved
    int32_t n, p, q;
};

// A round's probes; probes [run[i], run[i + 1]) belong to one interval.
struct ProbeTable {
    Probe probe[kProbeMasks];
    int32_t run[kProbeMasks + 1];
};

// out + j * stride = the first `planes` planes of probe j times its q, for
// count probes of at most n_max pixels (the caller has checked that no
// product leaves int32).
int launch_scale(const ProbeTable &t, int count, int n_max, int planes, int32_t *out, size_t stride, void *stream);

// For every probe j of `runs` runs: out[j] += the slopes (plane `planes` of
// its planes) of the pixels its mask holds, and for each pixel with ep >= 0
// that it does not hold ep / eq = min(ep / eq, p / q) (exact: cross-multiplied
// in int64).
int launch_probe_sets(const ProbeTable &t, int runs, int n_max, int planes, int64_t *out, void *stream);

// exit[p] (n pixels): lo -> 0, hi + 1 -> last, any other value -> -1.
int launch_exit_pieces_init(int32_t *exit, int n, int32_t lo, int32_t hi, int32_t last, void *stream);

// For each pixel of an interval's box with ep >= 0: the index j of ep / eq
// among its ascending breakpoints (bp: int64 pairs num, den of breakpoints
// first, first + 1, ...), and exit[y * W + x] = Interval::first + j + 1 (-2 if
// absent).
int launch_exit_place(const IntervalTable &t, int count, int n_max, int W, const int64_t *bp, int32_t first,
                      int32_t *exit, void *stream);

}  // namespace pmf
