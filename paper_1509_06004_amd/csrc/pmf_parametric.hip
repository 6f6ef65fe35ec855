// Kernels of the breakpoint searches: the sizes and slope sums of a round's
// minimal source sets and the running exit map of the integer search, and for
// the exact real-lambda search the contraction of a unit lambda interval's
// changing pixels (Sec. 2.1: the minimal source sets are nested in lambda, so
// between two nested sets the outer pixels are fixed to the sink and the
// inner ones to the source, as in the parametric algorithm of Gallo,
// Grigoriadis and Tarjan), scaling to a rational lambda, and the per-pixel
// exit bookkeeping.  All are one pass over the masks or boxes of a whole
// round, bound by memory latency; the reductions combine a wave's lanes by
// shuffles before any atomic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "pmf.h"
#include "pmf_border.h"
#include "pmf_parametric.h"

namespace pmf {

namespace {

constexpr int kBlock = 256;

inline int blocks(int64_t n) { return (int)((n + kBlock - 1) / kBlock); }

__global__ __launch_bounds__(kBlock) void k_fill_boxes(int32_t *boxes, int k) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < k) {
        boxes[4 * i] = INT_MAX;
        boxes[4 * i + 1] = INT_MAX;
        boxes[4 * i + 2] = -1;
        boxes[4 * i + 3] = -1;
    }
}

// A wave's lanes that hold pixels of the same change point combine their
// boxes by shuffles first (neighbouring pixels mostly leave together), so a
// change point of many pixels costs one set of atomics per wave, not per pixel.
__global__ __launch_bounds__(kBlock) void k_change_boxes(const int32_t *exit, int W, int n, const int32_t *changes,
                                                         int k, int32_t *boxes) {
    const int p = blockIdx.x * kBlock + threadIdx.x;
    int idx = -1;
    if (p < n) {
        const int32_t e = exit[p];
        int lo = 0, hi = k;  // first change >= e
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (changes[mid] < e)
                lo = mid + 1;
            else
                hi = mid;
        }
        if (lo < k && changes[lo] == e) idx = lo;
    }
    const int x = p % W, y = p / W, lane = (int)(threadIdx.x & 63);
    unsigned long long left = __ballot(idx >= 0);
    while (left) {  // wave-uniform
        const int leader = __ffsll((long long)left) - 1;
        const int li = __shfl(idx, leader);
        const bool mine = idx == li;
        int x0 = mine ? x : INT_MAX, y0 = mine ? y : INT_MAX, x1 = mine ? x : -1, y1 = mine ? y : -1;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            x0 = min(x0, __shfl_xor(x0, off));
            y0 = min(y0, __shfl_xor(y0, off));
            x1 = max(x1, __shfl_xor(x1, off));
            y1 = max(y1, __shfl_xor(y1, off));
        }
        if (lane == leader) {
            atomicMin(&boxes[4 * li], x0);
            atomicMin(&boxes[4 * li + 1], y0);
            atomicMax(&boxes[4 * li + 2], x1);
            atomicMax(&boxes[4 * li + 3], y1);
        }
        left &= ~__ballot(mine);
    }
}

// One pass over the nested masks of a round (ascending lambdas: each set holds
// the next) instead of two launches per mask.  A pixel's level is the number
// of sets that hold it, so the pixels and slopes are summed per level, in LDS
// first; the wave's lanes are combined level by level, which is one level for
// most waves.  Bound by the latency of the byte loads (many in flight per
// pixel), then by 256 workgroups' atomics per level: 28 masks of 500 x 375
// pixels take 16 us against 282 us in 56 launches, without their gaps.
__global__ __launch_bounds__(kBlock) void k_level_stats(MaskTable T, int n, const int32_t *slope, const uint8_t *seed,
                                                        unsigned long long *out, int32_t *exit) {
    __shared__ unsigned long long s_sum[2 * kProbeMasks];
    for (int i = threadIdx.x; i < 2 * T.count; i += kBlock) s_sum[i] = 0;
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63);
    for (int p0 = blockIdx.x * kBlock; p0 < n; p0 += gridDim.x * kBlock) {
        const int p = p0 + (int)threadIdx.x;
        int level = 0;
        if (p < n) {
#pragma unroll 8
            for (int i = 0; i < T.count; ++i) level += T.mask[i][p] != 0;
            if (exit && level < T.count) exit[p] = min(exit[p], T.lam[level]);
        }
        long long w = level > 0 && (!seed || seed[p] == 0) ? (slope ? slope[p] : 1) : 0;
        unsigned long long left = __ballot(level > 0);
        while (left) {
            const int leader = __ffsll((long long)left) - 1;
            const int lv = __shfl(level, leader);
            const unsigned long long mine = __ballot(level == lv);
            long long sum = level == lv ? w : 0;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
            if (lane == leader) {
                atomicAdd(&s_sum[2 * (lv - 1)], (unsigned long long)__popcll(mine));
                if (sum) atomicAdd(&s_sum[2 * (lv - 1) + 1], (unsigned long long)sum);
            }
            left &= ~mine;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * T.count; i += kBlock)
        if (s_sum[i]) atomicAdd(&out[i], s_sum[i]);
}

__global__ __launch_bounds__(kBlock) void k_fill_i32(int32_t *out, int n, int32_t v) {
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p < n) out[p] = v;
}

__global__ __launch_bounds__(kBlock) void k_zero_i64(int64_t *out, int n) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) out[i] = 0;
}

// One interval per grid row.  The statistics are combined in the wave before
// they reach LDS: nine atomics by every pixel serialised on nine addresses.
// The 30 intervals of a 320 x 240 image take 15 us in one launch, against 30
// launches of 16 us, each with a fill and a copy back of its own.
__global__ __launch_bounds__(kBlock) void k_contract(IntervalTable T, const int32_t *nlink, const int32_t *cap_src,
                                                     const int32_t *cap_snk0, const int32_t *slope,
                                                     const uint8_t *seed, int W, int H, int K, const int32_t *exit,
                                                     unsigned long long *stats) {
    __shared__ unsigned long long s[kCsCount];
    const Interval &I = T.iv[blockIdx.y];
    const int a = I.w * I.h, c = I.c;
    if ((int)blockIdx.x * kBlock >= a) return;  // the whole workgroup
    if (threadIdx.x < kCsCount) s[threadIdx.x] = 0;
    __syncthreads();
    int32_t *planes = I.planes, *ep = I.ep, *eq = I.eq;
    const int i = blockIdx.x * kBlock + threadIdx.x;
    unsigned long long v_st[kCsCount] = {};
    if (i < a) {
        const int x = I.x0 + i % I.w, y = I.y0 + i / I.w;
        const size_t n = (size_t)W * H, gp = (size_t)y * W + x;
        const bool in_d = exit[gp] == c;
        int64_t cs = 0, c0 = 0, sl = 0, mx_nl = 0;
        for (int k = 0; k < K; ++k) {
            int32_t v = 0;
            if (in_d) {
                // the arc p -> q (q = p + d_k): kept inside D, moved to the
                // sink capacity when q is outside S1, gone when q is in S2
                const int qx = x + DXk(k), qy = y + DYk(k);
                if (qx >= 0 && qy >= 0 && qx < W && qy < H) {
                    const int32_t eq_ = exit[(size_t)qy * W + qx];
                    const int32_t cap = nlink[(size_t)k * n + gp];
                    if (eq_ == c) {
                        v = cap;
                        mx_nl = cap > mx_nl ? cap : mx_nl;
                    } else if (eq_ < c) {
                        c0 += cap;
                    }
                }
                // the arc u -> p (u = p - d_k): moved to the source capacity
                // when u is in S2
                const int ux = x - DXk(k), uy = y - DYk(k);
                if (ux >= 0 && uy >= 0 && ux < W && uy < H) {
                    const size_t u = (size_t)uy * W + ux;
                    if (exit[u] > c) cs += nlink[(size_t)k * n + u];
                }
            }
            planes[(size_t)k * a + i] = v;
        }
        int32_t *pcs = planes + (size_t)K * a, *pc0 = pcs + a, *psl = pc0 + a;
        if (in_d) {
            cs += cap_src[gp];
            c0 += cap_snk0[gp];
            sl = slope ? slope[gp] : 1;
            const bool is_seed = seed && seed[gp] != 0;
            // sums stay far below 2^63; values above int32 are refused by the
            // caller from the maxima before any product is formed
            pcs[i] = cs > INT_MAX ? INT_MAX : (int32_t)cs;
            pc0[i] = c0 > INT_MAX ? INT_MAX : (int32_t)c0;
            psl[i] = (int32_t)sl;
            ep[i] = c;
            v_st[kCsD] = 1;
            v_st[kCsSumCs] = v_st[kCsMaxCs] = (unsigned long long)cs;
            v_st[kCsSumC0] = v_st[kCsMaxC0] = (unsigned long long)c0;
            v_st[kCsSumSl] = v_st[kCsMaxSl] = (unsigned long long)sl;
            v_st[kCsMaxNl] = (unsigned long long)mx_nl;
            v_st[kCsSeeds] = is_seed ? 1 : 0;
        } else {
            pcs[i] = 0;
            pc0[i] = 0;
            psl[i] = 0;
            ep[i] = -1;
        }
        eq[i] = 1;
    }
#pragma unroll
    for (int t = 0; t < kCsCount; ++t) {
        const bool top = t >= kCsMaxCs && t <= kCsMaxSl;
        unsigned long long v = v_st[t];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long o = __shfl_xor(v, off);
            v = top ? (o > v ? o : v) : v + o;
        }
        if ((threadIdx.x & 63) == 0 && v) {
            if (top)
                atomicMax(&s[t], v);
            else
                atomicAdd(&s[t], v);
        }
    }
    __syncthreads();
    if (threadIdx.x < kCsCount && s[threadIdx.x]) {
        const int t = threadIdx.x;
        stats += (size_t)blockIdx.y * kCsStride;
        if (t >= kCsMaxCs && t <= kCsMaxSl)
            atomicMax(&stats[t], s[t]);
        else
            atomicAdd(&stats[t], s[t]);
    }
}

// A round's probes, one per grid row: the contracted problem with every
// capacity multiplied by the probe's denominator.
__global__ __launch_bounds__(kBlock) void k_scale(ProbeTable T, int planes, int32_t *out, size_t stride) {
    const Probe &b = T.probe[blockIdx.y];
    const int64_t count = (int64_t)planes * b.n;
    int32_t *to = out + blockIdx.y * stride;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += (int64_t)gridDim.x * kBlock)
        to[i] = (int32_t)((int64_t)b.planes[i] * b.q);
}

// A round's solved probes, one grid row per run of probes of one interval
// (they share ep / eq, so one thread takes a pixel through all of them): each
// set's slope sum, and the pixels outside it exit at p / q at the latest.
__global__ __launch_bounds__(kBlock) void k_probe_sets(ProbeTable T, int planes, unsigned long long *out) {
    __shared__ long long s_w[kBlock / 64];
    const int wv = (int)(threadIdx.x >> 6);
    for (int j = T.run[blockIdx.y]; j < T.run[blockIdx.y + 1]; ++j) {
        const Probe &b = T.probe[j];
        const int32_t *slope = b.planes + (size_t)planes * b.n;
        long long w = 0;
        for (int i = blockIdx.x * kBlock + threadIdx.x; i < b.n; i += gridDim.x * kBlock) {
            if (b.mask[i]) {
                w += slope[i];
                continue;
            }
            const int32_t e = b.ep[i];
            if (e >= 0 && (int64_t)b.p * b.eq[i] < (int64_t)e * b.q) {
                b.ep[i] = b.p;
                b.eq[i] = b.q;
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) w += __shfl_xor(w, off);
        if ((threadIdx.x & 63) == 0) s_w[wv] = w;
        __syncthreads();
        if (threadIdx.x == 0) {
            long long tw = 0;
#pragma unroll
            for (int i = 0; i < kBlock / 64; ++i) tw += s_w[i];
            if (tw) atomicAdd(&out[j], (unsigned long long)tw);
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void k_exit_pieces_init(int32_t *exit, int n, int32_t lo, int32_t hi,
                                                             int32_t last) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int32_t v = exit[i];
    exit[i] = v == lo ? 0 : (int64_t)v == (int64_t)hi + 1 ? last : -1;
}

__global__ __launch_bounds__(kBlock) void k_exit_place(IntervalTable T, int W, const int64_t *table, int32_t first,
                                                       int32_t *exit) {
    const Interval &I = T.iv[blockIdx.y];
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= I.w * I.h || I.ep[i] < 0) return;
    const int64_t p = I.ep[i], q = I.eq[i];
    const int64_t *bp = table + 2 * (size_t)(I.first - first);
    const int nb = I.count;
    int lo = 0, hi = nb;  // first breakpoint >= p / q
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (bp[2 * mid] * q < p * bp[2 * mid + 1])
            lo = mid + 1;
        else
            hi = mid;
    }
    const bool hit = lo < nb && bp[2 * lo] * q == p * bp[2 * lo + 1];
    exit[(size_t)(I.y0 + i / I.w) * W + I.x0 + i % I.w] = hit ? I.first + lo + 1 : -2;
}

inline int launched() { return hipGetLastError() == hipSuccess ? 0 : -1; }

}  // namespace

int launch_level_stats(const MaskTable &t, int n, const int32_t *slope, const uint8_t *seed, int64_t *out,
                       int32_t *exit, void *stream) {
    if (t.count < 1 || t.count > kProbeMasks) return -1;
    hipLaunchKernelGGL(k_level_stats, dim3(std::min(blocks(n), 256)), dim3(kBlock), 0, (hipStream_t)stream, t, n,
                       slope, seed, (unsigned long long *)out, exit);
    return launched();
}

int launch_fill_i32(int32_t *out, int n, int32_t v, void *stream) {
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks(n)), dim3(kBlock), 0, (hipStream_t)stream, out, n, v);
    return launched();
}

int launch_change_boxes(const int32_t *exit, int W, int H, const int32_t *changes, int k, int32_t *boxes,
                        void *stream) {
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_fill_boxes, dim3(blocks(k)), dim3(kBlock), 0, s, boxes, k);
    hipLaunchKernelGGL(k_change_boxes, dim3(blocks((int64_t)W * H)), dim3(kBlock), 0, s, exit, W, W * H, changes, k,
                       boxes);
    return launched();
}

int launch_contract(const IntervalTable &t, int count, int n_max, const int32_t *nlink, const int32_t *cap_src,
                    const int32_t *cap_snk0, const int32_t *slope, const uint8_t *seed, int W, int H, int K,
                    const int32_t *exit, int64_t *stats, void *stream) {
    if (count < 1 || count > kProbeMasks) return -1;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_zero_i64, dim3(blocks(count * kCsStride)), dim3(kBlock), 0, s, stats, count * kCsStride);
    hipLaunchKernelGGL(k_contract, dim3(blocks(n_max), count), dim3(kBlock), 0, s, t, nlink, cap_src, cap_snk0, slope,
                       seed, W, H, K, exit, (unsigned long long *)stats);
    return launched();
}

int launch_scale(const ProbeTable &t, int count, int n_max, int planes, int32_t *out, size_t stride, void *stream) {
    if (count < 1 || count > kProbeMasks) return -1;
    hipLaunchKernelGGL(k_scale, dim3(std::min(blocks((int64_t)planes * n_max), 256), count), dim3(kBlock), 0,
                       (hipStream_t)stream, t, planes, out, stride);
    return launched();
}

int launch_probe_sets(const ProbeTable &t, int runs, int n_max, int planes, int64_t *out, void *stream) {
    if (runs < 1 || runs > kProbeMasks) return -1;
    hipLaunchKernelGGL(k_probe_sets, dim3(std::min(blocks(n_max), 256), runs), dim3(kBlock), 0, (hipStream_t)stream,
                       t, planes, (unsigned long long *)out);
    return launched();
}

int launch_exit_pieces_init(int32_t *exit, int n, int32_t lo, int32_t hi, int32_t last, void *stream) {
    hipLaunchKernelGGL(k_exit_pieces_init, dim3(blocks(n)), dim3(kBlock), 0, (hipStream_t)stream, exit, n, lo, hi,
                       last);
    return launched();
}

int launch_exit_place(const IntervalTable &t, int count, int n_max, int W, const int64_t *bp, int32_t first,
                      int32_t *exit, void *stream) {
    if (count < 1 || count > kProbeMasks) return -1;
    hipLaunchKernelGGL(k_exit_place, dim3(blocks(n_max), count), dim3(kBlock), 0, (hipStream_t)stream, t, W, bp, first,
                       exit);
    return launched();
}

}  // namespace pmf
