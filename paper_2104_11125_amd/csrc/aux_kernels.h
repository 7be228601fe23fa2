// Kernels beside the hot path: weight update on the index set (Alg. 1 lines 10, 12), similarity
// diagnostics (Sec. 2, Sec. 3), the copy yardstick.  Part of scalecom.hip's single translation unit.
#pragma once

#include <hip/hip_runtime.h>

#include "device_helpers.h"
#include "geometry.h"

namespace {

// Weight update on the index set (Alg. 1 lines 10 and 12): theta[idx[t]] -= scale * vals[t].
__global__ void __launch_bounds__(kBlock)
k_apply_update(float* __restrict__ theta, int64_t numel, const int32_t* __restrict__ idx, const float* __restrict__ vals,
               int64_t k, float neg_scale)
{
    const int64_t t = (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * kBlock + threadIdx.x;
    if (t >= k) return;
    const int32_t j = idx[t];
    if (j < 0 || j >= numel) return;                        // a position outside theta is skipped, never touched
    theta[j] = fmaf(neg_scale, vals[t], theta[j]);
}

// Similarity diagnostics (Sec. 3) --------------------------------------------------------------
// y[p] = sum over learners 0..n-1, left to right, of x_i[p] = fma(lr, grad_i[p], mem_i[p]): the
// all-reduced error-feedback gradient whose top-k is the "true top-k" (times n, which does not
// change the order of magnitudes).  Bound by the read of all (mem, grad): a block takes one wave tile, one wave per
// learner (the pattern that moves most bytes, see k_update) or, from ten learners on, per two of them (A), and adds the learners up
// through LDS.  us a call, A = 1 / 2: 16 x 20 M 746 / 604 (5.2 TB/s with blocks of 16 waves), 12 x 20 M 491 / 474, 64 x 4 M 424 / 421, but 8 x 25.6 M 415 / 419,
// 6 x 30 M 407 / 411.  At 8 x 25.6 M the kernel takes 281 us at best (6.2 TB/s; 299 on average over the 100 calls of another
// run); beside the 281: one thread per four positions and all learners 303, one per position 333, two tiles per block 304, four learners per wave 300, an
// eighth of the tiles per XCD 300.
// The first threads zero `clear_words` words from `clear_from` on the way: the selection's scratch
// zone, which the selection before this kernel has used and the one after it expects clean.
constexpr int kSumWaves = 16;                    // waves of a block at most: further learners take turns

template <typename G, int A>
__global__ void __launch_bounds__(kSumWaves * kLanes)
k_sum_x(const LearnerPtrs lp, int n_learners, float lr, int64_t begin, int64_t end, int64_t n_tiles, float* __restrict__ y,
        uint32_t* __restrict__ clear_from, size_t clear_words)
{
    extern __shared__ float4 sum_lds[];                     // [learner][lane]
    const int64_t tile = static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;
    for (size_t i = static_cast<size_t>(tile) * blockDim.x + threadIdx.x; i < clear_words;
         i += static_cast<size_t>(gridDim.x) * gridDim.y * blockDim.x)
        clear_from[i] = 0u;
    if (tile >= n_tiles) return;                            // whole block
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes), lane = threadIdx.x % kLanes;
    const int waves = static_cast<int>(blockDim.x) / kLanes;
    const int64_t p0 = (begin & ~static_cast<int64_t>(kVec - 1)) + tile * kWaveTile + lane * kVec;
    const bool full = p0 >= begin && p0 + 3 < end;
    for (int i0 = wave; i0 < n_learners; i0 += A * waves) {
        float4 m[A], g[A];
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int i = i0 + a * waves < n_learners ? i0 + a * waves : i0;   // (the last turn's second learner may be the first again)
            if (full) {
                m[a] = load4(lp.mem[i] + p0);
                g[a] = load4(static_cast<const G*>(lp.grad[i]) + p0);
            } else {
                leader_load(lp.mem[i], static_cast<const G*>(lp.grad[i]), p0, begin, end, m[a], g[a]);
            }
        }
#pragma unroll
        for (int a = 0; a < A; ++a)
            if (i0 + a * waves < n_learners) sum_lds[(i0 + a * waves) * kLanes + lane] = accumulate4(m[a], g[a], lr);
    }
    __syncthreads();
    if (wave != 0 || p0 >= end) return;
    float4 acc = sum_lds[lane];
    for (int i = 1; i < n_learners; ++i) {
        const float4 x = sum_lds[i * kLanes + lane];
        acc.x += x.x;
        acc.y += x.y;
        acc.z += x.z;
        acc.w += x.w;
    }
    if (full)                                               // (kept in the caches: the selection that follows reads it)
        *reinterpret_cast<float4*>(y + p0) = acc;
    else
        store_guarded(y, p0, begin, end, false, acc);
}

// What the diagnostic's two selections start from, per tensor: d = k; for the leader's vector the prediction
// that the steps keep, if they have one for the route this call takes (`is_short`; the learner count decides, so steps and
// diagnostics on one layout may go different ways), otherwise what this diagnostic's last call left.  (The steps' own
// predictions are only read.)
__global__ void __launch_bounds__(kBlock)
k_diag_begin(const SegDesc* __restrict__ segs, int n_tensors, const uint32_t* __restrict__ preds,
             const uint32_t* __restrict__ lead_mine, uint32_t* __restrict__ diag_preds, uint32_t* __restrict__ diag_lead,
             int32_t* __restrict__ d, bool is_short)
{
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= n_tensors) return;
    d[s] = segs[s].k;
    const uint32_t* src = preds + static_cast<size_t>(s) * kPredWords;
    if (src[is_short ? kPredShortWidth : 0] == 0u) return;
    for (int j = 0; j < kPredWords; ++j) diag_preds[static_cast<size_t>(s) * kPredWords + j] = src[j];
    diag_lead[s] = lead_mine[s];
}

// d[seg] -= |A and B| over the membership masks of two selections: with d preset to k, what is
// left is the number of positions of one index set that the other one lacks (Eq. 6: the binarised
// vectors differ in 2d places).  A wave takes consecutive supertiles, and a block adds its waves up where they end
// in the same segment: an atomic per supertile on the one word of a flat vector took 37 us at 25.6 M.
// Zeroes the scratch zone as k_sum_x does.
constexpr int kOverlapBlocks = 256;

__global__ void __launch_bounds__(kBlock)
k_mask_overlap(const StDesc* __restrict__ sts, int n_st, const uint64_t* __restrict__ mask_a,
               const uint64_t* __restrict__ mask_b, int32_t* __restrict__ d, uint32_t* __restrict__ clear_from, size_t clear_words)
{
    for (size_t i = blockIdx.x * static_cast<size_t>(kBlock) + threadIdx.x; i < clear_words;
         i += static_cast<size_t>(gridDim.x) * kBlock)
        clear_from[i] = 0u;
    const int lane = threadIdx.x % kLanes, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const int64_t n_waves = static_cast<int64_t>(gridDim.x) * kWaves, w_id = static_cast<int64_t>(blockIdx.x) * kWaves + wave;
    const int lo = static_cast<int>(n_st * w_id / n_waves), hi = static_cast<int>(n_st * (w_id + 1) / n_waves);
    static_assert(kTilesPerSuper * 4 == 2 * kLanes, "one 16-byte access per lane and supertile");
    int seg = -1;
    uint32_t both = 0;                                      // this lane's share of the members of both in `seg`
    auto flush = [&]() {
        const uint32_t n = wave_sum(both);
        if (lane == 0 && n) atomicSub(&d[seg], static_cast<int32_t>(n));
        both = 0;
    };
    for (int st = lo; st < hi; ++st) {
        const int here = sts[st].seg;
        const ulonglong2 a = reinterpret_cast<const ulonglong2*>(mask_a + static_cast<size_t>(st) * kTilesPerSuper * 4)[lane];
        const ulonglong2 b = reinterpret_cast<const ulonglong2*>(mask_b + static_cast<size_t>(st) * kTilesPerSuper * 4)[lane];
        if (here != seg) {                                  // wave-uniform
            if (seg >= 0) flush();
            seg = here;
        }
        both += __popcll(a.x & b.x) + __popcll(a.y & b.y);
    }
    __shared__ uint32_t part[kWaves];
    __shared__ int part_seg[kWaves];
    const uint32_t n = wave_sum(both);
    if (lane == 0) {
        part[wave] = n;
        part_seg[wave] = seg;
    }
    __syncthreads();
    if (threadIdx.x < kWaves && part_seg[threadIdx.x] >= 0) {
        // the first of the block's waves that ended in this segment adds them all up
        uint32_t sum = 0;
        for (int w = 0; w < kWaves; ++w) {
            if (part_seg[w] != part_seg[threadIdx.x]) continue;
            if (w < static_cast<int>(threadIdx.x)) return;
            sum += part[w];
        }
        if (sum) atomicSub(&d[part_seg[threadIdx.x]], static_cast<int32_t>(sum));
    }
}

// Partial sums of a.b, a.a and b.b in binary64, three per block.  Bound by the read of a and b: 16 bytes per
// access and thread with four accesses in flight, if both vectors start on 16 bytes (VEC); one element at a time
// took 57 us at 25.6 M, 3.6 TB/s.
constexpr int kDotsBlocks = 2048;

template <bool VEC>
__global__ void __launch_bounds__(kBlock)
k_dots(const float* __restrict__ a, const float* __restrict__ b, int64_t numel, double* __restrict__ partial)
{
    double ab = 0.0, aa = 0.0, bb = 0.0;
    auto add = [&](float fx, float fy) {
        const double x = fx, y = fy;
        ab += x * y;
        aa += x * x;
        bb += y * y;
    };
    const int64_t t = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x, stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const int64_t groups = VEC ? numel / kVec : 0;
    if (VEC) {
        constexpr int kAhead = 2;
        int64_t g = t;
        for (; g + (kAhead - 1) * stride < groups; g += kAhead * stride) {
            float4 x[kAhead], y[kAhead];
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                x[j] = load4(a + (g + j * stride) * kVec);
                y[j] = load4(b + (g + j * stride) * kVec);
            }
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                add(x[j].x, y[j].x);
                add(x[j].y, y[j].y);
                add(x[j].z, y[j].z);
                add(x[j].w, y[j].w);
            }
        }
        for (; g < groups; g += stride) {
            const float4 x = load4(a + g * kVec), y = load4(b + g * kVec);
            add(x.x, y.x);
            add(x.y, y.y);
            add(x.z, y.z);
            add(x.w, y.w);
        }
    }
    for (int64_t j = groups * kVec + t; j < numel; j += stride) add(a[j], b[j]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        ab += __shfl_xor(ab, off, kLanes);
        aa += __shfl_xor(aa, off, kLanes);
        bb += __shfl_xor(bb, off, kLanes);
    }
    __shared__ double part[3][kWaves];
    if (threadIdx.x % kLanes == 0) {
        part[0][threadIdx.x / kLanes] = ab;
        part[1][threadIdx.x / kLanes] = aa;
        part[2][threadIdx.x / kLanes] = bb;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double s = 0.0;
        for (int w = 0; w < kWaves; ++w) s += part[threadIdx.x][w];
        partial[threadIdx.x * static_cast<size_t>(kDotsBlocks) + blockIdx.x] = s;
    }
}

// out[1..3] = the sums over n_blocks blocks, out[0] = 1 - a.b / (|a| |b|), by one block.
__global__ void __launch_bounds__(kBlock) k_cosine_final(const double* __restrict__ partial, int n_blocks, double* __restrict__ out)
{
    double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int j = 0; j < kDotsBlocks / kBlock; ++j) {
            const int i = j * kBlock + static_cast<int>(threadIdx.x);
            s[c] += i < n_blocks ? partial[c * static_cast<size_t>(kDotsBlocks) + i] : 0.0;
        }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s[c] += __shfl_xor(s[c], off, kLanes);
    __shared__ double part[3][kWaves];
    if (threadIdx.x % kLanes == 0)
        for (int c = 0; c < 3; ++c) part[c][threadIdx.x / kLanes] = s[c];
    __syncthreads();
    if (threadIdx.x != 0) return;
    double tot[3];
    for (int c = 0; c < 3; ++c) {
        tot[c] = 0.0;
        for (int w = 0; w < kWaves; ++w) tot[c] += part[c][w];
        out[1 + c] = tot[c];
    }
    out[0] = 1.0 - tot[0] / (sqrt(tot[1]) * sqrt(tot[2]));
}

// Plain streaming copy, one 16-byte nontemporal load and store per thread: the yardstick the
// other kernels' bandwidth and the profiler's byte counters are compared with.
__global__ void __launch_bounds__(kBlock) k_copy(const vf4_t* __restrict__ src, vf4_t* __restrict__ dst, size_t n16)
{
    const size_t i = (static_cast<size_t>(blockIdx.y) * gridDim.x + blockIdx.x) * kBlock + threadIdx.x;
    if (i < n16) __builtin_nontemporal_store(__builtin_nontemporal_load(&src[i]), &dst[i]);
}

}  // namespace
