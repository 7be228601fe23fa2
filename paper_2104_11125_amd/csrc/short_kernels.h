// The exact step on short layouts (up to a few million positions), in two launches.
// Part of scalecom.hip's single translation unit.
#pragma once

#include <hip/hip_runtime.h>

#include "device_helpers.h"
#include "geometry.h"

namespace {

// What bounds a step on a short vector is launches and dependent trips to memory, not bytes: the
// chain of kernels for long vectors spends eight launches, one per level of the search, and most
// of their time is the way in and out of a kernel.  Here the search is done by every block for
// itself, from lists of keys that fit the caches:
//
//   k_short_collect  the leader's magnitude keys, one block per part (four consecutive positions per
//                    thread).  The part's keys go to its slice of the key array sorted into 61 columns:
//                    three above the threshold that the step expects, 48 narrow ones around it, ten
//                    below (without an expectation: around an estimate out of a sample of the segment).
//                    Zeros are only counted.  A row of running counts per column goes with it
//   k_short_step     every block adds up the rows of its segment: the column that holds the k-th largest
//                    key of the segment, whatever was expected.  That column of all parts, a few hundred
//                    keys as a rule, is searched by one wave; the columns above it and the members among
//                    those keys, in the parts before its own, give the block's first output slot.  Then the
//                    block updates its positions for all learners, sums its members' values and writes them
//
// No kernel reads what another block of the same launch wrote.  The price is that every block does the search: keys of
// the threshold's column beyond the first thousand are read by all blocks of the segment, several times (all keys of 2 M positions
// after a jump of the gradients by 64: 1.2 ms, where the long path takes 65 us).  So columns are kept small: the expectation is checked on a few
// keys before it is used (short_far_off), after a long search a sample takes its place until it would have held for a while (ShortTrust),
// columns that are crowded get narrower, and a part's keys of one column that are all equal count as one key with a weight (kShortEqual).
// A step of 2 x 2 M positions, us, against the long path: normal values 32 / 47, all magnitudes equal 36 / 121, two of them 71 / 154, a jump by
// 64 every third step 56 / 66, one jump 50 / 64 and the step after it 167 / 68.

constexpr int kShortCols = 64;                   // words of a row of running counts (16 bits each)
constexpr int kShortAbove = 3, kShortBins = 48;  // columns 0..2; 3..50 around the expected threshold, highest keys first
constexpr int kShortFirstBin = kShortAbove, kShortBelow = kShortAbove + kShortBins;   // 51..60: below
constexpr int kShortListed = 60;                 // running count of everything that is listed (all but zeros)
constexpr int kShortBulk = kShortListed - 1;     // the last two columns, where most keys are
constexpr int kShortValid = 61;                  // the part's positions inside the segment (not a running count)
constexpr int kShortEqual = 62;                  // two words, four bytes: columns whose keys are all equal, plus 1 (0: none)
constexpr int kShortSampleLog = 12;              // bins of the sample: the key's top twelve bits
constexpr int kShortGeneralLog = 11, kShortGeneral = 1 << kShortGeneralLog;   // bins of the general search
constexpr uint32_t kShortColumnMax = 1024;       // keys that one wave searches, 16 per lane
constexpr uint32_t kShortListMax = 256;          // keys of one bin that are ranked by comparing all pairs
constexpr uint32_t kShortWidthFirst = 12, kShortWidthMin = 2, kShortWidthMax = 15;   // log2 of the keys per narrow column
constexpr uint32_t kShortCalm = 8;               // steps with the threshold well inside before the columns get narrower

// The columns' lower ends: the narrow ones start at `base` and hold 2^w keys each, their span is 48 * 2^w.
// Above them a column of seven spans and one of two binades, then the rest (the index set's members, never
// many); below them, where magnitudes get denser, columns of 1/8, 1/8, 1/4, 1/4, 1/2, 1/2, 1 and 2 spans, one
// binade, then the rest.  At least 1: zeros are in no column.
struct ShortCols {
    uint32_t base, w;
    __device__ __forceinline__ ShortCols(uint32_t mid, uint32_t width) : w(width)
    {
        const uint32_t half = static_cast<uint32_t>(kShortBins / 2) << w;
        base = mid > half ? mid - half : 1u;
    }
    __device__ __forceinline__ uint32_t span() const { return static_cast<uint32_t>(kShortBins) << w; }
    __device__ __forceinline__ uint32_t low(uint32_t by) const { return base > by ? base - by : 1u; }
    // lower end of column kShortBelow + j, in eighths of the span below `base`: 1, 2, 4, 6, 10, 14, 22, 38
    __device__ __forceinline__ static constexpr uint32_t eighths(int j)
    {
        return j == 0 ? 1u : j == 1 ? 2u : j == 2 ? 4u : j == 3 ? 6u : j == 4 ? 10u : j == 5 ? 14u : j == 6 ? 22u : 38u;
    }
    __device__ __forceinline__ uint32_t end(int col) const   // the column's lower end
    {
        if (col == 0) return base + 8u * span() + (1u << 24);   // (below 2^31 + 2^26: no overflow)
        if (col == 1) return base + 8u * span();
        if (col < kShortBelow) return base + (static_cast<uint32_t>(kShortBelow - 1 - col) << w);   // column 2: base + span
        if (col >= kShortListed) return 1u;
        return low((span() / 8u) * eighths(col < kShortBulk ? col - kShortBelow : 7) + (col < kShortBulk ? 0u : 1u << 23));
    }
    __device__ __forceinline__ uint32_t column(uint32_t key) const   // of a key that is not 0
    {
        const uint32_t rel = key - base;
        if (key >= base)
            return rel < span() ? static_cast<uint32_t>(kShortBelow - 1) - (rel >> w)
                                : (key >= end(1) ? (key >= end(0) ? 0u : 1u) : 2u);
        uint32_t c = kShortBelow;
#pragma unroll
        for (int j = kShortBelow; j < kShortListed; ++j) c += key < end(j) ? 1u : 0u;
        return c;
    }
};
static_assert(kShortBelow + 8 == kShortBulk && kShortBulk + 1 == kShortListed && kShortListed < kShortValid &&
                  kShortValid < kShortEqual && kShortEqual % 2 == 0 && kShortEqual + 2 == kShortCols,
              "a row holds them all");

// What a segment's columns were laid around (the low two bits of word z of `used`; above them the trust as the step found it, which
// saves the step's first block a trip to memory).
constexpr uint32_t kShortNone = 0, kShortExpected = 1, kShortDoubted = 2;   // sample: nothing expected / expectation; sample: expectation not trusted

// How far a segment's expectation is trusted, packed into 24 bits: `count` steps in a row in which it held, or would have, of the
// 2^need that are asked for before it is used again (0: it is used), and a level that rises with every long search, so that searches by
// data that jump again and again get rarer (8 to 1024 steps), and falls in quiet times.  The sample costs 4 to 9 us a step, a long search
// 20 to 130.
struct ShortTrust {
    uint32_t count, need, level;
    __device__ __forceinline__ explicit ShortTrust(uint32_t w) : count(w & 0xffffu), need((w >> 16) & 0xfu), level((w >> 20) & 0xfu) {}
    __device__ __forceinline__ bool sampling() const { return need != 0u; }
    __device__ __forceinline__ uint32_t next(bool held, bool long_search)
    {
        if (!sampling() && !held && long_search) {
            level = level < 8u ? level + 1u : 8u;
            need = level + 2u;
            count = 0u;
        } else if (sampling()) {
            count = held ? count + 1u : 0u;
            if (count >> need) need = count = 0u;
        } else if (level != 0u && (++count >> (level + 4u)) != 0u) {
            --level;
            count = 0u;
        }
        return count | need << 16 | level << 20;
    }
};
constexpr uint32_t kShortLong = 8 * 1024;        // keys read by every block of a segment that make a search a long one

// The bin of h[0 .. NB) that holds the rem-th largest key counted there (rem >= 1), by all T
// threads of a block; wave_tot is T / 64 words of LDS.  The thread that owns the bin returns true.
template <int T, int NB>
__device__ __forceinline__ bool short_find_bin(const uint32_t* h, uint32_t rem, uint32_t* wave_tot, uint32_t& bin,
                                               uint32_t& n_bin, uint32_t& n_above)
{
    constexpr int CH = NB / T, W = T / kLanes;
    static_assert(CH % 2 == 0, "whole 8-byte reads");
    const int t = threadIdx.x, lane = t % kLanes, wave = t / kLanes;
    uint32_t c[CH];
    uint32_t mine = 0;
#pragma unroll
    for (int b = 0; b < CH; b += 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(h + t * CH + b);
        c[b] = v.x;
        c[b + 1] = v.y;
        mine += v.x + v.y;
    }
    uint32_t suf = mine;                                    // inclusive suffix sums over the threads
#pragma unroll
    for (int off = 1; off < kLanes; off <<= 1) {
        const uint32_t v = __shfl_down(suf, off, kLanes);
        if (lane + off < kLanes) suf += v;
    }
    if (lane == 0) wave_tot[wave] = suf;
    __syncthreads();
    for (int w = wave + 1; w < W; ++w) suf += wave_tot[w];
    uint32_t above = suf - mine;                            // keys in higher threads' bins
    if (!(above < rem && rem <= suf)) return false;
    bool found = false;
#pragma unroll
    for (int b = CH - 1; b >= 0; --b) {
        if (!found && above + c[b] >= rem) {
            bin = static_cast<uint32_t>(t * CH + b);
            n_bin = c[b];
            n_above = above;
            found = true;
        }
        above += found ? 0u : c[b];
    }
    return found;
}

// The expectation of a segment that has none: an estimate of its k-th largest key from a sample of T
// groups of four positions at equal distances (every group, if there are no more), every block of the
// segment for itself.  Only an estimate: it decides how many keys have to be searched.
template <typename G, int T>
__device__ __forceinline__ uint32_t short_sample(const float* __restrict__ mem, const G* __restrict__ grad, float lr,
                                                 const PartDesc& d, uint32_t* hist, uint32_t* wave_tot, uint32_t* res)
{
    const int t = threadIdx.x;
    const int64_t begin = d.begin, end = d.end, first = begin & ~static_cast<int64_t>(kVec - 1);
    const int64_t groups = (end - first + kVec - 1) / kVec;
    constexpr int NB = 1 << kShortSampleLog;
    for (int b = t; b < NB; b += T) hist[b] = 0u;
    if (t == 0) res[0] = res[1] = 0u;
    __syncthreads();
    const int64_t g = groups <= T ? t : groups * t / T;
    uint32_t n_ok = 0;
    if (g < groups) {
        uint32_t key[4];
        bool ok[4];
        leader_keys<true>(mem, grad, lr, first + g * kVec, begin, end, key, ok);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (!ok[c]) continue;
            ++n_ok;
            atomicAdd(&hist[key[c] >> (31 - kShortSampleLog)], 1u);
        }
    }
    n_ok = wave_sum(n_ok);
    if (t % kLanes == 0) atomicAdd(&res[1], n_ok);
    __syncthreads();
    const uint32_t sampled = res[1];
    const uint64_t len = static_cast<uint64_t>(end - begin);
    const uint64_t rank = static_cast<uint64_t>(d.k) * sampled / len + 1;
    uint32_t bin, n_bin, n_above;
    if (short_find_bin<T, NB>(hist, rank < sampled ? static_cast<uint32_t>(rank) : sampled, wave_tot, bin, n_bin, n_above))
        res[0] = (bin << (31 - kShortSampleLog)) + (1u << (30 - kShortSampleLog));   // the middle of the bin
    __syncthreads();
    return res[0];
}

// Is the expectation far off?  Every wave looks at the same 16 groups of four positions, one in each of 16 equal stretches of the
// segment (at equal distances they would share a memory channel), so all waves of all blocks come to the same answer without a word
// between them.  Far off: many more of the 64 keys above the near columns than the index set's share, or hardly any down to the
// end of column kShortBulk, where the last step had `below`.  m, g: every group in four lanes.  Costs 0.3 us a step.
constexpr int kShortCheckGroups = 16, kShortCheckParts = 32;  // (segments of few parts do without: a long column is read by few blocks)

__device__ __forceinline__ bool short_far_off(const float4& m, const float4& g, float lr, const PartDesc& d, const ShortCols& cols,
                                              uint32_t below)
{
    const float4 x = accumulate4(m, g, lr);
    const uint32_t key[4] = {magnitude_key(x.x), magnitude_key(x.y), magnitude_key(x.z), magnitude_key(x.w)};
    const uint32_t high = cols.end(1), low = cols.end(kShortBulk);
    uint32_t above = 0, near = 0;                           // four times as many: every key is in four lanes
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        above += __popcll(__builtin_amdgcn_ballot_w64(key[c] >= high));
        near += __popcll(__builtin_amdgcn_ballot_w64(key[c] >= low));
    }
    const float share = 64.0f * static_cast<float>(d.k) * __builtin_amdgcn_rcpf(static_cast<float>(d.end - d.begin));
    return static_cast<float>(above) > 4.0f * (2.0f * share + 8.0f) || 8u * near < 4u * below;
}

// The part that a block works on: an eighth of them on each XCD, or all in turn (see short_eighths).
__device__ __forceinline__ uint32_t short_piece(bool eighths)
{
    return eighths ? piece_by_xcd(blockIdx.x, gridDim.x) : blockIdx.x;
}

// One block per part: R rows of four consecutive positions per thread.  The loads of the part are
// requested before anything else is looked at.
template <typename G, int T, int R>
__device__ __forceinline__ void
short_collect(const float* __restrict__ mem, const G* __restrict__ grad, float lr, const PartDesc* __restrict__ parts, uint32_t part_index,
              const uint32_t* __restrict__ preds, const uint32_t* __restrict__ lead_mine, uint4* __restrict__ used,
              uint16_t* __restrict__ counts, uint32_t* __restrict__ keys, unsigned long long* __restrict__ stats)
{
    constexpr int W = T / kLanes, P = T * kVec * R;
    // the sample's counts, then the part's keys in the order in which they leave
    __shared__ __align__(16) uint32_t stage[(1 << kShortSampleLog) > P ? (1 << kShortSampleLog) : P];
    __shared__ uint32_t wave_tot[W];
    __shared__ uint32_t res[2];
    __shared__ uint32_t cnt[kShortCols], first[kShortCols], mixed[kShortCols];
    __shared__ uint64_t heavy;
    const PartDesc d = parts[part_index];
    const int t = threadIdx.x, lane = t % kLanes, wave = __builtin_amdgcn_readfirstlane(t / kLanes);
    const int64_t begin = d.begin, end = d.end;
    // (without a branch, or the compiler waits for these loads before it requests the part's; any valid address where they are not used)
    const bool check = d.n_parts > kShortCheckParts;        // block-uniform
    const float* s_mem = reinterpret_cast<const float*>(parts);
    const G* s_grad = reinterpret_cast<const G*>(parts);
    if (check) {
        const uint32_t up = (static_cast<uint32_t>(d.begin) + kVec - 1) & ~static_cast<uint32_t>(kVec - 1);
        const uint32_t stretch = (static_cast<uint32_t>(d.end) - up) / (kVec * kShortCheckGroups);   // whole groups, at least 512
        const uint32_t j = static_cast<uint32_t>(lane) % kShortCheckGroups;
        const int64_t p0 = up + static_cast<int64_t>(j * stretch + __umulhi(j * 0x9e3779b1u, stretch)) * kVec;
        s_mem = mem + p0;
        s_grad = grad + p0;
    }
    const float4 sm = cached4(s_mem), sg = cached4(s_grad);
    float4 m[R], g[R];
#pragma unroll
    for (int r = 0; r < R; ++r) leader_load<true>(mem, grad, static_cast<int64_t>(d.a0) + (r * T + t) * kVec, begin, end, m[r], g[r]);
    // the prediction's words in one access (a trip for each of them took as long as the part's loads)
    static_assert(kPredWords == 8 && kPredShortWidth == 5 && kPredShortCalm == 6 && kPredShortTrust == 7, "two groups of four");
    const uint4* pred = reinterpret_cast<const uint4*>(preds + static_cast<size_t>(d.seg) * kPredWords);
    const uint4 pred_lo = pred[0], pred_hi = pred[1];
    const uint32_t lead = lead_mine ? lead_mine[d.seg] : 0u;
    uint32_t width = pred_hi.y, mid = 0u;                   // 0: nothing to go by
    const uint32_t trust = pred_hi.w & 0xffffffu;
    uint32_t have = width == 0u ? kShortNone : (ShortTrust(trust).sampling() ? kShortDoubted : kShortExpected);
    if (t < kShortCols) cnt[t] = mixed[t] = 0u;
    uint32_t note = pred_hi.z;                              // calm steps; if the expectation is not used, its top 24 bits and width
    if (width != 0u) {                                      // block-uniform
        const uint32_t t24 = predicted_t24(pred_lo.y, pred_hi.x, lead);
        mid = (t24 << kBits2) | (kBins2 / 2);
        width = width < kShortWidthMin ? kShortWidthMin : (width > kShortWidthMax ? kShortWidthMax : width);
        if (have == kShortExpected && check && short_far_off(sm, sg, lr, d, ShortCols(mid, width), pred_hi.w >> 24))
            have = kShortDoubted;                           // in all blocks
        if (have == kShortDoubted) note = t24 | width << 24;
    }
    if (have != kShortExpected) {
        width = kShortWidthFirst;
        mid = d.k > 0 ? short_sample<G, T>(mem, grad, lr, d, stage, wave_tot, res) : 0u;
    }
    if (part_index == static_cast<uint32_t>(d.part_first) && t == 0)
        used[d.seg] = make_uint4(mid, width, have | trust << 2, note);
    if (stats && part_index == 0 && t == 0) atomicAdd(&stats[kStatSteps], 1ull);

    const ShortCols cols(mid, width);
    uint32_t key[4 * R], col[4 * R], rank[4 * R];
    uint32_t n_ok = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint32_t k4[4];
        bool ok[4];
        keys_from(m[r], g[r], lr, static_cast<int64_t>(d.a0) + (r * T + t) * kVec, begin, end, k4, ok);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            key[4 * r + c] = k4[c];
            col[4 * r + c] = ok[c] && k4[c] != 0u ? cols.column(k4[c]) : static_cast<uint32_t>(kShortCols);
            n_ok += __popcll(__builtin_amdgcn_ballot_w64(ok[c]));
        }
    }
    __syncthreads();                                        // the counts are cleared
    // Ranks inside the column, in no fixed order: one LDS atomic per wave in the two columns where almost
    // all keys are, one per key in the others.
#pragma unroll
    for (int c = 0; c < 4 * R; ++c) {
        rank[c] = 0;
        if (col[c] < static_cast<uint32_t>(kShortBulk)) rank[c] = atomicAdd(&cnt[col[c]], 1u);
    }
#pragma unroll
    for (uint32_t here = kShortBulk; here <= static_cast<uint32_t>(kShortListed); ++here) {
        uint32_t n = 0;
#pragma unroll
        for (int c = 0; c < 4 * R; ++c) n += __popcll(__builtin_amdgcn_ballot_w64(col[c] == here));
        if (n == 0) continue;                               // wave-uniform
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&cnt[here], n);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int c = 0; c < 4 * R; ++c) {
            const uint64_t b = __builtin_amdgcn_ballot_w64(col[c] == here);
            if (col[c] == here) rank[c] = at + lanes_below(b);
            at += __popcll(b);
        }
    }
    if (lane == 0 && n_ok) atomicAdd(&cnt[kShortValid], n_ok);
    __syncthreads();
    if (wave == 0) {                                        // one column per lane
        const uint32_t n = cnt[lane];
        uint32_t run = lane <= kShortListed ? n : 0u;
#pragma unroll
        for (int off = 1; off < kLanes; off <<= 1) {
            const uint32_t v = __shfl_up(run, off, kLanes);
            if (lane >= off) run += v;
        }
        first[lane] = run - (lane <= kShortListed ? n : 0u);
        // columns with so many keys that it pays to know whether they are equal (not the last ones, wide and full as a rule:
        // a sample's threshold is at most 0.9 spans below the narrow columns)
        const uint64_t many = __builtin_amdgcn_ballot_w64(lane < kShortBelow + 6 && n >= static_cast<uint32_t>(P / 32));
        if (lane == 0) heavy = many;
        counts[static_cast<size_t>(part_index) * kShortCols + lane] = static_cast<uint16_t>(lane <= kShortListed ? run : n);
    }
    __syncthreads();
    // through LDS, so that they leave with full-width stores (scattered 4-byte stores took longer than the rest)
#pragma unroll
    for (int c = 0; c < 4 * R; ++c)
        if (col[c] < static_cast<uint32_t>(kShortCols)) stage[first[col[c]] + rank[c]] = key[c];
    const uint32_t n_listed = first[kShortListed + 1];
    const uint64_t many = heavy;
    __syncthreads();
    uint32_t* slice = keys + static_cast<size_t>(part_index) * P;
#pragma unroll
    for (int r = 0; r < R; ++r) {                           // (what lies past the count is never read)
        const uint32_t at = static_cast<uint32_t>(r * T + t) * kVec;
        if (at < n_listed) *reinterpret_cast<uint4*>(slice + at) = *reinterpret_cast<const uint4*>(stage + at);
    }
    if (many == 0) return;                                  // whole block
#pragma unroll
    for (int c = 0; c < 4 * R; ++c)
        if (col[c] < static_cast<uint32_t>(kShortBulk) && stage[first[col[c]]] != key[c]) mixed[col[c]] = 1u;
    __syncthreads();
    if (wave == 0) {
        const uint64_t same = __builtin_amdgcn_ballot_w64(mixed[lane] == 0u) & many;
        uint64_t left = same;                               // the highest four (scalar)
        uint32_t four = 0;
        for (int j = 0; j < 32 && left != 0; j += 8, left &= left - 1) four |= static_cast<uint32_t>(__ffsll(static_cast<long long>(left))) << j;
        if (lane == 0)
            *reinterpret_cast<uint32_t*>(counts + static_cast<size_t>(part_index) * kShortCols + kShortEqual) = four;
    }
}

template <typename G, int T, int R>
__global__ void __launch_bounds__(T)
k_short_collect(const float* __restrict__ mem, const G* __restrict__ grad, float lr, const PartDesc* __restrict__ parts, bool eighths,
                const uint32_t* __restrict__ preds, const uint32_t* __restrict__ lead_mine, uint4* __restrict__ used,
                uint16_t* __restrict__ counts, uint32_t* __restrict__ keys, unsigned long long* __restrict__ stats)
{
    short_collect<G, T, R>(mem, grad, lr, parts, short_piece(eighths), preds, lead_mine, used, counts, keys, stats);
}

// What k_short_collect leaves of one vector, and where its expectations are kept.
struct ShortVector {
    uint32_t* preds;
    uint32_t* lead_mine;         // null: no record per leader
    uint4* used;
    uint16_t* counts;
    uint32_t* keys;
};

// For the similarity diagnostic: the leader's vector (blocks with y = 0) and the sum over learners.
template <typename G, int T, int R>
__global__ void __launch_bounds__(T)
k_short_collect_two(const float* __restrict__ mem, const G* __restrict__ grad, float lr, const float* __restrict__ sum,
                    const PartDesc* __restrict__ parts, ShortVector a, ShortVector b)
{
    if (blockIdx.y == 0)
        short_collect<G, T, R>(mem, grad, lr, parts, blockIdx.x, a.preds, a.lead_mine, a.used, a.counts, a.keys, nullptr);
    else
        short_collect<NoGrad, T, R>(sum, nullptr, 0.0f, parts, blockIdx.x, b.preds, b.lead_mine, b.used, b.counts, b.keys, nullptr);
}

// The listed keys of a segment's parts [0, n_parts), words [from[p], to[p]) of part p's slice, to `f`
// (key, part, how many keys it stands for).  One wave per part, AHEAD parts requested at once: the loads come from the L2 or from
// the memory-side cache, half a microsecond away, and nothing else hides that.
template <int T, int P, typename F>
__device__ __forceinline__ void short_for_keys(const uint32_t* __restrict__ slices, const uint16_t* from, const uint16_t* to,
                                               const uint16_t* weight, int n_parts, F&& f)
{
    constexpr int W = T / kLanes, AHEAD = 4;
    const int lane = threadIdx.x % kLanes, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    for (int p0 = wave; p0 < n_parts; p0 += AHEAD * W) {
        uint32_t s[AHEAD], e[AHEAD], w[AHEAD], longest = 0;
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            const int p = p0 + j * W;
            s[j] = p < n_parts ? from[p] : 0u;
            e[j] = p < n_parts ? to[p] : 0u;
            w[j] = p < n_parts ? weight[p] : 0u;
            const uint32_t len = e[j] - s[j];
            longest = len > longest ? len : longest;
        }
        longest = __builtin_amdgcn_readfirstlane(longest);
        for (uint32_t r = lane; r < ((longest + kLanes - 1) & ~static_cast<uint32_t>(kLanes - 1)); r += kLanes) {
            uint32_t key[AHEAD];
#pragma unroll
            for (int j = 0; j < AHEAD; ++j)
                key[j] = s[j] + r < e[j] ? slices[static_cast<size_t>(p0 + j * W) * P + s[j] + r] : 0u;
#pragma unroll
            for (int j = 0; j < AHEAD; ++j)
                if (s[j] + r < e[j]) f(key[j], p0 + j * W, w[j]);
        }
    }
}

// The rem-th largest of the n <= kShortListMax <= T values in `list`, by comparing all pairs (two
// instructions each, in as many waves as there are values): the smallest value that fewer than rem others
// exceed.  found[wave], for the waves that hold values: the smallest one of the wave as key << 32 | (rem less
// the number of larger values), all bits set if it has none.
// TAGGED: the values are keys shifted left by one, and the lowest bit does not count.
template <int T, bool TAGGED>
__device__ __forceinline__ void short_rank(const uint32_t* list, uint32_t n, uint32_t rem, unsigned long long* found)
{
    static_assert(kShortListMax <= T, "one value per thread");
    const uint32_t t = threadIdx.x, wave = t / kLanes;
    if (wave * kLanes >= n) return;                         // whole wave
    const uint32_t v = t < n ? (TAGGED ? list[t] | 1u : list[t]) : 0u;
    uint32_t higher = 0, j = 0;
    for (; j + 16 <= n; j += 16) {
        uint4 o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = *reinterpret_cast<const uint4*>(list + j + 4 * i);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            higher += (o[i].x > v ? 1u : 0u) + (o[i].y > v ? 1u : 0u) + (o[i].z > v ? 1u : 0u) + (o[i].w > v ? 1u : 0u);
    }
    for (; j < n; ++j) higher += list[j] > v ? 1u : 0u;
    const bool in = t < n && higher < rem;
    const uint32_t least = ~wave_max_u32(in ? ~v : 0u);     // (no value has all bits set)
    if (in && v == least) found[wave] = (static_cast<unsigned long long>(TAGGED ? v >> 1 : v) << 32) | (rem - higher);
}

__device__ __forceinline__ unsigned long long short_least(const unsigned long long* found)
{
    unsigned long long best = found[0];
#pragma unroll
    for (int w = 1; w < static_cast<int>(kShortListMax) / kLanes; ++w) best = found[w] < best ? found[w] : best;
    return best;
}

// Sum over the lanes with the same lane % 8, in all of them: a rotation inside each row of 16 lanes, then
// rows and halves of the wave exchanged inside the vector ALU.
__device__ __forceinline__ uint32_t sum_of_every_eighth(uint32_t v)
{
    constexpr int kRowRotate8 = 0x128;
    v += dpp_move<kRowRotate8, 0xf>(v);
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = a[0] + a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return b[0] + b[1];
}

// LDS of a block's search, and what the search finds.
template <int T>
struct ShortLds {
    static constexpr int W = T / kLanes;
    alignas(16) uint32_t hist[kShortGeneral];               // bins of the general search, or the column's keys
    alignas(16) uint32_t list[kShortListMax];
    unsigned long long found[kShortListMax / kLanes];       // per wave: threshold key, members among its holders
    uint32_t sums[W][kShortCols];
    uint32_t wave_tot[W];
    uint32_t res[4];                                        // found, bin, its count, keys above it
    uint32_t n_list, n_over, n_scan;
    uint32_t own[2][W];                                     // members for sure / ties in earlier parts
    uint16_t from[kShortSegParts], to[kShortSegParts], weight[kShortSegParts];
};
static_assert(kShortGeneral >= kShortColumnMax, "a column fits");

struct ShortFound {
    uint32_t T_key, q;           // threshold (all bits set: no member), members among its holders
    uint32_t gt_before, eq_before;   // members for sure / ties in the parts before the block's own
    uint32_t n_bins, n_col, n_valid; // keys of the narrow columns, of the threshold's column; positions of the segment
    uint32_t n_near;                 // keys down to the end of column kShortBulk
    uint32_t n_scan, n_same;         // keys that the whole block had to read, several times; how many of them are the threshold itself (if many)
    int col;
    bool missed;
};

// The search for the segment of a block's part, by all T threads; ends with a barrier.  `request` is called
// once the counts have been requested, `ahead` once the usual step's last keys have been: for loads that nothing here waits for
// (loads return in the order of their requests).
template <int T, int P, typename F, typename A>
__device__ __forceinline__ ShortFound short_search(ShortLds<T>& lds, const PartDesc& d, const uint4* __restrict__ used,
                                                   const uint16_t* __restrict__ counts, const uint32_t* __restrict__ keys,
                                                   F&& request, A&& ahead)
{
    constexpr int W = T / kLanes;
    uint32_t* hist = lds.hist;
    uint32_t* list = lds.list;
    uint32_t* wave_tot = lds.wave_tot;
    uint32_t* res = lds.res;
    unsigned long long* found = lds.found;
    const int t = threadIdx.x, lane = t % kLanes, wave = __builtin_amdgcn_readfirstlane(t / kLanes);
    const int mine = (d.a0 - (d.begin & ~(kVec - 1))) / P, n_parts = d.n_parts;
    const uint32_t k = static_cast<uint32_t>(d.k);

    // The counts of all parts, requested at once: eight lanes per part, eight parts per wave and turn.
    const uint16_t* my_counts = counts + static_cast<size_t>(d.part_first) * kShortCols;
    constexpr int kTurns = kShortSegParts / (W * 8);
    static_assert(kTurns * W * 8 == kShortSegParts && kShortSegParts <= T, "all of them, and one per thread");
    uint4 row[kTurns];
#pragma unroll
    for (int i = 0; i < kTurns; ++i) {
        const int r = (i * W + wave) * 8 + lane / 8;
        row[i] = make_uint4(0, 0, 0, 0);
        if (r < n_parts) row[i] = reinterpret_cast<const uint4*>(my_counts + static_cast<size_t>(r) * kShortCols)[lane % 8];
    }
    const uint4 u = used[d.seg];
    request();
    uint32_t acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < kTurns; ++i) {
        if (i * W * 8 >= n_parts) continue;                 // block-uniform
        const uint32_t v[4] = {row[i].x, row[i].y, row[i].z, row[i].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[2 * j] += v[j] & 0xffffu;
            acc[2 * j + 1] += v[j] >> 16;
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = sum_of_every_eighth(acc[j]);
    if (t < static_cast<int>(kShortListMax) / kLanes) found[t] = ~0ull;
    if (lane < 8) {
#pragma unroll
        for (int j = 0; j < 8; ++j) lds.sums[wave][lane * 8 + j] = acc[j];
    }
    __syncthreads();
    uint32_t total = 0;                                     // lane j: running count of column j over the segment
#pragma unroll
    for (int w = 0; w < W; ++w) total += lds.sums[w][lane];
    const uint32_t n_listed = __builtin_amdgcn_readlane(static_cast<int>(total), kShortListed);
    const uint32_t n_valid = __builtin_amdgcn_readlane(static_cast<int>(total), kShortValid);
    // the first column with which k keys are listed
    const uint64_t enough = __builtin_amdgcn_ballot_w64(lane <= kShortListed && total >= k);
    const int col = enough != 0 ? __ffsll(static_cast<unsigned long long>(enough)) - 1 : kShortListed;
    const uint32_t sure = col > 0 ? __builtin_amdgcn_readlane(static_cast<int>(total), col > 0 ? col - 1 : 0) : 0u;   // members
    const uint32_t n_col = __builtin_amdgcn_readlane(static_cast<int>(total), col) - sure;
    const uint32_t n_bins = __builtin_amdgcn_readlane(static_cast<int>(total), kShortBelow - 1) -
                            __builtin_amdgcn_readlane(static_cast<int>(total), kShortFirstBin - 1);
    const uint32_t n_near = __builtin_amdgcn_readlane(static_cast<int>(total), kShortBulk);
    const ShortCols cols(u.x, u.y);
    uint32_t T_key = 0xffffffffu, q = 0, n_scan = 0, n_same = 0;                    // no member
    uint32_t gt_mine = 0, eq_mine = 0;                      // this thread's share of the members for sure / ties in earlier parts
    // one part per thread from here on: what it lists before and in the column
    uint32_t lo_c = 0, hi_c = 0;
    const bool has_part = t < n_parts, earlier = t < mine;
    const bool no_search = k != 0 && (n_listed < k || k >= n_valid);
    if (k != 0 && has_part) {
        const uint16_t* mc = my_counts + static_cast<size_t>(t) * kShortCols;
        lo_c = col > 0 ? mc[col - 1] : 0u;
        hi_c = mc[col];
        if (no_search && earlier) {
            gt_mine = mc[kShortListed];
            eq_mine = mc[kShortValid] - gt_mine;
        }
    }
    // every branch from here on is block-uniform: k, the totals and `used` are the same in all threads
    bool missed = false;
    if (k == 0) {
        ahead();                                            // no member
    } else if (no_search) {
        ahead();
        // the k-th largest key is 0, or every position is a member: no key has to be looked at
        T_key = 0u;
        q = k > n_listed ? k - n_listed : 0u;
        missed = cols.end(kShortBulk - 1) > 1u;
    } else if (n_col <= kShortColumnMax) {
        // The usual step: the column is small.  Up to kShortListMax keys: one per thread, ranked against all
        // others.  More: one wave finds the threshold bit by bit (a ballot per bit and 64 keys, no barrier),
        // 2 us whatever the number.
        const uint32_t n_mine = hi_c - lo_c;
        uint32_t at = n_mine;                               // inclusive, then exclusive prefix: where my part's keys go
#pragma unroll
        for (int off = 1; off < kLanes; off <<= 1) {
            const uint32_t v = __shfl_up(at, off, kLanes);
            if (lane >= off) at += v;
        }
        if (lane == kLanes - 1) wave_tot[wave] = at;
        at -= n_mine;
        const uint32_t* src = keys + static_cast<size_t>(d.part_first + (has_part ? t : 0)) * P + lo_c;
        uint32_t early_key[4];                              // (most parts have fewer)
#pragma unroll
        for (int j = 0; j < 4; ++j) early_key[j] = static_cast<uint32_t>(j) < n_mine ? src[j] : 0u;
        ahead();
        __syncthreads();
#pragma unroll
        for (int w = 0; w < W; ++w) at += w < wave ? wave_tot[w] : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (static_cast<uint32_t>(j) < n_mine) hist[at + j] = early_key[j];
        for (uint32_t j = 4; j < n_mine; ++j) hist[at + j] = src[j];
        __syncthreads();
        if (n_col <= kShortListMax) {
            short_rank<T, false>(hist, n_col, k - sure, found);
        } else if (wave == 0) {
            constexpr int kMine = kShortColumnMax / kLanes;
            uint32_t v[kMine];
#pragma unroll
            for (int j = 0; j < kMine; ++j) {
                const uint32_t e = j * kLanes + lane;
                v[j] = e < n_col ? hist[e] : 0u;
            }
            auto at_least = [&](uint32_t cand) {            // cand >= 1
                uint32_t c = 0;
#pragma unroll
                for (int j0 = 0; j0 < kMine; j0 += 4) {
                    if (static_cast<uint32_t>(j0 * kLanes) >= n_col) continue;       // wave-uniform
#pragma unroll
                    for (int j = j0; j < j0 + 4; ++j) c += __popcll(__builtin_amdgcn_ballot_w64(v[j] >= cand));
                }
                return c;
            };
            const uint32_t rem = k - sure;
            uint32_t T_w = cols.end(col);
            const uint32_t range = col > 0 ? cols.end(col - 1) - T_w : 0x80000000u - T_w;   // at least 1: the column is not empty
            for (int bit = 31 - __clz(static_cast<int>(range)); bit >= 0; --bit)
                if (at_least(T_w + (1u << bit)) >= rem) T_w += 1u << bit;
            const uint32_t q_w = rem - at_least(T_w + 1u);
            if (lane == 0) found[0] = (static_cast<unsigned long long>(T_w) << 32) | q_w;
        }
        __syncthreads();
        const unsigned long long best = short_least(found);
        T_key = static_cast<uint32_t>(best >> 32);
        q = static_cast<uint32_t>(best);
        missed = col < kShortAbove - 1 || col >= kShortBulk;
        if (earlier) {
            gt_mine = lo_c;
            for (uint32_t j = 0; j < n_mine; ++j) {
                const uint32_t key = hist[at + j];
                gt_mine += key > T_key ? 1u : 0u;
                eq_mine += key == T_key ? 1u : 0u;
            }
        }
    } else {
        // The threshold is further off than expected, or many keys share its column: the whole block
        // searches the column, from the parts' slices.
        missed = col < kShortAbove - 1 || col >= kShortBulk;
        if (earlier) gt_mine = lo_c;
        uint32_t base = cols.end(col);
        uint32_t span = 24u;                                // log2 of the keys counted in bins
        if (col > 0) span = 32u - static_cast<uint32_t>(__clz(static_cast<int>(cols.end(col - 1) - base)));   // (not empty: at least 1)
        if (span > 31u) span = 31u;
        if (has_part) {                                     // equal keys: the first one for all of them
            const uint32_t four = *reinterpret_cast<const uint32_t*>(my_counts + static_cast<size_t>(t) * kShortCols + kShortEqual);
            bool one = false;
#pragma unroll
            for (int j = 0; j < 32; j += 8) one = one || ((four >> j) & 0xffu) == static_cast<uint32_t>(col) + 1u;
            lds.from[t] = static_cast<uint16_t>(lo_c);
            lds.to[t] = static_cast<uint16_t>(one ? lo_c + 1u : hi_c);
            lds.weight[t] = static_cast<uint16_t>(one ? hi_c - lo_c : 1u);
            n_scan = one ? 1u : hi_c - lo_c;
        }
        if (t == 0) lds.n_scan = 0u;
        n_scan = wave_sum(n_scan);
        const uint32_t* slices = keys + static_cast<size_t>(d.part_first) * P;
        bool by_list = false;
        uint32_t rem = 0;                                   // rank of the threshold inside the bin that was found
        for (int level = 0; level < 8; ++level) {           // (at most: bins above the range, then 31 bits)
            const uint32_t shift = span > kShortGeneralLog ? span - kShortGeneralLog : 0u;
            __syncthreads();                                // everybody has read what is cleared here
            for (int b = t; b < kShortGeneral; b += T) hist[b] = 0u;
            if (t == 0) lds.n_over = lds.n_list = res[0] = 0u;
            if (level == 0 && lane == 0 && n_scan) atomicAdd(&lds.n_scan, n_scan);
            __syncthreads();
            uint32_t over = 0;
            short_for_keys<T, P>(slices, lds.from, lds.to, lds.weight, n_parts, [&](uint32_t key, int, uint32_t w) {
                const uint32_t rel = key - base;
                if (key < base) return;
                if (rel >> span) {
                    over += w;
                    return;
                }
                // the lanes that share the first one's bin add once (few-valued data would wait for one word 64 times)
                const uint32_t bin = rel >> shift, lead = __builtin_amdgcn_readfirstlane(static_cast<int>(bin));
                const uint64_t same = __builtin_amdgcn_ballot_w64(bin == lead);
                if (bin != lead)
                    atomicAdd(&hist[bin], w);
                else if (lanes_below(same) == 0u)
                    atomicAdd(&hist[bin], w * static_cast<uint32_t>(__popcll(same)));
            });
            over = wave_sum(over);
            if (lane == 0 && over) atomicAdd(&lds.n_over, over);
            __syncthreads();
            over = sure + lds.n_over;
            if (over >= k) {                                // the threshold lies above the counted range
                base += 1u << span;
                span = 31u;                                 // everything above
                continue;
            }
            uint32_t bin, n_bin, n_above;
            if (short_find_bin<T, kShortGeneral>(hist, k - over, wave_tot, bin, n_bin, n_above)) {
                res[1] = bin;
                res[2] = n_bin;
                res[3] = n_above;
                res[0] = 1u;
            }
            __syncthreads();
            if (res[0] == 0u) break;                        // only if the counts were corrupted: nothing is selected
            rem = k - over - res[3];
            base += res[1] << shift;
            span = shift;
            if (shift == 0u) {                              // one key per bin
                T_key = base;
                q = rem;
                n_same = res[2];
                break;
            }
            if (res[2] <= kShortListMax) {
                by_list = true;
                break;
            }
        }
        if (by_list) {
            // the bin's few keys (lowest bit: from a part before mine), ranked against each other
            short_for_keys<T, P>(slices, lds.from, lds.to, lds.weight, n_parts, [&](uint32_t key, int p, uint32_t w) {
                if (key < base) return;
                if ((key - base) >> span) {
                    gt_mine += p < mine ? w : 0u;
                } else {
                    uint32_t at = atomicAdd(&lds.n_list, w);
                    for (const uint32_t past = at + w; at < past && at < kShortListMax; ++at)
                        list[at] = (key << 1) | (p < mine ? 1u : 0u);
                }
            });
            __syncthreads();
            const uint32_t n = lds.n_list < kShortListMax ? lds.n_list : kShortListMax;
            short_rank<T, true>(list, n, rem, found);
            __syncthreads();
            const unsigned long long best = short_least(found);
            T_key = static_cast<uint32_t>(best >> 32);
            q = static_cast<uint32_t>(best);
            if (static_cast<uint32_t>(t) < n && (list[t] & 1u)) {
                const uint32_t v = list[t] >> 1;
                gt_mine += v > T_key ? 1u : 0u;
                eq_mine += v == T_key ? 1u : 0u;
            }
        } else if (T_key != 0xffffffffu) {
            short_for_keys<T, P>(slices, lds.from, lds.to, lds.weight, n_parts, [&](uint32_t key, int p, uint32_t w) {
                gt_mine += p < mine && key > T_key ? w : 0u;
                eq_mine += p < mine && key == T_key ? w : 0u;
            });
        }
        n_scan = lds.n_scan;                                // (added up behind the first level's barrier)
        ahead();
    }
    {
        const uint32_t g = wave_sum(gt_mine), e = wave_sum(eq_mine);
        if (lane == 0) {
            lds.own[0][wave] = g;
            lds.own[1][wave] = e;
        }
    }

    __syncthreads();
    ShortFound f{T_key, q, 0u, 0u, n_bins, n_col, n_valid, n_near, n_scan, n_same, col, missed};
#pragma unroll
    for (int w = 0; w < W; ++w) {
        f.gt_before += lds.own[0][w];
        f.eq_before += lds.own[1][w];
    }
    return f;
}

// What the next steps expect, and the counters (stats: null for none): by the segment's first block.
__device__ __forceinline__ void short_record(const PartDesc& d, const uint4& u, const ShortFound& f, uint32_t* __restrict__ preds,
                                             uint32_t* __restrict__ lead_mine, unsigned long long* __restrict__ stats)
{
    const uint32_t k = static_cast<uint32_t>(d.k);
    const int col = f.col;
    if (d.a0 > d.begin || threadIdx.x != 0 || k == 0 || f.T_key == 0xffffffffu) return;
    uint32_t* pred = preds + static_cast<size_t>(d.seg) * kPredWords;
    const uint32_t have = u.z & 3u;
    bool held = !f.missed;
    uint32_t learned = u.y;                                 // width to go on from
    if (have == kShortDoubted) {                            // would it have been in or next to the narrow columns, with their width?
        learned = u.w >> 24;
        const ShortCols cols(((u.w & 0xffffffu) << kBits2) | (kBins2 / 2), learned);
        held = f.T_key < cols.end(kShortAbove - 1) + cols.span() && f.T_key >= cols.end(kShortBelow + 3);
    }
    pred[kPredShortTrust] = ShortTrust(u.z >> 2).next(held, f.n_scan > kShortLong && have == kShortExpected) |
                            static_cast<uint32_t>(64.0f * static_cast<float>(f.n_near) / static_cast<float>(f.n_valid)) << 24;
    // The narrow columns: wider at once if the threshold left their middle half or if they held few keys, narrower at once if
    // the threshold's own held too many different ones, and after some calm steps if they all held many more than a quarter of an index set's worth (and enough for
    // the spread of an order statistic of rank k): few keys to search, and a threshold that leaves the narrow
    // columns lands in one that is not much larger.  (As many as the index set: 24.5 us a step at 4 x 1 M, now 22.6.)
    uint32_t want = static_cast<uint32_t>(8.0f * sqrtf(static_cast<float>(k)));
    want = want > k / 4u ? want : k / 4u;
    want = want > 64u ? want : 64u;
    const bool middle = col >= kShortFirstBin + kShortBins / 4 && col < kShortBelow - kShortBins / 4;
    uint32_t width = learned, calm = middle ? u.w + 1u : 0u;
    const uint32_t crowd = f.n_scan > f.n_same ? f.n_scan - f.n_same : 0u;
    if (have == kShortDoubted) {                            // (the columns were the sample's)
        width += held ? 0u : 1u;
        calm = 0u;
    } else if (middle && crowd > kShortColumnMax) {
        uint32_t less = 32u - static_cast<uint32_t>(__clz(static_cast<int>(crowd / kShortColumnMax)));
        less = less < 4u ? less : 4u;
        width = width > less + kShortWidthMin ? width - less : kShortWidthMin;
        calm = 0u;
    } else if (!middle || 5u * f.n_bins < 3u * want) {
        ++width;
        calm = 0u;
    } else if (calm >= kShortCalm && 2u * f.n_bins > 3u * want) {
        --width;
        calm = 0u;
    }
    width = width < kShortWidthMin ? kShortWidthMin : (width > kShortWidthMax ? kShortWidthMax : width);
    pred[kPredShortWidth] = width;
    pred[kPredShortCalm] = calm;
    record_t24(pred, lead_mine, d.seg, f.T_key >> kBits2);
    if (stats && f.n_valid > static_cast<uint32_t>(kSuper)) {
        if (have == kShortNone)
            atomicAdd(&stats[kStatNoPrediction], 1ull);
        else if (!held)
            atomicAdd(&stats[kStatMissed], 1ull);
        if (f.n_scan != 0u) atomicAdd(&stats[kStatFullMode], 1ull);   // searched by the whole block
    }
}

// One block per part: search, output slots, update of all learners, sums (see the top of the file).
// The update walks the learners one after the other with one position group per thread: at these
// sizes that is as fast as one learner per block (4 M elements in all: 16 us either way; 28 M: 57 us
// against 53 us), and the sums over learners stay in registers.
//   OCC: waves per SIMD that the registers are kept for, 4 or 6.  Layouts of several tensors have more blocks than the chip runs at once: with few
// learners six hide more of each other's searches (60 tensors, 1183 blocks of 512 threads, 4 learners bfloat16 41.0 us a step with four, 39.4 with six;
// 150 tensors x 3 37.2 / 36.8; but 60 x 8 63.1 / 65.0, 200 x 8 52.2 / 54.0, 30 x 6 33.2 / 34.0).  With four the registers hold the first
// learners' loads of the block's only row while it searches: blocks that are all on the chip at once search together
// and leave memory idle meanwhile (4 x 1 M 22.9 -> 20.1 us, 3 x 200 003 13.5 -> 12.4, 8 x 300 000 17.0 -> 15.7; of two rows the first: no gain).
template <typename G, int T, int R, int OCC>
__global__ void __launch_bounds__(T, OCC)
k_short_step(LearnerPtrs lp, int n_learners, int leader, float lr, float beta, float one_minus_beta,
             const PartDesc* __restrict__ parts, bool eighths, uint32_t* __restrict__ preds, uint32_t* __restrict__ lead_mine,
             const uint4* __restrict__ used, const uint16_t* __restrict__ counts, const uint32_t* __restrict__ keys,
             int32_t* __restrict__ idx_out, float* __restrict__ red_out, unsigned long long* __restrict__ stats)
{
    constexpr int W = T / kLanes, P = T * kVec * R;
    constexpr int kAtOnce = T <= 512 && OCC <= 4 ? 8 : 4;   // learners whose loads are in flight together
    constexpr bool kAhead = OCC <= 4 && R == 1;
    __shared__ ShortLds<T> lds;
    __shared__ uint32_t in_row[2][2][W];                    // of two rows in turn: members for sure / ties
    const PartDesc d = parts[short_piece(eighths)];
    const int t = threadIdx.x, lane = t % kLanes, wave = __builtin_amdgcn_readfirstlane(t / kLanes);
    const int64_t begin = d.begin, end = d.end;
    const uint32_t k = static_cast<uint32_t>(d.k);
    float4 lm, lg;
    float4 m[kAtOnce];                                      // the first learners'
    Streamed<G> g[kAtOnce];
    const int64_t first = static_cast<int64_t>(d.a0) + t * kVec;
    const ShortFound f = short_search<T, P>(lds, d, used, counts, keys, [&]() {
        leader_load<true>(lp.mem[leader], static_cast<const G*>(lp.grad[leader]), first, begin, end, lm, lg);
    }, [&]() {
        if (kAhead && first >= begin && first + 3 < end) {
#pragma unroll
            for (int j = 0; j < kAtOnce; ++j) {
                if (j >= n_learners) continue;              // uniform
                m[j] = load4(lp.mem[j] + first);
                g[j] = stream4(static_cast<const G*>(lp.grad[j]) + first);
            }
        }
    });
    short_record(d, used[d.seg], f, preds, lead_mine, stats);
    const uint32_t T_key = f.T_key, q = f.q;
    uint32_t gt_run = f.gt_before, eq_run = f.eq_before;    // members for sure / ties before the row
#pragma unroll 1
    for (int r = 0; r < R; ++r) {
        // membership and output slots of my four positions (ties in position order until q are taken)
        const int64_t p0 = static_cast<int64_t>(d.a0) + (r * T + t) * kVec;
        uint32_t key[4];
        bool ok[4];
        keys_from(lm, lg, lr, p0, begin, end, key, ok);
        bool gt[4], eq[4];
        uint32_t gt_rank = 0, eq_rank = 0, n_gt = 0, n_eq = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            gt[c] = ok[c] && T_key != 0xffffffffu && key[c] > T_key;
            eq[c] = ok[c] && key[c] == T_key;
            const uint64_t bg = __builtin_amdgcn_ballot_w64(gt[c]), be = __builtin_amdgcn_ballot_w64(eq[c]);
            gt_rank += lanes_below(bg);
            eq_rank += lanes_below(be);
            n_gt += __popcll(bg);
            n_eq += __popcll(be);
        }
        if (lane == 0) {
            in_row[r & 1][0][wave] = n_gt;
            in_row[r & 1][1][wave] = n_eq;
        }
        __syncthreads();
        gt_rank += gt_run;
        eq_rank += eq_run;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t a = in_row[r & 1][0][w], b = in_row[r & 1][1][w];
            gt_run += a;
            eq_run += b;
            gt_rank += w < wave ? a : 0u;
            eq_rank += w < wave ? b : 0u;
        }
        bool sel[4];
        uint32_t slot[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            sel[c] = gt[c] || (eq[c] && eq_rank < q);
            slot[c] = static_cast<uint32_t>(d.out_base) + gt_rank + (eq_rank < q ? eq_rank : q);
            gt_rank += gt[c] ? 1u : 0u;
            eq_rank += eq[c] ? 1u : 0u;
        }
        if (r + 1 < R)                                      // the next row's, while this one is updated
            leader_load<true>(lp.mem[leader], static_cast<const G*>(lp.grad[leader]), p0 + T * kVec, begin, end, lm, lg);
        if (p0 >= end || p0 + 3 < begin) continue;          // none of the four positions (no barrier until the next row)
        const bool full = p0 >= begin && p0 + 3 < end;
        float4 sum = make_float4(0, 0, 0, 0);
        auto learner = [&](int i, const float4& m, const float4& g) {
            const float4 x = accumulate4(m, g, lr);
            if (i == 0) {
                sum = x;
            } else {                                        // Alg. 1 line 10, learner 0 first
                sum.x = sum.x + x.x;
                sum.y = sum.y + x.y;
                sum.z = sum.z + x.z;
                sum.w = sum.w + x.w;
            }
            float4 out;                                     // Eq. 5: residual is x off the index set, 0 on it
            out.x = fmaf(beta, sel[0] ? 0.0f : x.x, one_minus_beta * m.x);
            out.y = fmaf(beta, sel[1] ? 0.0f : x.y, one_minus_beta * m.y);
            out.z = fmaf(beta, sel[2] ? 0.0f : x.z, one_minus_beta * m.z);
            out.w = fmaf(beta, sel[3] ? 0.0f : x.w, one_minus_beta * m.w);
            store_guarded(lp.mem[i], p0, begin, end, full, out);
        };
        if (full) {
            int i = 0;
            if (kAhead) {
#pragma unroll
                for (int j = 0; j < kAtOnce; ++j)
                    if (j < n_learners) learner(j, m[j], widen4(g[j]));
                i = kAtOnce;
            }
            for (; i < n_learners; i += kAtOnce) {          // (registers of the turn's own: kept for the next row they cost one learner 6 %)
                float4 m[kAtOnce];
                Streamed<G> g[kAtOnce];
#pragma unroll
                for (int j = 0; j < kAtOnce; ++j) {
                    if (i + j >= n_learners) continue;      // uniform
                    m[j] = load4(lp.mem[i + j] + p0);
                    g[j] = stream4(static_cast<const G*>(lp.grad[i + j]) + p0);
                }
#pragma unroll
                for (int j = 0; j < kAtOnce; ++j)
                    if (i + j < n_learners) learner(i + j, m[j], widen4(g[j]));
            }
        } else {
            for (int i = 0; i < n_learners; ++i)
                learner(i, load_guarded(lp.mem[i], p0, begin, end, false),
                        load_guarded(static_cast<const G*>(lp.grad[i]), p0, begin, end, false));
        }
        const float s4[4] = {sum.x, sum.y, sum.z, sum.w};
        const uint32_t slot_end = static_cast<uint32_t>(d.out_base) + k;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (sel[c] && slot[c] < slot_end) {             // the bound only matters if the counts were corrupted
                idx_out[slot[c]] = static_cast<int32_t>(p0 + c);
                red_out[slot[c]] = s4[c];
            }
        }
    }
}

// The similarity diagnostic on a short layout: the searches for the leader's vector and for the sum over learners,
// then the positions that both index sets hold, taken off d (preset to k).
template <typename G, int T, int R>
__global__ void __launch_bounds__(T, T < 1024 ? 6 : 4)
k_short_overlap(const float* __restrict__ mem, const G* __restrict__ grad, float lr, const float* __restrict__ sum,
                const PartDesc* __restrict__ parts, ShortVector a, ShortVector b, int32_t* __restrict__ d_out)
{
    constexpr int W = T / kLanes, P = T * kVec * R;
    __shared__ ShortLds<T> lds;
    __shared__ uint32_t in_row[2][2][W];                    // of two rows in turn: ties of the two sets
    const PartDesc d = parts[blockIdx.x];
    if (d.k == 0) return;                                   // whole block: nothing in common
    const int t = threadIdx.x, lane = t % kLanes, wave = __builtin_amdgcn_readfirstlane(t / kLanes);
    const int64_t begin = d.begin, end = d.end;
    const ShortFound fa = short_search<T, P>(lds, d, a.used, a.counts, a.keys, []() {}, []() {});
    short_record(d, a.used[d.seg], fa, a.preds, a.lead_mine, nullptr);
    __syncthreads();                                        // the search's words are used again
    const ShortFound fb = short_search<T, P>(lds, d, b.used, b.counts, b.keys, []() {}, []() {});
    short_record(d, b.used[d.seg], fb, b.preds, b.lead_mine, nullptr);
    uint32_t run_a = fa.eq_before, run_b = fb.eq_before, both = 0;
#pragma unroll 1
    for (int r = 0; r < R; ++r) {
        const int64_t p0 = static_cast<int64_t>(d.a0) + (r * T + t) * kVec;
        uint32_t ka[4], kb[4];
        bool ok[4];
        leader_keys<true>(mem, grad, lr, p0, begin, end, ka, ok);
        leader_keys<true>(sum, static_cast<const NoGrad*>(nullptr), 0.0f, p0, begin, end, kb, ok);
        uint32_t rank_a = run_a, rank_b = run_b, n_a = 0, n_b = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint64_t ba = __builtin_amdgcn_ballot_w64(ok[c] && ka[c] == fa.T_key);
            const uint64_t bb = __builtin_amdgcn_ballot_w64(ok[c] && kb[c] == fb.T_key);
            rank_a += lanes_below(ba);
            rank_b += lanes_below(bb);
            n_a += __popcll(ba);
            n_b += __popcll(bb);
        }
        if (lane == 0) {
            in_row[r & 1][0][wave] = n_a;
            in_row[r & 1][1][wave] = n_b;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t x = in_row[r & 1][0][w], y = in_row[r & 1][1][w];
            run_a += x;
            run_b += y;
            rank_a += w < wave ? x : 0u;
            rank_b += w < wave ? y : 0u;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool ea = ok[c] && ka[c] == fa.T_key, eb = ok[c] && kb[c] == fb.T_key;
            const bool in_a = ok[c] && (ka[c] > fa.T_key || (ea && rank_a < fa.q));   // (no member: T_key is above every key)
            const bool in_b = ok[c] && (kb[c] > fb.T_key || (eb && rank_b < fb.q));
            both += in_a && in_b ? 1u : 0u;
            rank_a += ea ? 1u : 0u;
            rank_b += eb ? 1u : 0u;
        }
    }
    both = wave_sum(both);
    __syncthreads();
    if (lane == 0) lds.wave_tot[wave] = both;
    __syncthreads();
    if (t == 0) {
        uint32_t n = 0;
        for (int w = 0; w < W; ++w) n += lds.wave_tot[w];
        if (n) atomicSub(&d_out[d.seg], static_cast<int32_t>(n));
    }
}

}  // namespace
