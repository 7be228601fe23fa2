// Chunk-wise selection, the selector of the paper's own implementation (Sec. 4, App. E, Fig. A2).
// Part of scalecom.hip's single translation unit.
#pragma once

#include <hip/hip_runtime.h>

#include "device_helpers.h"
#include "geometry.h"
#include "update_kernels.h"

namespace {

// The chunks that a group of the kernels below owns: group u of a supertile takes G = (256 * Q - 3) / chunk chunks
// from the supertile's u * G-th on (a chunk belongs to the supertile in which it starts; the group's first
// position may lie up to 3 behind a multiple of 4).
template <int Q>
struct ChunkGroup {
    uint32_t begin, end, ch, recip;     // segment, elements per chunk; rel / ch = rel * recip >> 22 for rel < 1024
    uint32_t first, n;                  // first chunk (counted in the segment) and number of chunks
    uint32_t lo, hi, base;              // positions [lo, hi); lo rounded down to a multiple of 4
    int32_t out_base;
    __device__ __forceinline__ bool find(const StDesc& d, uint32_t u)   // false: no chunk left
    {
        // positions and chunk sizes are below 2^31 + 8192: 32-bit arithmetic throughout
        begin = static_cast<uint32_t>(d.begin);
        end = static_cast<uint32_t>(d.end);
        ch = static_cast<uint32_t>(d.sel_chunk);
        out_base = d.out_base;
        // 2^22 / ch rounded up, or a little more (the factor makes up for the reciprocal's last bit)
        recip = static_cast<uint32_t>(4194308.0f * __builtin_amdgcn_rcpf(static_cast<float>(ch))) + 1u;
        const uint32_t per_group = ((256u * Q - 3u) * recip) >> 22;
        const uint32_t a0 = static_cast<uint32_t>(d.a0), st_end = a0 + kSuper < end ? a0 + kSuper : end;
        first = static_cast<uint32_t>(d.chunk_first) + u * per_group;
        lo = begin + first * ch;
        if (lo >= st_end) return false;
        const uint32_t starts = st_end - 1u - lo;           // the last position at which a chunk of mine may start, from lo
        n = starts >= per_group * ch ? per_group : ((starts * recip) >> 22) + 1u;
        hi = n * ch < end - lo ? lo + n * ch : end;
        base = lo & ~static_cast<uint32_t>(kVec - 1);
        return true;
    }
};

// The whole chunk-wise step in one launch, for chunks of up to 1021 elements and little data (see chunks_in_one_launch).  What the step cannot do without is
// one read of (mem, grad) and one write of mem per learner, and
// a chunk's winner depends on nothing outside the chunk.  So a block takes whole chunks, at most
// 256 * Q - 3 positions, and all learners: one wave per learner and wave tile (the access pattern of the
// all-learner pass: one wave moves 256 consecutive positions of one learner; several tiles per wave or
// several learners per thread cost 5 to 20 % of the rate), the leader's first.  Winners and the members' values
// go through LDS.  Blocks share no chunk, so the memories can be updated in place.  Groups of four tiles are for chunks of 510 to 1021 elements (chunk 1000, us, against
// the leader first: 2 x 0.3 M 8 / 13, 1 x 3 M 10.6 / 13.2, 4 x 5 M 47 / 53).
constexpr int kChunkStepWaves = 16;              // waves of a block at most: further (learner, tile) pairs take turns

template <typename G, int Q>
__global__ void __launch_bounds__(kChunkStepWaves * kLanes)
k_chunk_step(const LearnerPtrs lp, int n_learners, int leader, float lr, float beta, float one_minus_beta,
             const StDesc* __restrict__ sts, int n_st, int max_chunks, int32_t* __restrict__ idx_out,
             float* __restrict__ red_out)
{
    // per chunk the largest word (magnitude key << 32 | ~position), then [chunk][learner] the learners' values there
    extern __shared__ unsigned long long chunk_lds[];
    unsigned long long* best = chunk_lds;
    float* xs = reinterpret_cast<float*>(chunk_lds + max_chunks);
    // (groups in turn: an eighth of them per XCD is faster on some vectors, 3 x 3 M, chunk 112 24.1 -> 23.2 us, 2 x 8 M, 25 41.6 -> 38.3, slower on
    // others, 4 x 3.75 M, 25 38.7 -> 42.1, 500 35.7 -> 42.3, and up to twice as slow where small tensors lie side by side)
    const int st = static_cast<int>(blockIdx.y + blockIdx.z * gridDim.y);
    if (st >= n_st) return;                                 // padding of the 3-d grid (whole block)
    const StDesc d = sts[st];
    ChunkGroup<Q> grp;
    if (!grp.find(d, blockIdx.x)) return;                   // whole block
    const uint32_t begin = grp.begin, end = grp.end, recip = grp.recip, cf = grp.first, n_ch = grp.n;
    const uint32_t lo = grp.lo, hi = grp.hi, base = grp.base;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes), lane = threadIdx.x % kLanes;
    const int n_waves = blockDim.x / kLanes;
    const int n_pairs = n_learners * Q;
    float4 m, g;
    // pair p: tile p % Q of learner (leader + p / Q) mod n.  Four positions that straddle the block's ends are
    // loaded whole where they lie inside the segment; what other blocks write there meanwhile is not used.
    auto place = [&](int p, int& l, uint32_t& p0) {
        l = leader + p / Q;
        if (l >= n_learners) l -= n_learners;
        p0 = base + static_cast<uint32_t>(p % Q) * kWaveTile + static_cast<uint32_t>(lane) * kVec;
    };
    auto fetch = [&](int l, uint32_t p0) {
        m = make_float4(0, 0, 0, 0);
        g = m;
        if (p0 >= hi) return;
        const bool whole = p0 >= begin && p0 + 3 < end;
        m = load_guarded(lp.mem[l], p0, begin, end, whole);
        g = load_guarded(static_cast<const G*>(lp.grad[l]), p0, begin, end, whole);
    };
    int l;
    uint32_t p0;
    place(wave, l, p0);
    if (wave < n_pairs) fetch(l, p0);
    for (uint32_t j = threadIdx.x; j < n_ch; j += blockDim.x) best[j] = 0ull;
    if (Q > 1) __syncthreads();                             // (of one tile wave 0 clears and uses all: at most 63 chunks)
    if (wave < Q) {                                         // the leader's tiles: the largest word of every chunk
        const float4 x = accumulate4(m, g, lr);
        const uint32_t key[4] = {magnitude_key(x.x), magnitude_key(x.y), magnitude_key(x.z), magnitude_key(x.w)};
        // a lane's elements lie in one chunk or, around a boundary, in two or more: one atomic per run
        unsigned long long word = 0ull;
        uint32_t cur = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t p = p0 + c;
            if (p < lo || p >= hi) continue;
            const uint32_t j = ((p - lo) * recip) >> 22;
            const unsigned long long w = (static_cast<unsigned long long>(key[c]) << 32) | (0xffffffffu - p);
            if (word != 0ull && j != cur) {
                atomicMax(&best[cur], word);
                word = 0ull;
            }
            cur = j;
            word = w > word ? w : word;
        }
        if (word != 0ull) atomicMax(&best[cur], word);
    }
    __syncthreads();
    for (int p = wave; p < n_pairs; p += n_waves) {
        if (p != wave) {
            place(p, l, p0);
            fetch(l, p0);
        }
        if (p0 >= hi) continue;
        const float4 x = accumulate4(m, g, lr);
        const float xv[4] = {x.x, x.y, x.z, x.w}, mv[4] = {m.x, m.y, m.z, m.w};
        float out[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t pos = p0 + c;
            const uint32_t rel = pos >= lo ? pos - lo : 0u;
            const uint32_t j = (rel * recip) >> 22;
            const bool in = pos >= lo && pos < hi;
            const bool sel = in && static_cast<uint32_t>(best[in ? j : 0u]) == 0xffffffffu - pos;
            if (sel) xs[j * n_learners + l] = xv[c];
            out[c] = fmaf(beta, sel ? 0.0f : xv[c], one_minus_beta * mv[c]);   // Eq. 5
        }
        store_guarded(lp.mem[l], p0, lo, hi, p0 >= lo && p0 + 3 < hi, make_float4(out[0], out[1], out[2], out[3]));
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < n_ch; j += blockDim.x) {   // Alg. 1 line 10, learner 0 first
        const uint32_t slot = static_cast<uint32_t>(d.out_base) + cf + j;
        float s = xs[j * n_learners];
        for (int i = 1; i < n_learners; ++i) s = s + xs[j * n_learners + i];
        idx_out[slot] = static_cast<int32_t>(0xffffffffu - static_cast<uint32_t>(best[j]));
        red_out[slot] = s;
    }
}

// The same for layouts with more data, where blocks of all learners, whose positions do not start on whole kilobytes, cost more than
// further launches: the leader by itself first, one wave per group of whole chunks (at most 256 * Q - 3 positions,
// the same groups as above).  A wave's chunks are nobody else's, so it finds their winners, updates the leader's memory
// in the same pass and leaves the winners in idx_out and the leader's values there in vals; the leader is read once.  No atomics in memory
// and nothing to clear.  Bound by memory (25.6 M, chunk 112: 55 us, 5.6 TB/s, with one tile per wave, 62 with four, whose registers leave fewer
// waves; without any work in LDS 54) once the reduction is left to LDS: a maximum per chunk, then the lowest position among the holders (one
// atomic per lane and run each, in words of the wave's own).  Where its positions begin makes no difference: groups laid on whole 128-byte lines, or an eighth of
// the vector per XCD, took as long.  8 x 25.6 M, us a step, winners / winners and memory in this pass: 420 / 387, 3 x 30 M 205 / 179,
// 1 x 30 M 74 (one launch) / 64.
constexpr int kChunkGroupMax = 256;              // chunks of a group at most (1021 positions, chunks of 4)

template <typename G, int Q>
__global__ void __launch_bounds__(kBlock)
k_chunk_lead(float* __restrict__ mem, const G* __restrict__ grad, float lr, float beta, float one_minus_beta,
             const StDesc* __restrict__ sts, int n_st, int32_t* __restrict__ idx_out, float* __restrict__ vals)
{
    constexpr int kMost = Q == 4 ? kChunkGroupMax : 64 * Q;
    __shared__ uint32_t key_max[kWaves][kMost], pos_min[kWaves][kMost];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes), lane = threadIdx.x % kLanes;
    const int st = static_cast<int>(blockIdx.y + blockIdx.z * gridDim.y);
    if (st >= n_st) return;
    const StDesc d = sts[st];
    ChunkGroup<Q> c;
    if (!c.find(d, blockIdx.x * kWaves + wave)) return;     // whole wave
    float4 m[Q], x[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t p0 = c.base + static_cast<uint32_t>(q * kWaveTile + lane * kVec);
        m[q] = make_float4(0, 0, 0, 0);
        x[q] = m[q];
        if (p0 < c.hi) {
            const bool whole = p0 >= c.begin && p0 + 3 < c.end;
            m[q] = load_guarded(mem, p0, c.begin, c.end, whole);
            x[q] = load_guarded(grad, p0, c.begin, c.end, whole);
        }
    }
    for (uint32_t j = lane; j < c.n; j += kLanes) {
        key_max[wave][j] = 0u;
        pos_min[wave][j] = 0xffffffffu;
    }
    wave_lds_fence();
    // A lane's elements belong to chunk j0 up to element nb, then to the next one.  Keys fit 31 bits, so -1 stands for
    // an element outside the group.
    auto key_of = [&](int q, int e) {
        const uint32_t p = c.base + static_cast<uint32_t>(q * kWaveTile + lane * kVec + e);
        const float v = e == 0 ? x[q].x : e == 1 ? x[q].y : e == 2 ? x[q].z : x[q].w;
        return p >= c.lo && p < c.hi ? static_cast<int32_t>(magnitude_key(v)) : -1;
    };
    uint32_t j0[Q], nb[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t p0 = c.base + static_cast<uint32_t>(q * kWaveTile + lane * kVec);
        x[q] = accumulate4(m[q], x[q], lr);
        const uint32_t rel = p0 > c.lo ? p0 - c.lo : 0u;
        j0[q] = (rel * c.recip) >> 22;
        nb[q] = c.lo + (j0[q] + 1u) * c.ch - p0;            // (at least 1; lane 0 may begin up to 3 before lo)
        int32_t head = -1, tail = -1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int32_t key = key_of(q, e);
            if (static_cast<uint32_t>(e) < nb[q])
                head = key > head ? key : head;
            else
                tail = key > tail ? key : tail;
        }
        if (head >= 0) atomicMax(&key_max[wave][j0[q]], static_cast<uint32_t>(head));
        if (tail >= 0) atomicMax(&key_max[wave][j0[q] + 1u], static_cast<uint32_t>(tail));
    }
    wave_lds_fence();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t p0 = c.base + static_cast<uint32_t>(q * kWaveTile + lane * kVec);
        const bool two = nb[q] < 4u && p0 + nb[q] < c.hi;
        const int32_t best0 = p0 < c.hi ? static_cast<int32_t>(key_max[wave][j0[q]]) : 0;
        const int32_t best1 = two ? static_cast<int32_t>(key_max[wave][j0[q] + 1u]) : 0;
        uint32_t at0 = 0xffffffffu, at1 = 0xffffffffu;
#pragma unroll
        for (int e = 3; e >= 0; --e) {
            if (static_cast<uint32_t>(e) < nb[q])
                at0 = key_of(q, e) == best0 ? p0 + e : at0;
            else
                at1 = key_of(q, e) == best1 ? p0 + e : at1;
        }
        if (at0 != 0xffffffffu) atomicMin(&pos_min[wave][j0[q]], at0);
        if (at1 != 0xffffffffu) atomicMin(&pos_min[wave][j0[q] + 1u], at1);
    }
    wave_lds_fence();
    const uint32_t slot0 = static_cast<uint32_t>(c.out_base) + c.first;
    for (uint32_t j = lane; j < c.n; j += kLanes) idx_out[slot0 + j] = static_cast<int32_t>(pos_min[wave][j]);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t p0 = c.base + static_cast<uint32_t>(q * kWaveTile + lane * kVec);
        if (p0 >= c.hi) continue;
        const bool two = nb[q] < 4u && p0 + nb[q] < c.hi;
        const uint32_t w0 = pos_min[wave][j0[q]], w1 = two ? pos_min[wave][j0[q] + 1u] : 0xffffffffu;
        const float xv[4] = {x[q].x, x[q].y, x[q].z, x[q].w}, mv[4] = {m[q].x, m[q].y, m[q].z, m[q].w};
        float out[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool sel = p0 + e == w0 || p0 + e == w1;
            if (sel) vals[slot0 + j0[q] + (p0 + e == w0 ? 0u : 1u)] = xv[e];
            out[e] = fmaf(beta, sel ? 0.0f : xv[e], one_minus_beta * mv[e]);   // Eq. 5
        }
        store_guarded(mem, p0, c.lo, c.hi, p0 >= c.lo && p0 + 3 < c.hi, make_float4(out[0], out[1], out[2], out[3]));
    }
}

// The other learners then, with the winners at hand: k_update's blocks and order, but an element is a member if
// its chunk's entry of idx_out names it, and the chunk is the slot.  (The masks and slots per wave tile that
// k_update reads would take one more launch.)  For chunks of 4 to 1021 elements.
template <typename G>
__global__ void __launch_bounds__(kBlock)
k_update_chunks(LearnerPtrs lp, float lr, float beta, float one_minus_beta, const StDesc* __restrict__ sts, int n_st,
                const int32_t* __restrict__ idx, float* __restrict__ vals, int64_t k_total, int leader, bool eighths)
{
    int learner = blockIdx.y;
    learner += learner >= leader ? 1 : 0;                   // (the leader's memory is updated already)
    const int group = update_group(n_st, eighths);
    if (group < 0) return;
    const int st = group / kUpdateBlocksPerSuper;
    const StDesc d = sts[st];
    const uint32_t begin = static_cast<uint32_t>(d.begin), end = static_cast<uint32_t>(d.end);
    const uint32_t blk0 = static_cast<uint32_t>(d.a0) + static_cast<uint32_t>(group % kUpdateBlocksPerSuper) * kWaves * kWaveTile;
    const uint32_t v_lo = blk0 > begin ? blk0 : begin;      // the block's positions of the segment
    const uint32_t v_hi = blk0 + kWaves * kWaveTile < end ? blk0 + kWaves * kWaveTile : end;
    if (v_lo >= v_hi) return;                               // whole block
    const uint32_t p0 = blk0 + threadIdx.x * kVec;
    const bool inside = blk0 >= begin && blk0 + kWaves * kWaveTile <= end;     // block-uniform
    const bool full = inside || (p0 >= begin && p0 + 3 < end), any = inside || (p0 + 3 >= begin && p0 < end);
    float* mem = lp.mem[learner];
    const G* grad = static_cast<const G*>(lp.grad[learner]);
    float4 m = make_float4(0, 0, 0, 0), g = m;
    if (inside) {
        m = load4(mem + p0);
        g = load4(grad + p0);
    } else if (any) {
        m = load_guarded(mem, p0, begin, end, full);
        g = load_guarded(grad, p0, begin, end, full);
    }
    // chunk numbers from the supertile's first one on; x / ch for x < 16384 and ch < 1024 by a product: the
    // reciprocal is 2^32 / ch rounded up, or more by at most its float's last bits (one element per chunk: x is 0)
    const uint32_t ch = static_cast<uint32_t>(d.sel_chunk);
    const uint32_t recip = static_cast<uint32_t>(4294968320.0f * __builtin_amdgcn_rcpf(static_cast<float>(ch > 1u ? ch : 2u))) + 1u;
    auto over_ch = [&](uint32_t x) { return __umulhi(x, recip); };
    const uint32_t c0 = static_cast<uint32_t>(d.chunk_first), start0 = begin + c0 * ch;   // (at most a0 + ch)
    // the chunk that holds the block's first position: the one before c0, or one from c0 on
    const uint32_t j_lo = v_lo < start0 ? c0 - 1u : c0 + over_ch(v_lo - start0);
    const uint32_t lo_pos = begin + j_lo * ch;
    const uint32_t n_j = over_ch(v_hi - 1u - lo_pos) + 1u;  // chunks that the block has a part of
    const int32_t* my_idx = idx + d.out_base + j_lo;
    const uint32_t q0 = p0 > v_lo ? p0 : v_lo, q3 = p0 + 3 < v_hi ? p0 + 3 : v_hi - 1u;
    const uint32_t r0 = any ? over_ch(q0 - lo_pos) : 0u, r3 = any ? over_ch(q3 - lo_pos) : 0u;
    const uint32_t w0 = static_cast<uint32_t>(my_idx[r0]), w3 = static_cast<uint32_t>(my_idx[r3]);
    __shared__ float stage[kWaves * kWaveTile / 4 + 2];
    const uint32_t win_t = threadIdx.x < n_j ? static_cast<uint32_t>(my_idx[threadIdx.x]) : 0xffffffffu;
    const float4 x = accumulate4(m, g, lr);
    const float xv[4] = {x.x, x.y, x.z, x.w}, mv[4] = {m.x, m.y, m.z, m.w};
    float out[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t p = p0 + c;
        const bool sel = (p == w0 || p == w3) && p >= v_lo && p < v_hi;
        if (sel) stage[p == w0 ? r0 : r3] = xv[c];
        out[c] = fmaf(beta, sel ? 0.0f : xv[c], one_minus_beta * mv[c]);       // Eq. 5
    }
    const float4 o = make_float4(out[0], out[1], out[2], out[3]);
    if (inside)
        store4(mem + p0, o);
    else if (any)
        store_guarded(mem, p0, begin, end, full, o);
    __syncthreads();
    float* my_vals = vals + static_cast<size_t>(learner) * static_cast<size_t>(k_total) + d.out_base + j_lo;
    if (win_t >= v_lo && win_t < v_hi) my_vals[threadIdx.x] = stage[threadIdx.x];
    for (uint32_t j = kBlock + threadIdx.x; j < n_j; j += kBlock) {            // (chunks of 4: up to 257)
        const uint32_t w = static_cast<uint32_t>(my_idx[j]);
        if (w >= v_lo && w < v_hi) my_vals[j] = stage[j];
    }
}

// Chunks beyond those sizes: maxima per chunk by atomics, then masks and slots for k_update.
// Leader pass of the chunk-wise selector, one wave per wave tile: every element becomes the word
// (magnitude key << 32 | ~position), so that the largest word of a chunk is its largest
// magnitude at the lowest position; for each chunk of the tile's segment that overlaps the tile
// the wave reduces its part and merges it into best[out_base + chunk] with one 64-bit atomic max
// (a chunk touches at most chunk/256 + 2 tiles).  Chunks are counted from the segment's first
// element.  Also clears the tile's membership mask.
template <typename G>
__global__ void __launch_bounds__(kBlock)
k_chunk_select(const float* __restrict__ mem, const G* __restrict__ grad, float lr, const SegDesc* __restrict__ segs,
               const StDesc* __restrict__ sts, int n_st, unsigned long long* __restrict__ best,
               uint64_t* __restrict__ sel_mask)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes), lane = threadIdx.x % kLanes;
    const int64_t group = static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;   // 4 wave tiles
    const int st = static_cast<int>(group / kUpdateBlocksPerSuper);
    if (st >= n_st) return;                                 // whole block
    const int wt = static_cast<int>(group % kUpdateBlocksPerSuper) * kWaves + wave;
    const StDesc d = sts[st];
    const SegDesc sd = segs[d.seg];
    const size_t tile = static_cast<size_t>(st) * kTilesPerSuper + wt;
    if (lane == 0) {
        const uint64_t zero[4] = {0, 0, 0, 0};
        store_tile_masks(sel_mask, tile, zero);
    }
    // positions and chunk sizes are below 2^31 + 8192: 32-bit arithmetic throughout
    const uint32_t begin = static_cast<uint32_t>(sd.begin), end = static_cast<uint32_t>(sd.end);
    const uint32_t ch = static_cast<uint32_t>(sd.sel_chunk);
    const uint32_t tile_first = static_cast<uint32_t>(d.a0) + static_cast<uint32_t>(wt) * kWaveTile;
    const uint32_t v_lo = tile_first > begin ? tile_first : begin;             // the tile's part of the segment
    const uint32_t v_hi = tile_first + kWaveTile < end ? tile_first + kWaveTile : end;
    if (v_lo >= v_hi) return;                               // whole wave: the tile lies outside the segment
    const uint32_t p0 = tile_first + lane * kVec;
    float4 m, g;
    if (tile_first >= begin && tile_first + kWaveTile <= end) {   // wave-uniform: the whole tile belongs to the segment
        m = load4(mem + p0);
        g = load4(grad + p0);
    } else {
        leader_load(mem, grad, p0, static_cast<int64_t>(begin), static_cast<int64_t>(end), m, g);
    }
    const float4 x = accumulate4(m, g, lr);
    const uint32_t key[4] = {magnitude_key(x.x), magnitude_key(x.y), magnitude_key(x.z), magnitude_key(x.w)};
    const uint32_t j_first = (v_lo - begin) / ch, j_last = (v_hi - 1 - begin) / ch;
    uint32_t lo = begin + j_first * ch;                     // at most v_lo: no overflow
    for (uint32_t j = j_first; j <= j_last; ++j, lo += ch) { // wave-uniform trip count
        // positions of chunk j: lo <= p < lo + chunk, i.e. p - lo < chunk (unsigned; lo + chunk may pass 2^32),
        // and p < end.  The largest word (key << 32 | ~position) in two 32-bit steps: the largest key,
        // then the largest ~position among the elements that have it.  ~position is never 0, so a
        // result of 0 means that no element of the chunk lies in this tile.
        bool in[4];
        uint32_t k_here = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            in[c] = p0 + c - lo < ch && p0 + c < end;
            if (in[c] && key[c] > k_here) k_here = key[c];
        }
        const uint32_t k_max = wave_max_u32(k_here);
        uint32_t inv_here = 0;                              // element c = 0 has the largest ~position of the lane
#pragma unroll
        for (int c = 3; c >= 0; --c)
            if (in[c] && key[c] == k_max) inv_here = 0xffffffffu - (p0 + c);
        const uint32_t inv_max = wave_max_u32(inv_here);
        if (lane == 0)
            atomicMax(&best[static_cast<uint32_t>(sd.out_base) + j],
                      (static_cast<unsigned long long>(k_max) << 32) | inv_max);
    }
}

// After the leader pass: position of each chunk's winner to idx_out and to the membership mask;
// first output slot of every wave tile (chunk j of a segment owns slot out_base + j).  (best[] is
// zeroed again by the all-learner pass that follows.)
__global__ void __launch_bounds__(kBlock)
k_chunk_marks(const SegDesc* __restrict__ segs, int n_tensors, const StDesc* __restrict__ sts,
              const unsigned long long* __restrict__ best, int64_t k_total, int64_t n_tiles,
              uint64_t* __restrict__ sel_mask, uint32_t* __restrict__ tile_slot, int32_t* __restrict__ idx_out)
{
    const int64_t t = (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * kBlock + threadIdx.x;
    if (t < k_total) {
        // the segment that owns output slot t: the last one whose first slot is <= t (a segment without
        // slots shares its first slot with its successor, so it is never the last such one while t < k_total)
        int lo = 0, hi = n_tensors - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (segs[mid].out_base <= t) lo = mid; else hi = mid - 1;
        }
        const SegDesc sd = segs[lo];
        const uint32_t pos = 0xffffffffu - static_cast<uint32_t>(best[t]);
        idx_out[t] = static_cast<int32_t>(pos);
        if (pos >= static_cast<uint32_t>(sd.begin) && pos < static_cast<uint32_t>(sd.end)) {   // always, unless best[] was corrupted
            const uint32_t rel = pos - (static_cast<uint32_t>(sd.begin) & ~static_cast<uint32_t>(kVec - 1));
            const size_t tile = static_cast<size_t>(sd.st_first) * kTilesPerSuper + rel / kWaveTile;
            const uint32_t l = (rel % kWaveTile) / kVec, c = rel % kVec;
            atomicOr(reinterpret_cast<uint32_t*>(sel_mask) + (tile * 4 + c) * 2 + (l >> 5), 1u << (l & 31));
        }
    }
    if (t < n_tiles) {
        // winners of the segment before this tile: one per chunk that ends before it, plus the
        // straddling chunk's winner if it lies before the tile
        const StDesc d = sts[t / kTilesPerSuper];
        const SegDesc sd = segs[d.seg];
        const uint32_t begin = static_cast<uint32_t>(sd.begin), end = static_cast<uint32_t>(sd.end);
        const uint32_t ch = static_cast<uint32_t>(sd.sel_chunk);
        const uint32_t first = static_cast<uint32_t>(d.a0) + static_cast<uint32_t>(t % kTilesPerSuper) * kWaveTile;
        uint32_t slot = static_cast<uint32_t>(sd.out_base);
        if (first >= end) {
            slot += static_cast<uint32_t>(sd.k);            // past the segment: its mask is empty
        } else if (first > begin) {
            const uint32_t j = (first - begin) / ch;
            slot += j;
            if (begin + j * ch < first) {
                const uint32_t pos = 0xffffffffu - static_cast<uint32_t>(best[static_cast<uint32_t>(sd.out_base) + j]);
                if (pos < first) ++slot;
            }
        }
        tile_slot[t] = slot;
    }
}

}  // namespace
