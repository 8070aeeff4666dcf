// Spatial index of a reference cloud and the exact nearest-neighbour search
// (Eq. 1) over it.
//
// Index: the references in the order of a balanced k-d partition, kFan to a
// leaf, under a tree of axis-aligned boxes of fan-out kFan. Level 0 holds the
// points (x, y, z, original index), level 1 one box per leaf, level l + 1 one
// box per kFan boxes of level l, up to a level of at most kFan boxes. Every
// level is padded to whole blocks of kFan entries: points by copies of a
// point of their leaf, boxes by empty ones, which no query can enter. Any
// order of the points gives a correct index; the order only decides how tight
// the boxes are. (Morton order needs no splits but took 2 to 3.5 times the
// blocks per query: 24.9 against 7.3 for the 100,000-point street scan.)
//
// Search: kFan lanes share a query, kWave / kFan queries share a wavefront.
// One step loads the kFan entries of a block, one per lane, forms each lane's
// squared distance, and descends into the nearest entry that the best
// distance so far does not exclude; a lane keeps the distances of the levels
// above in LDS, so that a finished block resumes its parent where it left
// off. A point is a box without extent, so that points and boxes take one
// code path and queries of a wavefront that stand at different levels do not
// diverge.
//
// Exactness: the FP32 distance of a point p of a box [lo, hi] is
// fma(dz, dz, fma(dy, dy, dx dx)) with dx = fl(q - p). Rounding is monotone
// and lo <= p <= hi, so |dx| >= max(fl(lo - q), fl(q - hi), 0), and products
// and sums of non-negative terms keep the order: the same expression over
// those three bounds never exceeds the point's distance, with no margin. A
// block is skipped only when its bound is larger than a distance that was
// found, so the result is the smallest (distance, index) key of the whole
// cloud, ties to the lowest index as in the brute-force search, bit for bit.
//
// Figures and what bounds the search: at index_nn_kernel.
#pragma once

#include <algorithm>
#include <utility>
#include <vector>

#include "common.hpp"

namespace sicp {

constexpr int kFan = 16;                    // entries per block, lanes per query
constexpr int kIndexLevels = 8;             // most levels, the points included
constexpr int kIndexThreads = 256;
constexpr int kChunk = kFan * kFan * kFan;  // slots a workgroup of the build orders in LDS
constexpr int kChunkThreads = kChunk / 4;
constexpr int64_t kIndexMaxRef = (int64_t)1 << 24;   // block numbers and offsets then stay small integers

// One indexed cloud. Offsets are in float4 elements of the context's index
// array; a point takes one, a box two (lower and upper corner).
struct IndexDesc {
    int64_t ref_off;                  // packed references (original order)
    int64_t n;                        // real references
    int64_t level_off[kIndexLevels];
    int32_t levels;                   // levels in use, points included
    int32_t chunks;                   // chunks of at most kChunk points
};

// ------------------------------------------------------------------- build
// A cloud of more than kChunk points is first cut into chunks of equal size:
// rounds of splits, each cutting a segment of chunks into up to four parts
// along its longest side at exact ranks (a histogram of the coordinate, then
// a partition; points of a bin that holds a cut go to either side of it).
// Parts are multiples of 16^j chunks, so that a block of any level is a cell
// of the partition. One workgroup then orders each chunk in LDS and writes
// its three lower levels; a last launch forms the levels above.
constexpr int kSplitBins = 2048;
constexpr int kSplitThreads = 256;
constexpr int kSplitTile = 8 * kSplitThreads;
constexpr int kSplitParts = 4;

struct IndexSeg {
    int64_t src;                    // first point, in the source array of its round
    int64_t dst;                    // the same in the round's output array
    int32_t n, parts;
    int32_t cut[kSplitParts - 1];   // ranks of the cuts
    int32_t child;                  // number of the first part's segment, the others follow
    int32_t tile0;                  // first tile of the segment in its round
};

struct IndexTile {
    int32_t seg, first;             // segment, and the tile's first point in it
};

struct IndexChunk {
    int64_t src;                    // first point, in the source array
    int32_t n, slots;               // points, and slots (a power of two >= n, at least kFan^2)
    int32_t from;                   // source: -1 the packed references, else an array of the split rounds
    int32_t desc, number;           // cloud, and the chunk's number in it
};

// What the build of a context's clouds reads: written by the host, uploaded
// as one block.
struct IndexPlan {
    std::vector<IndexDesc> desc;
    std::vector<IndexSeg> seg;
    std::vector<IndexTile> tile;        // by round
    std::vector<int32_t> round_tile;    // first tile of each round, and the end
    std::vector<IndexTile> top_tile;    // tiles of the clouds that are cut (their bounding boxes)
    std::vector<IndexChunk> chunk;
    int64_t nodes = 0;                  // float4 elements of all levels
    int64_t points = 0;                 // points of the clouds that are cut
    bool uppers = false;                // some cloud has levels above its chunks
};

// Plan for clouds (ref_off, n); false where a cloud is too large.
inline bool index_plan(const std::vector<std::pair<int64_t, int64_t>>& clouds, IndexPlan& pl)
{
    struct Node {
        int32_t seg, c0, cn, desc;      // chunks [c0, c0 + cn) of the cloud
        int64_t per, off;               // points per chunk, the cloud's offset in the split arrays
    };
    std::vector<Node> open;
    for (const auto& cl : clouds) {
        const int64_t n = cl.second;
        if (n > kIndexMaxRef) return false;
        IndexDesc d{};
        d.ref_off = cl.first;
        d.n = n;
        const int32_t di = (int32_t)pl.desc.size();
        auto level = [&](int64_t elements) {
            d.level_off[d.levels++] = pl.nodes;
            pl.nodes += elements;
        };
        if (n <= kChunk) {
            int32_t slots = kFan * kFan;
            while (slots < n) slots *= 2;
            d.chunks = 1;
            level(slots);
            level(2 * slots / kFan);
            if (slots > kFan * kFan) level(2 * kFan);
            pl.chunk.push_back(IndexChunk{cl.first, (int32_t)n, slots, -1, di, 0});
        } else {
            const int64_t s0 = (n + kChunk - 1) / kChunk;
            const int64_t per = ((n + s0 - 1) / s0 + kFan - 1) / kFan * kFan;
            const int64_t S = (n + per - 1) / per;
            d.chunks = (int32_t)S;
            level(S * kChunk);
            level(2 * S * kFan * kFan);
            level(2 * S * kFan);
            for (int64_t e = S;; e = (e + kFan - 1) / kFan) {   // entries of the level
                level(2 * ((e + kFan - 1) / kFan * kFan));
                if (e <= kFan) break;
            }
            pl.uppers = true;
            const int32_t sg = (int32_t)pl.seg.size();
            pl.seg.push_back(IndexSeg{cl.first, pl.points, (int32_t)n, 0, {0, 0, 0}, 0, 0});
            open.push_back(Node{sg, 0, (int32_t)S, di, per, pl.points});
            for (int64_t f = 0; f < n; f += kSplitTile) pl.top_tile.push_back(IndexTile{sg, (int32_t)f});
            pl.points += n;
        }
        pl.desc.push_back(d);
    }
    for (int round = 0; !open.empty(); ++round) {
        pl.round_tile.push_back((int32_t)pl.tile.size());
        std::vector<Node> next;
        for (const Node& nd : open) {
            int32_t unit = 1;
            while (unit * kFan < nd.cn) unit *= kFan;
            const int32_t units = (nd.cn + unit - 1) / unit;
            const int32_t parts = std::min<int32_t>(kSplitParts, units);
            const int32_t child = (int32_t)pl.seg.size();
            IndexSeg sg = pl.seg[nd.seg];
            sg.parts = parts;
            sg.child = child;
            sg.tile0 = (int32_t)pl.tile.size();
            for (int64_t f = 0; f < sg.n; f += kSplitTile) pl.tile.push_back(IndexTile{nd.seg, (int32_t)f});
            for (int32_t k = 0; k < parts; ++k) {
                const int32_t a = std::min(nd.cn, units * k / parts * unit);
                const int32_t b = std::min(nd.cn, units * (k + 1) / parts * unit);
                const int64_t pa = a * nd.per, pb = std::min<int64_t>(b * nd.per, sg.n);
                if (k) sg.cut[k - 1] = (int32_t)pa;
                const int64_t at = sg.dst + pa;
                pl.seg.push_back(IndexSeg{at, at, (int32_t)(pb - pa), 0, {0, 0, 0}, 0, 0});
                if (b - a > 1)
                    next.push_back(Node{child + k, nd.c0 + a, b - a, nd.desc, nd.per, nd.off});
                else
                    pl.chunk.push_back(IndexChunk{at, (int32_t)(pb - pa), kChunk, round & 1, nd.desc, nd.c0 + a});
            }
            pl.seg[nd.seg] = sg;
        }
        open.swap(next);
    }
    pl.round_tile.push_back((int32_t)pl.tile.size());
    return true;
}

// Order-preserving map of a finite float to an unsigned integer above 0.
__device__ __forceinline__ uint32_t order_bits(float x)
{
    const uint32_t b = __float_as_uint(x);
    return (b >> 31) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float from_order_bits(uint32_t o)
{
    return __uint_as_float((o >> 31) ? (o & 0x7fffffffu) : ~o);
}

// Per segment: the bounding box (largest order bits of x, y, z and of their
// complements), the fill of each part and the arrivals at each cut's bin.
struct IndexSegState {
    uint32_t box[6];
    uint32_t fill[kSplitParts], arrived[kSplitParts - 1];
    uint32_t pad_[3];
};

struct IndexBuildArgs {
    const IndexDesc* desc;
    const IndexSeg* seg;
    const IndexTile* tile;
    const IndexChunk* chunk;
    const float4* ref4;
    float4* nodes;
    float4* split[2];       // outputs of the even and the odd rounds
    IndexSegState* state;   // per segment, zeroed before
    uint32_t* hist;         // per segment: kSplitBins counts, zeroed before
    int32_t round, pad_;
};

// Point j of a segment in the round's input, its original index in w.
__device__ __forceinline__ float4 split_point(const IndexBuildArgs& a, const IndexSeg& sg, int64_t j)
{
    if (a.round > 0) return a.split[(a.round - 1) & 1][sg.src + j];
    float4 p = a.ref4[sg.src + j];
    p.w = __uint_as_float((uint32_t)j);
    return p;
}

// Longest side of a box of order bits: its axis, lower end and the factor
// that takes the coordinate to [0, steps).
__device__ __forceinline__ void split_axis(const uint32_t* __restrict__ box, float steps, int& axis, float& lo,
                                           float& scale)
{
    axis = 0;
    lo = 0.f;
    float side = -1.f;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const float l = from_order_bits(~box[3 + e]), len = from_order_bits(box[e]) - l;
        if (len > side) {
            side = len;
            lo = l;
            axis = e;
        }
    }
    scale = side > 0.f ? steps / side : 0.f;
}

__device__ __forceinline__ float coord(float4 p, int axis) { return axis == 0 ? p.x : (axis == 1 ? p.y : p.z); }

__device__ __forceinline__ int split_bin(float c, float lo, float scale)
{
    return (int)fminf(fmaxf((c - lo) * scale, 0.f), (float)(kSplitBins - 1));
}

// Fold a thread's box (largest order bits of the coordinates and of their
// complements) over the wavefront into dst.
__device__ __forceinline__ void fold_box(const uint32_t (&v)[6], uint32_t* dst)
{
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        uint32_t x = v[e];
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) x = max(x, (uint32_t)__shfl_xor((int)x, o));
        if ((threadIdx.x & (kWave - 1)) == 0 && x) atomicMax(dst + e, x);
    }
}

__device__ __forceinline__ void grow_box(uint32_t (&v)[6], float4 p)
{
    const uint32_t o[3] = {order_bits(p.x), order_bits(p.y), order_bits(p.z)};
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        v[e] = max(v[e], o[e]);
        v[3 + e] = max(v[3 + e], ~o[e]);
    }
}

// Bounding boxes of the clouds that are cut; a workgroup per tile.
__global__ __launch_bounds__(kSplitThreads) void index_bounds_kernel(IndexBuildArgs a)
{
    const IndexTile t = a.tile[blockIdx.x];
    const IndexSeg sg = a.seg[t.seg];
    uint32_t v[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < kSplitTile / kSplitThreads; ++u) {
        const int j = t.first + u * kSplitThreads + (int)threadIdx.x;
        grow_box(v, a.ref4[sg.src + min(j, sg.n - 1)]);
    }
    fold_box(v, a.state[t.seg].box);
}

// Histogram of the segments' coordinates along their longest sides.
__global__ __launch_bounds__(kSplitThreads) void index_hist_kernel(IndexBuildArgs a)
{
    __shared__ uint32_t cnt[kSplitBins];
    const IndexTile t = a.tile[blockIdx.x];
    const IndexSeg sg = a.seg[t.seg];
    for (int b = threadIdx.x; b < kSplitBins; b += kSplitThreads) cnt[b] = 0;
    int axis;
    float lo, scale;
    split_axis(a.state[t.seg].box, (float)kSplitBins, axis, lo, scale);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSplitTile / kSplitThreads; ++u) {
        const int j = t.first + u * kSplitThreads + (int)threadIdx.x;
        if (j < sg.n) atomicAdd(&cnt[split_bin(coord(split_point(a, sg, j), axis), lo, scale)], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kSplitBins; b += kSplitThreads)
        if (cnt[b]) atomicAdd(a.hist + (int64_t)t.seg * kSplitBins + b, cnt[b]);
}

// Cut the segments: every point goes to the part its rank by bin (and, in a
// bin that holds a cut, by arrival) falls in; the parts' boxes follow.
__global__ __launch_bounds__(kSplitThreads) void index_split_kernel(IndexBuildArgs a)
{
    constexpr int BPT = kSplitBins / kSplitThreads;
    constexpr int CUTS = kSplitParts - 1;
    __shared__ uint32_t wsum[kSplitThreads / kWave];
    __shared__ int cut_bin[CUTS];
    __shared__ uint32_t cut_below[CUTS], count[kSplitParts], base[kSplitParts];
    __shared__ int cut_rank[CUTS];
    const IndexTile t = a.tile[blockIdx.x];
    const IndexSeg sg = a.seg[t.seg];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const uint32_t* h = a.hist + (int64_t)t.seg * kSplitBins + BPT * tid;
    uint32_t c[BPT], sum = 0;
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
        c[b] = h[b];
        sum += c[b];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)inc, o);
        if (lane >= o) inc += v;
    }
    if (lane == kWave - 1) wsum[wave] = inc;
    if (tid < kSplitParts) count[tid] = 0;
    if (tid < CUTS) {
        cut_bin[tid] = kSplitBins;
        cut_below[tid] = 0;
        cut_rank[tid] = tid < sg.parts - 1 ? a.seg[t.seg].cut[tid] : sg.n;
    }
    __syncthreads();
    uint32_t run = inc - sum;
    for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
#pragma unroll
        for (int k = 0; k < CUTS; ++k)
            if (k < sg.parts - 1 && run <= (uint32_t)sg.cut[k] && (uint32_t)sg.cut[k] < run + c[b]) {
                cut_bin[k] = BPT * tid + b;
                cut_below[k] = run;
            }
        run += c[b];
    }
    __syncthreads();
    int axis;
    float lo, scale;
    split_axis(a.state[t.seg].box, (float)kSplitBins, axis, lo, scale);
    float4 pt[kSplitTile / kSplitThreads];
    int part[kSplitTile / kSplitThreads];
    uint32_t slot[kSplitTile / kSplitThreads];
#pragma unroll
    for (int u = 0; u < kSplitTile / kSplitThreads; ++u) {
        const int j = t.first + u * kSplitThreads + tid;
        part[u] = -1;
        if (j >= sg.n) continue;
        pt[u] = split_point(a, sg, j);
        const int b = split_bin(coord(pt[u], axis), lo, scale);
        int p = 0, in = -1;
#pragma unroll
        for (int k = CUTS - 1; k >= 0; --k) {
            if (cut_bin[k] < b) ++p;
            if (cut_bin[k] == b) in = k;
        }
        if (in >= 0) {
            const uint32_t rank = cut_below[in] + atomicAdd(&a.state[t.seg].arrived[in], 1u);
            p = 0;
#pragma unroll
            for (int k = 0; k < CUTS; ++k)
                if ((uint32_t)cut_rank[k] <= rank) ++p;   // ranks stay below n
        }
        part[u] = p;
        slot[u] = atomicAdd(&count[p], 1u);
    }
    __syncthreads();
    if (tid < sg.parts) base[tid] = atomicAdd(&a.state[t.seg].fill[tid], count[tid]);
    __syncthreads();
    float4* out = a.split[a.round & 1] + sg.dst;
#pragma unroll
    for (int u = 0; u < kSplitTile / kSplitThreads; ++u)
        if (part[u] >= 0) {
            const int64_t at = (part[u] ? (int64_t)cut_rank[part[u] - 1] : 0) + base[part[u]] + slot[u];
            if (at < sg.n) out[at] = pt[u];
        }
    for (int k = 0; k < sg.parts; ++k) {
        uint32_t v[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < kSplitTile / kSplitThreads; ++u)
            if (part[u] == k) grow_box(v, pt[u]);
        fold_box(v, a.state[sg.child + k].box);
    }
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
// Lane exchanges of reductions over 2, 4, 8 and 16 lanes.
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141, kDppMirror = 0x140;

// LDS written by the wavefront's other lanes may be read after this (the
// LDS serves a wavefront in order: only the compiler must keep to it).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Order one chunk and write its points and its three lower box levels (two,
// or one, where a lone chunk's points need no more). kChunkThreads threads,
// thread t at slots 4 t .. 4 t + 3; slots past the points are padding, which
// sorts to the end. A segment of s slots (first the whole chunk) is sorted
// along its longest side and quartered, down to leaves of kFan slots; keys
// hold 20 bits of the coordinate in the segment's box and 12 of the point's
// number, so that the sorts move 4 bytes per slot.
__global__ __launch_bounds__(kChunkThreads) void index_chunk_kernel(IndexBuildArgs a)
{
    __shared__ float xyz[3][kChunk];
    __shared__ uint32_t orig[kChunk];
    __shared__ uint32_t key[kChunk];
    __shared__ uint32_t gbox[6][kChunk / 64];   // boxes of 64 slots, then of their segment
    const IndexChunk ch = a.chunk[blockIdx.x];
    const IndexDesc& d = a.desc[ch.desc];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const float4* src = (ch.from < 0 ? a.ref4 : a.split[ch.from]) + ch.src;
    for (int i = tid; i < kChunk; i += kChunkThreads) {
        key[i] = (uint32_t)i;
        if (i < ch.n) {
            const float4 p = src[i];
            xyz[0][i] = p.x;
            xyz[1][i] = p.y;
            xyz[2][i] = p.z;
            orig[i] = ch.from < 0 ? (uint32_t)i : __float_as_uint(p.w);
        }
    }
    __syncthreads();
    // box of the points in this thread's four slots, as order bits
    auto slots_box = [&](uint32_t (&v)[6]) {
#pragma unroll
        for (int e = 0; e < 6; ++e) v[e] = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t i = key[4 * tid + u] & (kChunk - 1);
            if ((int)i < ch.n) grow_box(v, make_float4(xyz[0][i], xyz[1][i], xyz[2][i], 0.f));
        }
    };
    int s = ch.slots;
    while (s > kFan) {
        uint32_t v[6];
        slots_box(v);
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            v[e] = max(v[e], dpp<kDppXor1>(v[e]));
            v[e] = max(v[e], dpp<kDppXor2>(v[e]));
            v[e] = max(v[e], dpp<kDppHalfMirror>(v[e]));   // 32 slots
        }
        if (s > 32) {
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                v[e] = max(v[e], dpp<kDppMirror>(v[e]));   // 64 slots
                if ((lane & 15) == 0) gbox[e][tid / 16] = v[e];
            }
            __syncthreads();
            if (wave < 6) {
                uint32_t x = gbox[wave][lane];
                for (int o = 1; o < s / 64; o <<= 1) x = max(x, (uint32_t)__shfl_xor((int)x, o));
                gbox[wave][lane] = x;
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 6; ++e) v[e] = gbox[e][tid / 16];
        }
        int axis;
        float lo, scale;
        split_axis(v, 1048574.f, axis, lo, scale);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t i = key[4 * tid + u] & (kChunk - 1);
            uint32_t q = 0xfffffu;   // padding
            if ((int)i < ch.n) q = (uint32_t)fminf(fmaxf((xyz[axis][i] - lo) * scale, 0.f), 1048574.f);
            key[4 * tid + u] = (q << 12) | i;
        }
        __syncthreads();
        // bitonic sort of every segment, ascending. Pair p of a step of
        // distance j holds slots i = 2 j (p / j) + p % j and i + j; a
        // wavefront's 64 consecutive pairs stay inside 128 slots for j <= 64
        for (int k = 2; k <= s; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int p = h * kChunkThreads + tid;
                    const int i = ((p & ~(j - 1)) << 1) | (p & (j - 1));
                    if (i < ch.slots) {
                        const uint32_t x = key[i], y = key[i + j];
                        const bool up = (i & k) == 0 || k == s;
                        if (up == (x > y)) {
                            key[i] = y;
                            key[i + j] = x;
                        }
                    }
                }
                if (j > 64 || (j == 1 && k >= 64)) __syncthreads();
                else wave_sync();
            }
        __syncthreads();
        s = s >= 4 * kFan ? s / 4 : s / 2;
    }
    // points; padding copies the first point of its leaf
    float4* pts = a.nodes + d.level_off[0] + (int64_t)ch.number * kChunk;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int at = u * kChunkThreads + tid;
        if (at < ch.slots) {
            uint32_t i = key[at] & (kChunk - 1);
            if ((int)i >= ch.n) i = key[at & ~(kFan - 1)] & (kChunk - 1);
            if ((int)i >= ch.n) i = 0;
            pts[at] = make_float4(xyz[0][i], xyz[1][i], xyz[2][i], __uint_as_float(orig[i]));
        }
    }
    // boxes: a leaf is four threads, a box of level 2 a wavefront
    auto put = [&](int64_t at, const uint32_t (&v)[6]) {
        const float inf = __builtin_inff();
        const bool any = v[0] != 0;   // order bits of a number are above 0
        a.nodes[at] = any ? make_float4(from_order_bits(~v[3]), from_order_bits(~v[4]), from_order_bits(~v[5]), 0.f)
                          : make_float4(inf, inf, inf, 0.f);
        a.nodes[at + 1] = any ? make_float4(from_order_bits(v[0]), from_order_bits(v[1]), from_order_bits(v[2]), 0.f)
                              : make_float4(-inf, -inf, -inf, 0.f);
    };
    uint32_t v[6];
    slots_box(v);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        v[e] = max(v[e], dpp<kDppXor1>(v[e]));
        v[e] = max(v[e], dpp<kDppXor2>(v[e]));
    }
    if ((tid & 3) == 0 && 4 * tid < ch.slots)
        put(d.level_off[1] + 2 * ((int64_t)ch.number * (kFan * kFan) + tid / 4), v);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        v[e] = max(v[e], dpp<kDppHalfMirror>(v[e]));
        v[e] = max(v[e], dpp<kDppMirror>(v[e]));
        v[e] = max(v[e], (uint32_t)__shfl_xor((int)v[e], 16));
        v[e] = max(v[e], (uint32_t)__shfl_xor((int)v[e], 32));
        if (lane == 0) gbox[e][wave] = v[e];
    }
    if (lane == 0 && d.levels > 2) put(d.level_off[2] + 2 * ((int64_t)ch.number * kFan + wave), v);
    __syncthreads();
    if (d.levels > 3 && tid == 0) {
        for (int e = 0; e < 6; ++e)
            for (int w = 0; w < kChunkThreads / kWave; ++w) v[e] = max(v[e], gbox[e][w]);
        put(d.level_off[3] + 2 * (int64_t)ch.number, v);
    }
}

// The levels above the chunks of the clouds that are cut, one workgroup per
// cloud, a thread per box; level 3 (a box per chunk) only gets its padding.
__global__ __launch_bounds__(kIndexThreads) void index_upper_kernel(IndexBuildArgs a)
{
    const IndexDesc& d = a.desc[blockIdx.x];
    int64_t below = d.chunks;
    for (int l = 3; l < d.levels; ++l) {
        const int64_t real = l == 3 ? below : (below + kFan - 1) / kFan;
        const int64_t padded = (real + kFan - 1) / kFan * kFan;
        for (int64_t e = (l == 3 ? real : 0) + threadIdx.x; e < padded; e += kIndexThreads) {
            const float inf = __builtin_inff();
            float4 lo = make_float4(inf, inf, inf, 0.f), hi = make_float4(-inf, -inf, -inf, 0.f);
            if (e < real) {
                const float4* c = a.nodes + d.level_off[l - 1] + 2 * e * kFan;   // padding boxes are empty
#pragma unroll 4
                for (int u = 0; u < kFan; ++u) {
                    const float4 x = c[2 * u], y = c[2 * u + 1];
                    lo.x = fminf(lo.x, x.x);
                    lo.y = fminf(lo.y, x.y);
                    lo.z = fminf(lo.z, x.z);
                    hi.x = fmaxf(hi.x, y.x);
                    hi.y = fmaxf(hi.y, y.y);
                    hi.z = fmaxf(hi.z, y.z);
                }
            }
            a.nodes[d.level_off[l] + 2 * e] = lo;
            a.nodes[d.level_off[l] + 2 * e + 1] = hi;
        }
        __threadfence_block();
        __syncthreads();
        below = real;
    }
}

// ------------------------------------------------------------------ search
// Minimum over the kFan = 16 lanes of a query.
__device__ __forceinline__ uint32_t fan_min(uint32_t v)
{
    v = min(v, dpp<kDppXor1>(v));
    v = min(v, dpp<kDppXor2>(v));
    v = min(v, dpp<kDppHalfMirror>(v));
    v = min(v, dpp<kDppMirror>(v));
    return v;
}

template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v)
{
    return ((uint64_t)dpp<CTRL>((uint32_t)(v >> 32)) << 32) | dpp<CTRL>((uint32_t)v);
}

__device__ __forceinline__ uint64_t fan_min64(uint64_t v)
{
    auto take = [&](uint64_t o) { v = o < v ? o : v; };
    take(dpp64<kDppXor1>(v));
    take(dpp64<kDppXor2>(v));
    take(dpp64<kDppHalfMirror>(v));
    take(dpp64<kDppMirror>(v));
    return v;
}

struct IndexSearchArgs {
    const IndexDesc* desc;    // per cloud
    const int32_t* cloud;     // cloud of each pair (NULL: cloud 0)
    const float4* nodes;
    const float4* ref4;
    const float4* queries;    // pair p's at p K m: query k m + i
    uint64_t* keys;           // (distance bits, original index), as the queries
    int32_t K, m;
    int32_t run, pad_;        // consecutive queries per group of lanes
};

// Key of no match yet: distance infinity, reference 0 (what the brute-force
// search returns where no distance is finite).
constexpr uint64_t kIndexNoMatch = 0x7f80000000000000ull;

// grid (ceil(K m / run / (kIndexThreads / kFan)), pairs). A group of kFan
// lanes takes `run` queries in turn; queries are ordered by minibatch point,
// then particle, so that the groups of a wavefront and the turns of a group
// look for (nearly) the same place: they read the same blocks, and the match
// of one query bounds the next one's search from the start.
//
// Bound by the instructions and the load latency of the dependent steps, 5
// (2,000 references) to 8 (100,000) blocks a query; the whole index stays in
// L2. Against the brute-force searches, per launch: 300,000 queries x 100,000
// street references 1,055 -> 112 us (FP16 screen), 30,000 x 20,000 tabletop
// 34 -> 14 us, 16,247 x 12,345 85 -> 10 us (BF16 screen), 10,000 x 2,000
// 9.9 -> 9.0 us (FP32); 64 uneven pairs of 30,000 queries 1,114 -> 523 us.
__global__ __launch_bounds__(kIndexThreads) void index_nn_kernel(IndexSearchArgs a)
{
    __shared__ uint32_t above[kIndexLevels][kIndexThreads];   // a lane's remaining distances, per level
    __shared__ int64_t level_off[kIndexLevels];
    const int tid = threadIdx.x;
    const int64_t p = blockIdx.y;
    const IndexDesc& d = a.desc[a.cloud ? a.cloud[p] : 0];
    const int top = d.levels - 1;
    if (tid < kIndexLevels) level_off[tid] = d.level_off[tid];
    __syncthreads();
    const uint32_t fl = tid & (kFan - 1);
    const int64_t nq = (int64_t)a.K * a.m;
    int64_t w = ((int64_t)blockIdx.x * (kIndexThreads / kFan) + tid / kFan) * a.run;
    const int64_t wend = min(w + a.run, nq);
    if (w >= wend) return;   // no barrier below
    const float4* __restrict__ ref4 = a.ref4 + d.ref_off;
    int32_t k = (int32_t)(w % a.K), i = (int32_t)(w / a.K);
    uint64_t key = kIndexNoMatch;
    float4 q;
    uint32_t bound;
    auto start = [&] {
        q = a.queries[p * nq + (int64_t)k * a.m + i];
        // the previous match is a reference like any other: its distance
        // bounds the search from the start
        const uint32_t j = (uint32_t)key;
        const float4 r = ref4[j];
        const float d0 = dist2_f32(q.x, q.y, q.z, r.x, r.y, r.z);
        const uint64_t k0 = pack_key(d0, j);
        key = k0 < kIndexNoMatch ? k0 : kIndexNoMatch;
        // no distance of a query with a NaN is a number: nothing to search
        const bool nan = !(q.x == q.x && q.y == q.y && q.z == q.z);
        bound = nan ? 0u : (uint32_t)(key >> 32);
        if (nan) q = make_float4(__builtin_inff(), 0.f, 0.f, 0.f);
    };
    start();
    int level = top;
    uint32_t block = 0;
    for (;;) {
        // distances of the block's entries
        const uint32_t e = block * kFan + fl;
        const bool box = level > 0;
        const float4* src = a.nodes + level_off[level] + (box ? 2 * (int64_t)e : (int64_t)e);
        const float4 lo = src[0];
        const float4 hi = src[box ? 1 : 0];
        uint32_t cur;
        {
#pragma clang fp contract(off)
            const float dx = __builtin_fmaxf(__builtin_fmaxf(lo.x - q.x, q.x - hi.x), 0.f);
            const float dy = __builtin_fmaxf(__builtin_fmaxf(lo.y - q.y, q.y - hi.y), 0.f);
            const float dz = __builtin_fmaxf(__builtin_fmaxf(lo.z - q.z, q.z - hi.z), 0.f);
            cur = __float_as_uint(__builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx)));
        }
        if (!box) {
            const uint64_t here = ((uint64_t)cur << 32) | __float_as_uint(lo.w);
            key = here < key ? here : key;
            bound = min(bound, fan_min(cur));
            level = 1;
            block /= kFan;
            cur = above[1][tid];
        }
        // the nearest entry left, of this block or of the levels above: the
        // low bits of its distance make room for the lane (rounded down, so
        // the bound still holds)
        uint32_t best;
        for (;;) {
            best = fan_min((cur & ~(uint32_t)(kFan - 1)) | fl);
            if (((best & ~(uint32_t)(kFan - 1)) <= bound && best < 0x7f800000u) || level == top) break;
            ++level;
            block /= kFan;
            cur = above[level][tid];
        }
        if ((best & ~(uint32_t)(kFan - 1)) <= bound && best < 0x7f800000u) {
            const uint32_t c = best & (kFan - 1);
            above[level][tid] = c == fl ? 0x7f800000u : cur;
            --level;
            block = block * kFan + c;
        } else {
            key = fan_min64(key);
            if (fl == 0) a.keys[p * nq + (int64_t)k * a.m + i] = key;
            if (++w >= wend) break;
            if (++k == a.K) {
                k = 0;
                ++i;
            }
            start();
            level = top;
            block = 0;
        }
    }
}

}  // namespace sicp
