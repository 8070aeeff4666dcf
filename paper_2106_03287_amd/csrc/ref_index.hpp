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
// Search: L lanes share a query, kWave / L queries a wavefront. One step takes
// the kFan entries of a block, kFan / L per lane, forms their squared
// distances, and descends into the nearest entry that the best distance so
// far does not exclude; a lane keeps the distances of the levels above in
// LDS, so that a finished block resumes its parent where it left off. A point
// is a box without extent, so that points and boxes take one code path and
// queries of a wavefront that stand at different levels do not diverge.
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

constexpr int kFan = 16;                    // entries per block, and points per leaf
constexpr int kIndexLevels = 8;             // most levels, the points included
constexpr int kIndexThreads = 256;
constexpr int kChunk = kFan * kFan * kFan;  // slots a workgroup of the build orders in LDS
constexpr int kChunkThreads = kChunk / 4;
constexpr int64_t kIndexMaxRef = (int64_t)1 << 24;   // block numbers and offsets then stay small integers

// One indexed cloud. Offsets are in float4 elements of the context's index
// array. Entries are stored by fours, coordinate by coordinate: a quad of
// points is x, y, z, original index; a quad of boxes the lower x, y, z and the
// upper x, y, z.
constexpr int kPointQuad = 4, kBoxQuad = 6;   // float4 elements
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
// Parts are multiples of kFan^j chunks, so that a block of a level above the
// chunks is (nearly) a cell of the partition. One workgroup then orders each chunk in LDS and writes
// its boxes; a last launch forms the levels above.
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
    int32_t n, slots;               // points, and slots (a power of two >= n, at least 256)
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
        auto take = [&](int64_t elements) {
            const int64_t o = pl.nodes;
            pl.nodes += elements;
            return o;
        };
        // points, then boxes until one block holds a level
        auto levels = [&](int64_t slots) {
            d.level_off[d.levels++] = take(slots / 4 * kPointQuad);
            for (int64_t e = slots / kFan;; e = (e + kFan - 1) / kFan) {
                d.level_off[d.levels++] = take((e + kFan - 1) / kFan * kFan / 4 * kBoxQuad);
                if (e <= kFan) break;
            }
        };
        if (n <= kChunk) {
            int32_t slots = kFan * kFan;
            while (slots < n) slots *= 2;
            d.chunks = 1;
            levels(slots);
            pl.chunk.push_back(IndexChunk{cl.first, (int32_t)n, slots, -1, di, 0});
        } else {
            const int64_t s0 = (n + kChunk - 1) / kChunk;
            const int64_t per = ((n + s0 - 1) / s0 + kFan - 1) / kFan * kFan;
            const int64_t S = (n + per - 1) / per;
            d.chunks = (int32_t)S;
            levels(S * kChunk);
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

// Box number `box` of a level.
__device__ __forceinline__ void put_box(float4* level, int64_t box, const float (&lo)[3], const float (&hi)[3])
{
    float* o = (float*)(level + box / 4 * kBoxQuad) + box % 4;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        o[4 * e] = lo[e];
        o[12 + 4 * e] = hi[e];
    }
}

// LDS written by the wavefront's other lanes may be read after this (the
// LDS serves a wavefront in order: only the compiler must keep to it).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Order one chunk and write its points and its boxes of 16, 256 and 4096
// slots, as far as the cloud has those levels. kChunkThreads threads,
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
    float* pts = (float*)(a.nodes + d.level_off[0] + (int64_t)ch.number * (kChunk / 4 * kPointQuad));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int at = u * kChunkThreads + tid;
        if (at < ch.slots) {
            uint32_t i = key[at] & (kChunk - 1);
            if ((int)i >= ch.n) i = key[at & ~(kFan - 1)] & (kChunk - 1);
            if ((int)i >= ch.n) i = 0;
            float* o = pts + 4 * kPointQuad * (at / 4) + at % 4;
            o[0] = xyz[0][i];
            o[4] = xyz[1][i];
            o[8] = xyz[2][i];
            o[12] = __uint_as_float(orig[i]);
        }
    }
    // boxes: 16 slots are four threads, 256 a wavefront
    auto put = [&](int level, int64_t box, const uint32_t (&v)[6]) {
        const float inf = __builtin_inff();
        const bool any = v[0] != 0;   // order bits of a number are above 0
        float lo[3], hi[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            lo[e] = any ? from_order_bits(~v[3 + e]) : inf;
            hi[e] = any ? from_order_bits(v[e]) : -inf;
        }
        put_box(a.nodes + d.level_off[level], box, lo, hi);
    };
    uint32_t v[6];
    slots_box(v);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        v[e] = max(v[e], dpp<kDppXor1>(v[e]));
        v[e] = max(v[e], dpp<kDppXor2>(v[e]));
    }
    if ((tid & 3) == 0 && 4 * tid < ch.slots) put(1, (int64_t)ch.number * (kFan * kFan) + tid / 4, v);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        v[e] = max(v[e], dpp<kDppHalfMirror>(v[e]));
        v[e] = max(v[e], dpp<kDppMirror>(v[e]));
        v[e] = max(v[e], (uint32_t)__shfl_xor((int)v[e], 16));
        v[e] = max(v[e], (uint32_t)__shfl_xor((int)v[e], 32));
        if (lane == 0) gbox[e][wave] = v[e];
    }
    if (lane == 0 && d.levels > 2) put(2, (int64_t)ch.number * kFan + wave, v);   // idle wavefronts pad the block
    __syncthreads();
    if (d.levels > 3 && tid == 0) {
        for (int e = 0; e < 6; ++e)
            for (int w = 0; w < kChunkThreads / kWave; ++w) v[e] = max(v[e], gbox[e][w]);
        put(3, ch.number, v);
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
            float lo[3] = {inf, inf, inf}, hi[3] = {-inf, -inf, -inf};
            if (e < real) {   // the children are one block; padding boxes are empty
                const float4* c = a.nodes + d.level_off[l - 1] + e * (kFan / 4 * kBoxQuad);
                for (int u = 0; u < kFan / 4; ++u)
#pragma unroll
                    for (int f = 0; f < 3; ++f) {
                        const float4 x = c[u * kBoxQuad + f], y = c[u * kBoxQuad + 3 + f];
                        lo[f] = fminf(lo[f], fminf(fminf(x.x, x.y), fminf(x.z, x.w)));
                        hi[f] = fmaxf(hi[f], fmaxf(fmaxf(y.x, y.y), fmaxf(y.z, y.w)));
                    }
            }
            put_box(a.nodes + d.level_off[l], e, lo, hi);
        }
        __threadfence_block();
        __syncthreads();
        below = real;
    }
}

// ------------------------------------------------------------------ search
// Minimum over the L = 4 or 16 lanes of a query.
template <int L>
__device__ __forceinline__ uint32_t lanes_min(uint32_t v)
{
    v = min(v, dpp<kDppXor1>(v));
    v = min(v, dpp<kDppXor2>(v));
    if (L == 16) {
        v = min(v, dpp<kDppHalfMirror>(v));
        v = min(v, dpp<kDppMirror>(v));
    }
    return v;
}

template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v)
{
    return ((uint64_t)dpp<CTRL>((uint32_t)(v >> 32)) << 32) | dpp<CTRL>((uint32_t)v);
}

template <int L>
__device__ __forceinline__ uint64_t lanes_min64(uint64_t v)
{
    auto take = [&](uint64_t o) { v = o < v ? o : v; };
    take(dpp64<kDppXor1>(v));
    take(dpp64<kDppXor2>(v));
    if (L == 16) {
        take(dpp64<kDppHalfMirror>(v));
        take(dpp64<kDppMirror>(v));
    }
    return v;
}

// E consecutive entries of one coordinate row of a quad.
template <int E>
struct alignas(4 * E) Row {
    float v[E];
};

struct IndexSearchArgs {
    const IndexDesc* desc;    // per cloud
    const int32_t* cloud;     // cloud of each pair (NULL: cloud 0)
    const float4* nodes;
    const float4* queries;    // pair p's at p K m: query k m + i
    uint64_t* keys;           // (distance bits, original index), as the queries
    int32_t K, m;
};

// Key of no match yet: distance infinity, reference 0 (what the brute-force
// search returns where no distance is finite).
constexpr uint64_t kIndexNoMatch = 0x7f80000000000000ull;

// Threads of a search workgroup: 16 queries. Larger ones hold their slots
// until the last of more queries ends (4 lanes, street scan: 64 threads 62.6
// us a launch, 128 65.0, 256 66.6).
constexpr int search_threads(int lanes) { return 16 * lanes; }

// Dynamic LDS: a thread's remaining distances, per box level.
template <int L>
inline size_t index_nn_lds_bytes(int levels)
{
    return (size_t)(levels - 1) * search_threads(L) * (kFan / L) * 4;
}

// grid (ceil(K m / 16), pairs), search_threads(L) threads; dynamic LDS
// index_nn_lds_bytes<L>(most levels of the clouds). A query to L lanes; the
// queries are ordered by minibatch point, then particle, so that those of a
// wavefront look for (nearly) the same place and read the same blocks.
//
// Bound by the vector instructions and the latency of the dependent steps, 5
// (2,000 references) to 8 (100,000) a query; the whole index stays in L2.
// us a launch with 4 and with 16 lanes (what it replaced: the brute-force
// search of the mode): 300,000 queries of 100,000 street references 63 and 85
// (1,055), 64 uneven pairs of 30,000 queries 348 and 506 (1,114), 1,000 runs
// of 300 queries of 20,000 68 and 80 (231), 30,000 of 20,000 tabletop 17.4
// and 13.9 (34), 16,247 of 12,345 13.1 and 10.2 (85), 10,000 of 2,000 11.8
// and 9.1 (9.9). Left out after measuring: upper levels staged in LDS
// (slower throughout: the staging and the occupancy cost more than the
// loads), a second query in turn per group (street 72 -> 82), fan-out 64 on
// 16 lanes (tabletop 16.6, street 112) and 4 on one lane (41, 94).
template <int L>
__global__ __launch_bounds__(search_threads(L)) void index_nn_kernel(IndexSearchArgs a)
{
    constexpr int T = search_threads(L);
    constexpr int E = kFan / L;                   // entries of a block per lane
    constexpr uint32_t kInf = 0x7f800000u, kEntry = kFan - 1;
    extern __shared__ float4 lds4[];
    Row<E>* above = (Row<E>*)lds4;                // [box level - 1][thread]
    __shared__ int32_t level_off[kIndexLevels];
    const int tid = threadIdx.x;
    const int64_t p = blockIdx.y;
    const IndexDesc& d = a.desc[a.cloud ? a.cloud[p] : 0];
    const int top = d.levels - 1;
    const float* __restrict__ nodes = (const float*)(a.nodes + d.level_off[0]);
    const uint32_t fl = tid & (L - 1);
    if (tid < kIndexLevels) level_off[tid] = 4 * (int32_t)(d.level_off[tid] - d.level_off[0]);
    __syncthreads();
    const uint32_t nq = (uint32_t)a.K * (uint32_t)a.m;   // at most 2^31
    const uint32_t w = blockIdx.x * (T / L) + tid / L;
    if (w >= nq) return;   // whole groups; no barrier below
    const uint64_t qi = p * (uint64_t)nq + (uint64_t)(w % (uint32_t)a.K) * (uint32_t)a.m + w / (uint32_t)a.K;
    float4 q = a.queries[qi];
    uint64_t key = kIndexNoMatch;
    uint32_t bound = kInf;
    // no distance of a query with a NaN is a number: nothing to search
    if (!(q.x == q.x && q.y == q.y && q.z == q.z)) q = make_float4(__builtin_inff(), 0.f, 0.f, 0.f);
    const uint32_t quad0 = fl * E / 4, place = fl * E % 4;
    int level = top;
    uint32_t block = 0;
    for (;;) {
        // this lane's entries of the block, and their distances
        const bool box = level > 0;
        const uint32_t quad = block * (kFan / 4) + quad0;
        const uint32_t at = (uint32_t)level_off[level] + 16 * quad + (box ? 8 * quad : 0) + place;
        const Row<E>* src = (const Row<E>*)(nodes + at);
        const Row<E>* up = (const Row<E>*)(nodes + at + (box ? 12 : 0));
        const Row<E> lx = src[0], ly = src[4 / E], lz = src[8 / E], hx = up[0], hy = up[4 / E], hz = up[8 / E];
        uint32_t cur[E];
#pragma unroll
        for (int u = 0; u < E; ++u) {
#pragma clang fp contract(off)
            const float dx = __builtin_fmaxf(__builtin_fmaxf(lx.v[u] - q.x, q.x - hx.v[u]), 0.f);
            const float dy = __builtin_fmaxf(__builtin_fmaxf(ly.v[u] - q.y, q.y - hy.v[u]), 0.f);
            const float dz = __builtin_fmaxf(__builtin_fmaxf(lz.v[u] - q.z, q.z - hz.v[u]), 0.f);
            cur[u] = __float_as_uint(__builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx)));
        }
        auto least = [&] {
            uint32_t v = cur[0];
#pragma unroll
            for (int u = 1; u < E; ++u) v = min(v, cur[u]);
            return lanes_min<L>(v);
        };
        auto resume = [&](int lv) {   // the distances left of a block of level lv
            const Row<E> r = above[(lv - 1) * T + tid];
#pragma unroll
            for (int u = 0; u < E; ++u) cur[u] = __float_as_uint(r.v[u]);
        };
        if (box) {
            // the low bits make room for the entry (rounded down, so the
            // bound still holds): the smallest value names the nearest entry
#pragma unroll
            for (int u = 0; u < E; ++u) cur[u] = (cur[u] & ~kEntry) | (E * fl + u);
        } else {
            const Row<E> id = src[12 / E];
#pragma unroll
            for (int u = 0; u < E; ++u) {
                const uint64_t o = ((uint64_t)cur[u] << 32) | __float_as_uint(id.v[u]);
                key = o < key ? o : key;
            }
            bound = min(bound, least());
            level = 1;
            block /= kFan;
            resume(1);
        }
        // the nearest entry left, of this block or of the levels above
        uint32_t best;
        bool open;
        for (;;) {
            best = least();
            open = (best & ~kEntry) <= bound && best < kInf;
            if (open || level == top) break;
            resume(++level);
            block /= kFan;
        }
        if (!open) break;
        Row<E> r;
#pragma unroll
        for (int u = 0; u < E; ++u) r.v[u] = __uint_as_float(cur[u] == best ? kInf : cur[u]);
        --level;
        above[level * T + tid] = r;
        block = block * kFan + (best & kEntry);
    }
    key = lanes_min64<L>(key);
    if (fl == 0) a.keys[qi] = key;
}

}  // namespace sicp
