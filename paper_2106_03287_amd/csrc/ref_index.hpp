// Spatial index of a reference cloud and the exact nearest-neighbour search
// (Eq. 1) over it.
//
// Index: the references in the order of a balanced k-d partition, kFan to a
// leaf, under a tree of axis-aligned boxes of fan-out kFan. Level 0 holds the
// points (x, y, z, original index), level 1 one box per leaf, level l + 1 one
// box per kFan boxes of level l, up to a level of at most kFan boxes. Every
// level is padded to whole blocks of kFan entries: points by copies of a
// point of their leaf, numbered kNoPoint, boxes by empty ones (both corners at
// infinity), which no query can enter. Any
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
// and lo <= p <= hi, so |dx| >= |fl(q - c)| for the box's nearest coordinate
// c = med(q, lo, hi), and products and sums of non-negative terms keep the
// order: the same expression over those three differences never exceeds the
// point's distance, with no margin. A
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
#include "svgd_select.hpp"

namespace sicp {

constexpr int kFan = 16;                    // entries per block, and points per leaf
constexpr uint32_t kNoPoint = 0xffffffffu;  // number of a padding point: loses every tie to the point it copies
constexpr int kIndexLevels = 8;             // most levels, the points included
constexpr int kIndexThreads = 256;
constexpr int kChunk = kFan * kFan * kFan;  // slots a workgroup of the build orders in LDS
constexpr int kChunkThreads = kChunk / 4;
constexpr int kCoincident = 2 * kFan;       // of coincident references a search finds so many, at least as many as any asks for
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

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
// Lane exchanges of reductions over 2, 4, 8 and 16 lanes.
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141, kDppMirror = 0x140;
// The lane before (0 for the first of 16; or its last).
constexpr int kDppShr1 = 0x111, kDppRor1 = 0x121;

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

// Fold the threads' boxes (largest order bits of the coordinates and of their
// complements) over the wavefront into dst, in LDS.
__device__ __forceinline__ void fold_box(const uint32_t (&v)[6], uint32_t* dst)
{
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        uint32_t x = v[e];
        x = max(x, dpp<kDppXor1>(x));
        x = max(x, dpp<kDppXor2>(x));
        x = max(x, dpp<kDppHalfMirror>(x));
        x = max(x, dpp<kDppMirror>(x));
        if ((threadIdx.x & 15) == 0 && x) atomicMax(dst + e, x);
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
    __shared__ uint32_t box[6];
    if (threadIdx.x < 6) box[threadIdx.x] = 0;
    __syncthreads();
    fold_box(v, box);
    __syncthreads();
    if (threadIdx.x < 6) atomicMax(a.state[t.seg].box + threadIdx.x, box[threadIdx.x]);
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
// bin that holds a cut, by arrival) falls in; the parts' boxes follow. Bound by
// latency: the arrivals and the parts' fills take one global atomic per
// workgroup and counter (a global atomic per arrival and four LDS counters for
// every point: 25.8 us a round on 100,000 points, against 13.2).
__global__ __launch_bounds__(kSplitThreads) void index_split_kernel(IndexBuildArgs a)
{
    constexpr int BPT = kSplitBins / kSplitThreads, CUTS = kSplitParts - 1, N = kSplitTile / kSplitThreads;
    constexpr int W = kSplitThreads / kWave;
    __shared__ uint32_t wsum[W];
    __shared__ int cut_bin[CUTS], cut_rank[CUTS];
    __shared__ uint32_t cut_below[CUTS], arrived[CUTS], arrived0[CUTS];
    __shared__ uint32_t count[W][kSplitParts], base[kSplitParts], box[kSplitParts][6];
    const IndexTile t = a.tile[blockIdx.x];
    const IndexSeg sg = a.seg[t.seg];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    int axis;
    float lo, scale;
    split_axis(a.state[t.seg].box, (float)kSplitBins, axis, lo, scale);
    float4 pt[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int j = t.first + u * kSplitThreads + tid;
        pt[u] = split_point(a, sg, min(j, sg.n - 1));
    }
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
    if (tid < 6 * kSplitParts) (&box[0][0])[tid] = 0;
    if (tid < CUTS) {
        cut_bin[tid] = kSplitBins;
        cut_below[tid] = 0;
        arrived[tid] = 0;
        cut_rank[tid] = tid < sg.parts - 1 ? a.seg[t.seg].cut[tid] : sg.n;
    }
    __syncthreads();
    uint32_t run = inc - sum;
    for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
#pragma unroll
        for (int k = 0; k < CUTS; ++k)
            if (run <= (uint32_t)cut_rank[k] && (uint32_t)cut_rank[k] < run + c[b]) {   // no bin for rank n
                cut_bin[k] = BPT * tid + b;
                cut_below[k] = run;
            }
        run += c[b];
    }
    __syncthreads();
    // the part of every point; of one in a cut's bin, its arrival there
    int part[N], in[N];
    uint32_t slot[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int b = split_bin(coord(pt[u], axis), lo, scale);
        part[u] = 0;
        in[u] = -1;
#pragma unroll
        for (int k = CUTS - 1; k >= 0; --k) {
            if (cut_bin[k] < b) ++part[u];
            if (cut_bin[k] == b) in[u] = k;
        }
        if (t.first + u * kSplitThreads + tid >= sg.n) part[u] = in[u] = -1;
        if (in[u] >= 0) slot[u] = atomicAdd(&arrived[in[u]], 1u);
    }
    __syncthreads();
    if (tid < CUTS && arrived[tid]) arrived0[tid] = cut_below[tid] + atomicAdd(&a.state[t.seg].arrived[tid], arrived[tid]);
    __syncthreads();
    uint32_t mine[kSplitParts] = {0, 0, 0, 0};   // the wavefront's points of each part so far
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (in[u] >= 0) {
            const uint32_t rank = arrived0[in[u]] + slot[u];
            part[u] = 0;
#pragma unroll
            for (int k = 0; k < CUTS; ++k)
                if ((uint32_t)cut_rank[k] <= rank) ++part[u];   // ranks stay below n
        }
#pragma unroll
        for (int k = 0; k < kSplitParts; ++k) {
            const uint64_t m = __ballot(part[u] == k);
            if (part[u] == k) slot[u] = mine[k] + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull));
            mine[k] += (uint32_t)__builtin_popcountll(m);
        }
    }
    if (lane == 0)
        for (int k = 0; k < kSplitParts; ++k) count[wave][k] = mine[k];
    __syncthreads();
    if (tid < sg.parts) {
        uint32_t n = 0;
        for (int w = 0; w < W; ++w) {
            const uint32_t x = count[w][tid];
            count[w][tid] = n;
            n += x;
        }
        base[tid] = (tid ? (uint32_t)cut_rank[tid - 1] : 0u) + atomicAdd(&a.state[t.seg].fill[tid], n);
    }
    for (int k = 0; k < sg.parts; ++k) {
        uint32_t v[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (part[u] == k) grow_box(v, pt[u]);
        fold_box(v, box[k]);
    }
    __syncthreads();
    float4* out = a.split[a.round & 1] + sg.dst;
#pragma unroll
    for (int u = 0; u < N; ++u)
        if (part[u] >= 0) {
            const uint32_t at = base[part[u]] + count[wave][part[u]] + slot[u];
            if (at < (uint32_t)sg.n) out[at] = pt[u];
        }
    if (tid < 6 * sg.parts) atomicMax(a.state[sg.child + tid / 6].box + tid % 6, box[tid / 6][tid % 6]);
}

// Order one chunk and write its points and its boxes of 16, 256 and 4096
// slots, as far as the cloud has those levels. kChunkThreads threads, thread t
// at slots 4 t .. 4 t + 3; slots past the points are padding, which sorts to
// the end. A segment of s slots (first the whole chunk) is sorted along its
// longest side and quartered, down to leaves of kFan slots. The sort counts
// into s bins of equal width: points of a bin keep any order, which only
// loosens a box where a quarter ends inside a bin. Bound by the latency of
// its four passes over LDS: 25 us, also for many chunks (a bitonic sort of
// keys of 20 bits of the coordinate took 53 us for 2,048 slots and 77 for
// 4,096).
// References that coincide (the zeros of a scanner's empty returns) fill leaves
// of the same single point, which a search that ends there would have to visit
// all: its bound excludes no tie. Of three such leaves and more in a row, the
// first two take the kCoincident lowest indices, more than any answer holds, and
// the others get empty boxes: their points are found in no search. 100,000
// queries of 100,000 street references, 30 % of both zero: 71 us a launch,
// 2,798 with every leaf visited (1,436 by brute force in FP32); all zero 131,
// 15,263 and 1,331. A wavefront takes a run of such leaves: one workgroup for
// one run after another made a stand-alone search of a cloud of 492 such places
// 506 us, 271 so and 266 without looking for them. To look takes about 1 us of
// the launch.
__global__ __launch_bounds__(kChunkThreads) void index_chunk_kernel(IndexBuildArgs a)
{
    __shared__ float xyz[3][kChunk];
    __shared__ uint32_t orig[kChunk];
    __shared__ uint16_t order[kChunk];          // point of each slot
    __shared__ uint32_t hist[kChunk], wsum[kChunkThreads / kWave];
    __shared__ uint32_t gbox[6][kChunk / 64];   // boxes of 64 slots, then of their segment
    const IndexChunk ch = a.chunk[blockIdx.x];
    const IndexDesc& d = a.desc[ch.desc];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const float4* src = (ch.from < 0 ? a.ref4 : a.split[ch.from]) + ch.src;
    for (int i = tid; i < kChunk; i += kChunkThreads) {
        order[i] = (uint16_t)i;
        hist[i] = 0;
        if (i < ch.n) {
            const float4 p = src[i];
            xyz[0][i] = p.x + 0.f;   // -0 as 0: one place, and the same distances
            xyz[1][i] = p.y + 0.f;
            xyz[2][i] = p.z + 0.f;
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
            const uint32_t i = order[4 * tid + u];
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
        // counting sort of every segment along its longest side, as many
        // bins as slots, the last one for padding
        int axis;
        float lo, scale;
        split_axis(v, (float)(s - 1), axis, lo, scale);
        const int seg0 = 4 * tid & ~(s - 1);
        uint32_t pid[4], rank[4];
        int bin[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            pid[u] = order[4 * tid + u];
            bin[u] = seg0 + s - 1;
            if ((int)pid[u] < ch.n)
                bin[u] = seg0 + (int)fminf(fmaxf((xyz[axis][pid[u]] - lo) * scale, 0.f), (float)(s - 2));
            rank[u] = atomicAdd(&hist[bin[u]], 1u);
        }
        __syncthreads();
        uint32_t c[4], sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u] = hist[4 * tid + u];
            sum += c[u];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t x = (uint32_t)__shfl_up((int)inc, o);
            if (lane >= o) inc += x;
        }
        if (lane == kWave - 1) wsum[wave] = inc;
        __syncthreads();
        uint32_t run = inc - sum;
        for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            hist[4 * tid + u] = run;
            run += c[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) order[hist[bin[u]] + rank[u]] = (uint16_t)pid[u];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) hist[4 * tid + u] = 0;   // the next barrier lies before its use
        s = s >= 4 * kFan ? s / 4 : s / 2;
    }
    // boxes of the leaves: four threads each
    uint32_t v[6];
    auto leaf_box = [&] {
        slots_box(v);
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            v[e] = max(v[e], dpp<kDppXor1>(v[e]));
            v[e] = max(v[e], dpp<kDppXor2>(v[e]));
        }
    };
    leaf_box();
    // coincident references
    constexpr int kLeaves = kChunk / kFan;
    uint32_t* at_leaf = hist;   // the one point of each leaf, as order bits; 0: none
    const int leaf = tid / 4;
    __syncthreads();
    if ((tid & 3) == 0) {
        const bool one = v[0] != 0 && v[0] == ~v[3] && v[1] == ~v[4] && v[2] == ~v[5];
#pragma unroll
        for (int e = 0; e < 3; ++e) at_leaf[e * kLeaves + leaf] = one ? v[e] : 0;
    }
    __syncthreads();
    auto same = [&](int a, int b) {
        return at_leaf[a] && at_leaf[a] == at_leaf[b] && at_leaf[kLeaves + a] == at_leaf[kLeaves + b] &&
               at_leaf[2 * kLeaves + a] == at_leaf[2 * kLeaves + b];
    };
    const bool left_out = leaf >= 2 && same(leaf, leaf - 1) && same(leaf, leaf - 2);
    if (__syncthreads_or(left_out)) {
        __shared__ uint16_t run[kLeaves / 3], beyond[kChunkThreads / kWave][kCoincident];
        __shared__ uint32_t few[kChunkThreads / kWave][kWave];
        __shared__ int runs;
        auto wave_fence = [] {   // between a wavefront's own LDS stores and loads
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
        };
        if (tid == 0) runs = 0;
        __syncthreads();
        if ((tid & 3) == 2 && left_out && !(leaf >= 3 && same(leaf, leaf - 3))) run[atomicAdd(&runs, 1)] = (uint16_t)(leaf - 2);
        __syncthreads();
        for (int r = wave; r < runs; r += kChunkThreads / kWave) {   // a wavefront per run
            const int h = run[r];
            int end = kLeaves;
            for (int e0 = h + 3; e0 < end; e0 += kWave) {
                const int e = e0 + lane;
                const uint64_t other = __ballot(e < kLeaves && !same(e, h));
                if (other) end = e0 + __builtin_ctzll(other);
            }
            uint16_t* slot = order + kFan * h;
            const int n = kFan * (end - h);
            auto index = [&](int i) -> uint32_t { return i < n && slot[i] < ch.n ? orig[slot[i]] : kNoPoint; };
            // the kCoincident-th lowest index, `low`: of a wavefront's values by
            // bisection; that of the lanes' least indices bounds it, and the few
            // up to the bound decide
            auto nth = [&](uint32_t x, uint32_t hi) {
                uint32_t lo = 0;
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) / 2;
                    if (__builtin_popcountll(__ballot(x <= mid)) >= kCoincident) hi = mid;
                    else lo = mid + 1;
                }
                return hi;
            };
            uint32_t least = kNoPoint;
#pragma unroll 4
            for (int i = lane; i < n; i += kWave) least = min(least, index(i));
            uint32_t low = nth(least, (uint32_t)d.n);
            int c = 0;
            for (int i = lane; i - lane < n; i += kWave) {
                const uint32_t id = index(i);
                const uint64_t m = __ballot(id <= low);
                const int at = c + __builtin_popcountll(m & ((1ull << lane) - 1ull));
                if (id <= low && at < kWave) few[wave][at] = id;
                c += __builtin_popcountll(m);
            }
            wave_fence();
            if (c <= kWave) {
                low = nth(lane < c ? few[wave][lane] : kNoPoint, low);
            } else {   // lanes that hold many low indices: over all points
                uint32_t lo = 0;
                while (lo < low) {
                    const uint32_t mid = (lo + low) / 2;
                    c = 0;
                    for (int i = lane; i - lane < n; i += kWave) c += __builtin_popcountll(__ballot(index(i) <= mid));
                    if (c >= kCoincident) low = mid;
                    else lo = mid + 1;
                }
            }
            // the points up to it that lie beyond the first two leaves change
            // places with the others in these
            int b = 0;
            for (int i = kCoincident + lane; i - lane < n; i += kWave) {
                const bool in = index(i) <= low;
                const uint64_t m = __ballot(in);
                const int at = b + __builtin_popcountll(m & ((1ull << lane) - 1ull));
                if (in && at < kCoincident) beyond[wave][at] = (uint16_t)i;
                b += __builtin_popcountll(m);
            }
            wave_fence();
            const bool high = lane < kCoincident && index(lane) > low;
            const int at = __builtin_popcountll(__ballot(high) & ((1ull << lane) - 1ull));
            if (high && at < b) {
                const int i = beyond[wave][at];
                const uint16_t p = slot[lane];
                slot[lane] = slot[i];
                slot[i] = p;
            }
        }
        __syncthreads();
        leaf_box();
        if (left_out)
#pragma unroll
            for (int e = 0; e < 6; ++e) v[e] = 0;
    }
    // points; padding copies the first point of its leaf
    float* pts = (float*)(a.nodes + d.level_off[0] + (int64_t)ch.number * (kChunk / 4 * kPointQuad));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int at = u * kChunkThreads + tid;
        if (at < ch.slots) {
            uint32_t i = order[at];
            const bool real = (int)i < ch.n;
            if (!real) i = order[at & ~(kFan - 1)];
            if ((int)i >= ch.n) i = 0;
            float* o = pts + 4 * kPointQuad * (at / 4) + at % 4;
            o[0] = xyz[0][i];
            o[4] = xyz[1][i];
            o[8] = xyz[2][i];
            o[12] = __uint_as_float(real ? orig[i] : kNoPoint);
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
            hi[e] = any ? from_order_bits(v[e]) : inf;
        }
        put_box(a.nodes + d.level_off[level], box, lo, hi);
    };
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
            float lo[3] = {inf, inf, inf}, hi[3] = {inf, inf, inf};
            if (e < real) {   // the children are one block, the first of them real
                const float4* c = a.nodes + d.level_off[l - 1] + e * (kFan / 4 * kBoxQuad);
                auto upper = [&](float x, float y) { return x == inf ? -inf : y; };   // of an empty box: none
#pragma unroll
                for (int f = 0; f < 3; ++f) hi[f] = -inf;
                for (int u = 0; u < kFan / 4; ++u)
#pragma unroll
                    for (int f = 0; f < 3; ++f) {
                        const float4 x = c[u * kBoxQuad + f], y = c[u * kBoxQuad + 3 + f];
                        lo[f] = fminf(lo[f], fminf(fminf(x.x, x.y), fminf(x.z, x.w)));
                        hi[f] = fmaxf(hi[f], fmaxf(fmaxf(upper(x.x, y.x), upper(x.y, y.y)),
                                                   fmaxf(upper(x.z, y.z), upper(x.w, y.w))));
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
    // side_blocks > 0: each pair's first side_blocks workgroups work on its
    // bandwidths instead, beside the search: BW, two of them select the
    // medians; else they form the distances between the particles, from which
    // the next launch selects
    int32_t side_blocks, side_form;
    SvgdArgs side;
};

// Key of no match yet: distance infinity, reference 0 (what the brute-force
// search returns where no distance is finite).
constexpr uint64_t kIndexNoMatch = 0x7f80000000000000ull;

// Threads of a search workgroup: 16 queries. Larger ones hold their slots
// until the last of more queries ends (4 lanes, street scan: 64 threads 62.6
// us a launch, 128 65.0, 256 66.6).
// With the bandwidths beside the search, the selection's 1,024.
constexpr int search_threads(int lanes, bool bw = false) { return bw ? kSvgdThreads : 16 * lanes; }

// Dynamic LDS: a thread's remaining distances, per box level.
template <int L, bool BW = false>
inline size_t index_nn_lds_bytes(int levels)
{
    return (size_t)(levels - 1) * search_threads(L, BW) * (kFan / L) * 4;
}

// Workgroups of `threads` threads for the distances between K particles: a
// wavefront per particle and kernel.
inline int pair_distance_blocks(int K, int threads) { return (2 * K * kWave + threads - 1) / threads; }

// grid (side_blocks + ceil(K m L / T), pairs), T = search_threads(L, BW)
// threads; dynamic LDS index_nn_lds_bytes<L, BW>(most levels of the clouds)
// and what the bandwidths need. A query to L lanes; the
// queries are ordered by minibatch point, then particle, so that those of a
// wavefront look for (nearly) the same place and read the same blocks.
//
// Many queries are bound by the vector units and the load path at once: 64
// uneven pairs of 30,000 queries have the returns of their loads busy for 92 %
// of the launch, and a vector instruction every 3.6 cycles of a SIMD, with 46 %
// of the lanes active (102 to 111 vector instructions a query; a wavefront's 70
// to 76 loads hit the L1 nine times in ten). 300,000 queries keep both at two
// thirds to three quarters; few queries wait for the dependent steps, 5 (2,000
// references) to 8 (100,000) a query. The index stays in the caches: 42 MB a
// launch come from HBM for the street, 11 for the 1,000 runs. us a launch, the
// first five / the middle / the last of a solve with 4 lanes, and with 16 at
// its start (what the search replaced: the mode's brute-force one): 300,000
// queries of 100,000 street references 160 / 66 / 58, 212 (1,055); 64 uneven
// pairs of 30,000 queries 335 / 305 / 290, 608 (1,114); 1,000 runs of 300
// queries of 20,000 67 / 65 / 65, 98 (231). From the 75th iteration on, 4 and
// 16 lanes: 30,000 queries of 20,000 tabletop references 17.0 and 14.4 (34),
// 100,000 22.9 and 31.8; 30,000 of 100,000 street references 22.6 and 20.1,
// 100,000 29.7 and 42.6. Left out after measuring: upper levels staged in LDS
// (street +0 to 7 %, tabletop +4 %, 64 pairs -1 %: their loads are few), several
// queries in turn per group (street 72 -> 82), fan-out 64 on 16 lanes (tabletop
// 16.6, street 112) and 4 on one lane (41, 94).
template <int L, bool BW>
__global__ __launch_bounds__(search_threads(L, BW), BW ? 8 : 1) void index_nn_kernel(IndexSearchArgs a)
{
    constexpr int T = search_threads(L, BW);
    constexpr int E = kFan / L;                   // entries of a block per lane
    constexpr uint32_t kInf = 0x7f800000u, kEntry = kFan - 1;
    extern __shared__ float4 lds4[];
    Row<E>* above = (Row<E>*)lds4;                // [box level - 1][thread]
    __shared__ int32_t level_off[kIndexLevels];
    const int tid = threadIdx.x;
    const int64_t p = blockIdx.y;
    const int wg = (int)blockIdx.x - a.side_blocks;
    if (wg < 0) {   // whole workgroup
        if constexpr (BW) {
            bandwidth_role<T>(a.side, 2 * p + blockIdx.x, a.side_form, false, (double*)lds4);
        } else {
            const int row = uniform(((int)blockIdx.x * T + tid) / kWave);
            if (row < 2 * a.K) pair_distances_row(a.side.theta, a.side.dscr, a.K, p, row / a.K, row % a.K);
        }
        return;
    }
    const IndexDesc& d = a.desc[a.cloud ? a.cloud[p] : 0];
    const int top = d.levels - 1;
    const float* __restrict__ nodes = (const float*)(a.nodes + d.level_off[0]);
    const uint32_t fl = tid & (L - 1);
    if (tid < kIndexLevels) level_off[tid] = 4 * (int32_t)(d.level_off[tid] - d.level_off[0]);
    __syncthreads();
    const uint32_t nq = (uint32_t)a.K * (uint32_t)a.m;   // below 2^30
    const uint32_t w = (uint32_t)wg * (T / L) + tid / L;
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
        const Row<E> lx = src[0], ly = src[4 / E], lz = src[8 / E];
        Row<E> hx = lx, hy = ly, hz = lz;   // of a point; a box's upper corner follows its lower one
        const Row<E> fourth = src[12 / E];
        if (box) {
            hx = fourth;
            hy = src[16 / E];
            hz = src[20 / E];
        }
        uint32_t cur[E];
#pragma unroll
        for (int u = 0; u < E; ++u) {
#pragma clang fp contract(off)
            const float dx = q.x - __builtin_amdgcn_fmed3f(q.x, lx.v[u], hx.v[u]);
            const float dy = q.y - __builtin_amdgcn_fmed3f(q.y, ly.v[u], hy.v[u]);
            const float dz = q.z - __builtin_amdgcn_fmed3f(q.z, lz.v[u], hz.v[u]);
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
            const Row<E> id = fourth;
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

// --------------------------------------------------- nearest neighbours, k
struct IndexKnnArgs {
    const IndexDesc* desc;   // of the one cloud
    const float4* nodes;
    uint64_t* lists;         // k keys (distance bits, index) per reference, ascending, kNoKey past the cloud
    int32_t k, pad_;
};

// The k nearest references of every reference (itself included), k <= 16 R:
// the search above with 16 lanes, its bound the list's k-th distance. The
// lanes hold the list in ascending order, entry 16 r + lane in list[r]; a
// leaf's points that come before its k-th are inserted one by one. The queries
// are taken in the order of the index, so that the four of a wavefront share
// most of their blocks. The lists equal the brute-force scan's: both keep the
// k smallest (distance, index) keys. grid ceil(slots / 16), 256 threads;
// dynamic LDS index_nn_lds_bytes<16>(levels).
// Bound like the search. Normals of a 20,000-point tabletop, k = 10, with the
// covariances: 31 us (22 here) against 328 by brute force.
template <int R>
__global__ __launch_bounds__(search_threads(16)) void index_knn_kernel(IndexKnnArgs a)
{
    constexpr int T = search_threads(16);
    constexpr uint32_t kInf = 0x7f800000u, kEntry = kFan - 1;
    constexpr uint64_t kNone = ~0ull;
    extern __shared__ uint32_t left[];            // [box level - 1][thread]
    __shared__ int32_t level_off[kIndexLevels];
    const int tid = threadIdx.x;
    const IndexDesc& d = *a.desc;
    const int top = d.levels - 1;
    const float* __restrict__ nodes = (const float*)(a.nodes + d.level_off[0]);
    if (tid < kIndexLevels) level_off[tid] = 4 * (int32_t)(d.level_off[tid] - d.level_off[0]);
    __syncthreads();
    const uint32_t fl = tid & 15, quad0 = fl / 4, place = fl % 4;
    const uint32_t slot = blockIdx.x * (T / 16) + tid / 16;
    if (slot >= (uint32_t)(d.level_off[1] - d.level_off[0])) return;   // whole groups; no barrier below
    const float* self = nodes + slot / 4 * (4 * kPointQuad) + slot % 4;
    const float qx = self[0], qy = self[4], qz = self[8];
    const uint32_t id = __float_as_uint(self[12]);
    if (id == kNoPoint) return;
    uint64_t list[R];
#pragma unroll
    for (int r = 0; r < R; ++r) list[r] = kNone;
    uint32_t bound = kInf;
    int level = top;
    uint32_t block = 0;
    for (;;) {
        const bool box = level > 0;
        const uint32_t quad = block * (kFan / 4) + quad0;
        const float* src = nodes + ((uint32_t)level_off[level] + 16 * quad + (box ? 8 * quad : 0) + place);
        const float* up = src + (box ? 12 : 0);
        uint32_t cur;
        {
#pragma clang fp contract(off)
            const float dx = qx - __builtin_amdgcn_fmed3f(qx, src[0], up[0]);
            const float dy = qy - __builtin_amdgcn_fmed3f(qy, src[4], up[4]);
            const float dz = qz - __builtin_amdgcn_fmed3f(qz, src[8], up[8]);
            cur = __float_as_uint(__builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx)));
        }
        if (box) {
            cur = (cur & ~kEntry) | fl;
        } else {
            const uint32_t j = __float_as_uint(src[12]);
            uint64_t cand = j == kNoPoint ? kNone : ((uint64_t)cur << 32) | j;
            uint64_t worst;
            for (;;) {
                worst = __shfl(R == 1 || a.k <= 16 ? list[0] : list[R - 1], (a.k - 1) & 15, 16);
                const uint32_t open = (uint32_t)(__ballot(cand < worst) >> (tid & 48)) & 0xffffu;
                if (!open) break;
                const int c = __builtin_ctz(open);
                const uint64_t x = __shfl(cand, c, 16);
                if ((int)fl == c) cand = kNone;
                // entries from x on move up one place (nothing lies before entry 0)
                uint64_t before[R];
                before[0] = dpp64<kDppShr1>(list[0]);
                if constexpr (R == 2) {
                    // both exchanges with all lanes: a lane that sits one out gives nothing
                    const uint64_t last = dpp64<kDppRor1>(list[0]), shifted = dpp64<kDppShr1>(list[1]);
                    before[1] = fl == 0 ? last : shifted;
                }
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (x < list[r]) list[r] = x < before[r] ? before[r] : x;
            }
            bound = min(kInf, (uint32_t)(worst >> 32));
            level = 1;
            block /= kFan;
            cur = left[tid];
        }
        uint32_t best;
        bool open;
        for (;;) {
            best = lanes_min<16>(cur);
            open = (best & ~kEntry) <= bound && best < kInf;
            if (open || level == top) break;
            cur = left[level * T + tid];
            ++level;
            block /= kFan;
        }
        if (!open) break;
        --level;
        left[level * T + tid] = cur == best ? kInf : cur;
        block = block * kFan + (best & kEntry);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (16 * r + (int)fl < a.k) a.lists[(int64_t)id * a.k + 16 * r + fl] = list[r];
}

}  // namespace sicp
