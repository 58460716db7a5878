// build.hip -- GPU linear BVH over primitive boxes (gfx950): triangle boxes
// for ray casting, or ready-made Gaussian boxes.
//
// FGGS-LiDAR Sec. IV-A "LBVH construction" (reused for triangles in
// Sec. IV-C): every primitive centre is quantised inside the scene box,
//   u_i = floor(2^b (c_i - o) / L),  m_i = Morton(u_i),
// the primitives are radix-sorted by m_i, the hierarchy follows from the
// longest common prefix of the sorted codes (Karras 2012: ties between equal
// codes are broken by the index, so every internal node splits on a distinct
// bit of the 3b + 32 bit augmented key), and node boxes are reduced bottom-up.
//
// Stages:
//   tri_bounds   triangle boxes + per-block partial scene boxes (or: partial
//                unions of ready-made primitive boxes)
//   morton       scene box from the partials, centre of each primitive box ->
//                3b-bit code, digit counts of the first sort pass
//   radix sort   per pass: per-tile digit counts / (large inputs: per-digit
//                scan of the tiles' counts) / stable scatter, ranked in LDS
//                with wave64 ballots
//   tree_chunk   one workgroup per 512 consecutive leaves: triangle records in
//                leaf order (not for ready-made boxes), a heap of box unions
//                over the leaves in LDS, and every internal node whose leaf
//                range lies in the chunk: children, parent, child boxes (range
//                unions from the heap), depth within the chunk
//   tree_span    the few nodes whose range crosses chunks, from the chunks'
//                heaps and a pyramid over the chunk boxes; then node depths
//   collapse     optional: 4-wide nodes with 8-bit child boxes in each node's
//                frame (prefix count of even-depth nodes, then one thread per
//                4-wide node)
//
// The tree's boxes are unions over contiguous leaf ranges, so every node
// asks for its children's ranges directly: no node waits for another one,
// and no arrival counters are needed.
#include "mesh_internal.h"

#include <math.h>

#include <type_traits>

namespace {

constexpr int kBlock = 256;

// Radix sort shapes.  Small inputs (at most kSmallTiles tiles) are bound by
// the number of dependent launches, so they take wide digits (30-bit codes in
// three passes) and every scatter block adds up the tiles' counts itself
// instead of a scan launch per pass.  Large inputs are bound by the scatter's
// scattered writes: 8-bit digits over larger tiles keep a digit's run of a
// tile near a 64-byte line.
constexpr int kSmallBlock = 256, kSmallItems = 8, kSmallBits = 10;
constexpr int kSmallTile = kSmallBlock * kSmallItems;
constexpr int kSmallTiles = 64;
constexpr int kLargeBlock = 512, kLargeItems = 8, kLargeBits = 8;
constexpr int kLargeTile = kLargeBlock * kLargeItems;

__device__ __forceinline__ float wave_min(float v)
{
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_max(float v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

constexpr int kBoundBlocks = 1024;   // blocks of the box reductions, at most

// Block-wide min/max of acc[0..2] / acc[3..5]; threads 0..5 write out[6].
template <int B>
__device__ __forceinline__ void block_box(float acc[6], float *out)
{
    __shared__ float red[B / 64][6];
    for (int a = 0; a < 3; ++a) {
        acc[a] = wave_min(acc[a]);
        acc[3 + a] = wave_max(acc[3 + a]);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        for (int a = 0; a < 6; ++a) red[w][a] = acc[a];
    __syncthreads();
    if (threadIdx.x < 6) {
        const int a = threadIdx.x;
        float v = red[0][a];
        for (int ww = 1; ww < B / 64; ++ww) v = a < 3 ? fminf(v, red[ww][a]) : fmaxf(v, red[ww][a]);
        out[a] = v;
    }
}

// Triangle boxes (AoS lo.xyz hi.xyz) and one partial scene box per block
// (grid-stride loop; the partials are folded by k_morton_hist, so no
// atomics: min/max are exact in any order).
__global__ __launch_bounds__(kBlock) void k_tri_bounds(const float *__restrict__ verts,
                                                       const int32_t *__restrict__ tris,
                                                       int64_t nt, float *__restrict__ bounds,
                                                       float *__restrict__ partial)
{
    float acc[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nt;
         i += (int64_t)gridDim.x * blockDim.x) {
        float lo[3] = {INFINITY, INFINITY, INFINITY};
        float hi[3] = {-INFINITY, -INFINITY, -INFINITY};
        for (int k = 0; k < 3; ++k) {
            const float *v = verts + 3 * (int64_t)tris[3 * i + k];
            for (int a = 0; a < 3; ++a) {
                lo[a] = fminf(lo[a], v[a]);
                hi[a] = fmaxf(hi[a], v[a]);
            }
        }
        float *b = bounds + 6 * i;
        b[0] = lo[0]; b[1] = lo[1]; b[2] = lo[2];
        b[3] = hi[0]; b[4] = hi[1]; b[5] = hi[2];
        for (int a = 0; a < 3; ++a) {
            acc[a] = fminf(acc[a], lo[a]);
            acc[3 + a] = fmaxf(acc[3 + a], hi[a]);
        }
    }
    block_box<kBlock>(acc, partial + 6 * blockIdx.x);
}

// Boxes of points, and partial unions as above.
__global__ __launch_bounds__(kBlock) void k_point_bounds(const float *__restrict__ p, int64_t n,
                                                         float *__restrict__ bounds,
                                                         float *__restrict__ partial)
{
    float acc[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        for (int a = 0; a < 3; ++a) {
            const float v = p[3 * i + a];
            bounds[6 * i + a] = v;
            bounds[6 * i + 3 + a] = v;
            acc[a] = fminf(acc[a], v);
            acc[3 + a] = fmaxf(acc[3 + a], v);
        }
    }
    block_box<kBlock>(acc, partial + 6 * blockIdx.x);
}

// Partial unions of ready-made primitive boxes.
__global__ __launch_bounds__(kBlock) void k_box_union(const float *__restrict__ bounds, int64_t n,
                                                      float *__restrict__ partial)
{
    float acc[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float *b = bounds + 6 * i;
        for (int a = 0; a < 3; ++a) {
            acc[a] = fminf(acc[a], b[a]);
            acc[3 + a] = fmaxf(acc[3 + a], b[3 + a]);
        }
    }
    block_box<kBlock>(acc, partial + 6 * blockIdx.x);
}

__device__ __forceinline__ uint32_t expand_bits(uint32_t v)
{
    // spread the low 10 bits of v so that bit k moves to bit 3k
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// ---- Morton codes and radix sort --------------------------------------------
// Digit counts are laid out [tile][digit] for the small shape (a scatter
// block reads whole rows) and [digit][tile] for the large one (the scan
// kernel reads whole rows).
template <int RB, bool SMALL>
__device__ __forceinline__ int64_t hist_at(int digit, int tile, int ntiles)
{
    return SMALL ? ((int64_t)tile << RB) + digit : (int64_t)digit * ntiles + tile;
}

// Scene box from the per-block partials, then the Morton code of each
// primitive-box centre (x takes the most significant position of every 3-bit
// group) and the tile's digit counts for the first sort pass.  Every block
// folds the partials itself: at most four loads a thread, against a launch.
template <int B, int IT, int RB, bool SMALL>
__global__ __launch_bounds__(B) void k_morton_hist(const float *__restrict__ bounds,
                                                   const float *__restrict__ partial, int nparts,
                                                   float *__restrict__ scene_box, int64_t n,
                                                   int bits, uint32_t *__restrict__ morton,
                                                   uint32_t *__restrict__ hist, int ntiles,
                                                   uint32_t *__restrict__ span_count)
{
    __shared__ float box[6];
    __shared__ uint32_t h[1 << RB];
    float acc[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int p = threadIdx.x; p < nparts; p += B)
        for (int a = 0; a < 3; ++a) {
            acc[a] = fminf(acc[a], partial[6 * p + a]);
            acc[3 + a] = fmaxf(acc[3 + a], partial[6 * p + 3 + a]);
        }
    block_box<B>(acc, box);
    for (int d = threadIdx.x; d < (1 << RB); d += B) h[d] = 0;
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x < 6) scene_box[threadIdx.x] = box[threadIdx.x];
    if (blockIdx.x == 0 && threadIdx.x == 0) *span_count = 0;   // for k_tree_chunk
    const float cells = (float)(1u << bits);
    float o[3], scale[3];
    for (int a = 0; a < 3; ++a) {
        o[a] = box[a];
        const float L = box[3 + a] - o[a];
        scale[a] = L > 0.0f ? cells / L : 0.0f;
    }
    const int64_t base = (int64_t)blockIdx.x * (B * IT);
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int64_t i = base + r * B + threadIdx.x;
        if (i < n) {
            const float2 *b = reinterpret_cast<const float2 *>(bounds + 6 * i);
            const float2 b0 = b[0], b1 = b[1], b2 = b[2];
            const float lo[3] = {b0.x, b0.y, b1.x}, hi[3] = {b1.y, b2.x, b2.y};
            uint32_t u[3];
            for (int a = 0; a < 3; ++a) {
                const float c = (lo[a] + hi[a]) * 0.5f;
                float q = floorf((c - o[a]) * scale[a]);
                q = fminf(fmaxf(q, 0.0f), cells - 1.0f);
                u[a] = (uint32_t)q;
            }
            const uint32_t m = (expand_bits(u[0]) << 2) | (expand_bits(u[1]) << 1) | expand_bits(u[2]);
            morton[i] = m;
            atomicAdd(&h[m & ((1u << RB) - 1u)], 1u);
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < (1 << RB); d += B)
        hist[hist_at<RB, SMALL>(d, blockIdx.x, ntiles)] = h[d];
}

template <int B, int IT, int RB, bool SMALL>
__global__ __launch_bounds__(B) void k_hist(const uint32_t *__restrict__ keys, int64_t n, int shift,
                                            uint32_t *__restrict__ hist, int ntiles)
{
    __shared__ uint32_t h[1 << RB];
    for (int d = threadIdx.x; d < (1 << RB); d += B) h[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (B * IT);
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int64_t i = base + r * B + threadIdx.x;
        if (i < n) atomicAdd(&h[(keys[i] >> shift) & ((1u << RB) - 1u)], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < (1 << RB); d += B)
        hist[hist_at<RB, SMALL>(d, blockIdx.x, ntiles)] = h[d];
}

// block-wide exclusive scan of one value per thread (B threads); returns
// the exclusive prefix, *total receives the block sum
template <int B>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *total)
{
    __shared__ uint32_t wsum[B / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int ww = 0; ww < B / 64; ++ww) {
        if (ww < w) off += wsum[ww];
        tot += wsum[ww];
    }
    __syncthreads();
    *total = tot;
    return off + x - v;
}

// one block per digit: exclusive scan of that digit's per-tile counts
// (in place) and the digit's total
__global__ __launch_bounds__(kBlock) void k_scan_digits(uint32_t *__restrict__ hist, int nblocks,
                                                        uint32_t *__restrict__ digit_tot)
{
    uint32_t *h = hist + (int64_t)blockIdx.x * nblocks;
    uint32_t carry = 0;
    for (int base = 0; base < nblocks; base += kBlock) {
        const int i = base + threadIdx.x;
        const uint32_t v = i < nblocks ? h[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan<kBlock>(v, &tot);
        if (i < nblocks) h[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) digit_tot[blockIdx.x] = carry;
}

// Stable scatter of one tile.  Each wave owns IT x 64 consecutive keys and
// ranks them against its own digit counters in LDS (the keys of one digit in
// a group of 64 find each other by RB ballots; the first of them advances
// the counter), so the ranking needs no workgroup barrier; one scan over the
// waves and digits then gives every key its slot in the tile's digit order.
// Keys and values are laid out in that order in LDS first: neighbouring
// threads then write neighbouring addresses of a digit's run.  FIRST: the
// value is the key's index.
template <int B, int IT, int RB, bool SMALL, bool FIRST>
__global__ __launch_bounds__(B) void k_scatter(const uint32_t *__restrict__ keys_in,
                                               const uint32_t *__restrict__ vals_in,
                                               uint32_t *__restrict__ keys_out,
                                               uint32_t *__restrict__ vals_out, int64_t n,
                                               int shift, const uint32_t *__restrict__ hist,
                                               const uint32_t *__restrict__ digit_tot, int ntiles)
{
    constexpr int R = 1 << RB, W = B / 64, T = B * IT;
    constexpr int PER = R / B > 0 ? R / B : 1;   // digits per thread
    static_assert(!SMALL || PER == 4, "the small shape reads four counts at a time");
    __shared__ uint32_t wcnt[W][R];
    __shared__ uint32_t tile_at[R];    // first slot of the digit in the tile's order
    __shared__ uint32_t out_at[R];     // where the digit's keys of this tile go
    __shared__ uint32_t skey[T], sval[T];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, tile = blockIdx.x;
    const int64_t base = (int64_t)tile * T;
    const int cnt = n - base < T ? (int)(n - base) : T;
    uint32_t key[IT], val[IT], rank[IT];
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int j = (w * IT + r) * 64 + lane;
        key[r] = j < cnt ? keys_in[base + j] : 0xffffffffu;
        val[r] = FIRST ? (uint32_t)(base + j) : (j < cnt ? vals_in[base + j] : 0u);
    }
    for (int j = tid; j < W * R; j += B) (&wcnt[0][0])[j] = 0;
    // this tile's output offsets: the digits below, then the tiles before
    uint32_t pre[PER], tot[PER], sum = 0;
    if constexpr (SMALL) {
        for (int d = 0; d < PER; ++d) pre[d] = tot[d] = 0;
        const uint4 *rows = reinterpret_cast<const uint4 *>(hist);
#pragma unroll 8
        for (int t = 0; t < ntiles; ++t) {
            const uint4 c = rows[(int64_t)t * (R / 4) + tid];
            const uint32_t m = t < tile ? ~0u : 0u;
            tot[0] += c.x; tot[1] += c.y; tot[2] += c.z; tot[3] += c.w;
            pre[0] += c.x & m; pre[1] += c.y & m; pre[2] += c.z & m; pre[3] += c.w & m;
        }
        for (int d = 0; d < PER; ++d) sum += tot[d];
    } else {
        static_assert(SMALL || PER == 1, "one digit per thread");
        pre[0] = tid < R ? hist[(int64_t)tid * ntiles + tile] : 0u;
        tot[0] = tid < R ? digit_tot[tid] : 0u;
        sum = tot[0];
    }
    uint32_t all;
    uint32_t ex = block_exclusive_scan<B>(sum, &all);   // its barriers also publish the zeroed counters
    for (int d = 0; d < PER; ++d) {
        if (tid * PER + d < R) out_at[tid * PER + d] = ex + pre[d];
        ex += tot[d];
    }
    // ranks within the wave
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const bool valid = (w * IT + r) * 64 + lane < cnt;
        const uint32_t d = (key[r] >> shift) & (R - 1);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < RB; ++bit) {
            const bool set = (d >> bit) & 1u;
            const uint64_t m = __ballot(set);
            peers &= set ? m : ~m;
        }
        const int first = valid ? __ffsll((unsigned long long)peers) - 1 : lane;
        uint32_t at = 0;
        if (valid && lane == first) at = atomicAdd(&wcnt[w][d], (uint32_t)__popcll(peers));
        rank[r] = __shfl(at, first, 64) + (uint32_t)__popcll(peers & lt);
    }
    __syncthreads();
    // exclusive over waves per digit, then over digits
    uint32_t own[PER];
    sum = 0;
    for (int d = 0; d < PER; ++d) {
        uint32_t run = 0;
        if (tid * PER + d < R)
            for (int ww = 0; ww < W; ++ww) {
                const uint32_t c = wcnt[ww][tid * PER + d];
                wcnt[ww][tid * PER + d] = run;
                run += c;
            }
        own[d] = run;
        sum += run;
    }
    ex = block_exclusive_scan<B>(sum, &all);
    for (int d = 0; d < PER; ++d) {
        if (tid * PER + d < R) tile_at[tid * PER + d] = ex;
        ex += own[d];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        if ((w * IT + r) * 64 + lane < cnt) {
            const uint32_t d = (key[r] >> shift) & (R - 1);
            const uint32_t slot = tile_at[d] + wcnt[w][d] + rank[r];
            skey[slot] = key[r];
            sval[slot] = val[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int j = r * B + tid;
        if (j < cnt) {
            const uint32_t k = skey[j], d = (k >> shift) & (R - 1);
            const uint32_t at = out_at[d] + ((uint32_t)j - tile_at[d]);
            keys_out[at] = k;
            vals_out[at] = sval[j];
        }
    }
}

// ---- hierarchy --------------------------------------------------------------
// Node i of the radix tree over the sorted codes (Karras 2012, Sec. 4) has
// one end of its leaf range at i; it splits at gamma into children gamma and
// gamma + 1.  The length of the longest common prefix with code i falls
// monotonically with the distance from i, so both the far end of the range
// and the split are binary searches.
//
// A chunk of kChunk leaves is one workgroup's: its codes and box heap sit in
// LDS and nodes are independent of each other, where a bottom-up pass waits a
// memory round trip for each of some 20 levels.  It is bound by those LDS
// chains (searches, heap queries), so a thread has one leaf and one node.
// 512 leaves keep the LDS use at 33 KB (4 workgroups a CU, all the threads it
// takes) and give a 54k-triangle tree 105 workgroups; about 1 node in 60
// crosses chunks and is left to k_tree_span.  Hierarchy, boxes, triangle
// records and depths of 1.03M triangles: 102 us (chunk 55, pyramid 8, span 18,
// depth 12, parity 8), where separate topology, bottom-up and depth walks
// took 249; of 54k triangles 35 us against 114.
constexpr int kChunk = 512;
constexpr int kTreeBlock = kChunk;
constexpr int kGroup = 8;                       // leaves under the lowest stored heap level
constexpr int kHeap = 2 * kChunk / kGroup;      // heap boxes stored per chunk (1..kHeap-1 used)
constexpr int kPyramid = 8;                     // fan-in of the pyramid over chunk boxes
constexpr int kTopChunks = 512;                 // up to here a node looks at chunk boxes one by one

constexpr uint8_t kCrosses = 0xff;              // sub_height of a node that crosses chunks

struct Box {
    float lo[3], hi[3];
};

__device__ __forceinline__ Box empty_box()
{
    return Box{{INFINITY, INFINITY, INFINITY}, {-INFINITY, -INFINITY, -INFINITY}};
}

__device__ __forceinline__ void grow(Box &b, const Box &o)
{
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = fminf(b.lo[a], o.lo[a]);
        b.hi[a] = fmaxf(b.hi[a], o.hi[a]);
    }
}

__device__ __forceinline__ Box load_box(const float *__restrict__ p, int64_t i)
{
    const float2 *q = reinterpret_cast<const float2 *>(p + 6 * i);
    const float2 a = q[0], b = q[1], c = q[2];
    return Box{{a.x, a.y, b.x}, {b.y, c.x, c.y}};
}

__device__ __forceinline__ void store_box(float *__restrict__ p, int64_t i, const Box &b)
{
    float2 *q = reinterpret_cast<float2 *>(p + 6 * i);
    q[0] = make_float2(b.lo[0], b.lo[1]);
    q[1] = make_float2(b.lo[2], b.hi[0]);
    q[2] = make_float2(b.hi[1], b.hi[2]);
}

__device__ __forceinline__ NodeRec node_record(const Box &l, const Box &r, int32_t left, int32_t right,
                                               uint32_t pack_l, uint32_t pack_r)
{
    NodeRec nd;
    nd.q0 = make_float4(l.lo[0], l.hi[0], r.lo[0], r.hi[0]);
    nd.q1 = make_float4(l.lo[1], l.hi[1], r.lo[1], r.hi[1]);
    nd.q2 = make_float4(l.lo[2], l.hi[2], r.lo[2], r.hi[2]);
    nd.q3 = make_int4(left, right, (int32_t)pack_l, (int32_t)pack_r);
    return nd;
}

// common prefix length of codes a (leaf i) and b (leaf j): equal codes are
// told apart by the leaf index
__device__ __forceinline__ int prefix(uint32_t a, uint32_t b, int32_t i, int32_t j)
{
    return a == b ? 32 + __clz(i ^ j) : __clz(a ^ b);
}

struct TreeArrays {
    const uint32_t *keys;     // sorted codes
    const uint32_t *sorted;   // primitive of each leaf
    int32_t n;
    const float *bounds;      // primitive boxes, input order
    int32_t *topo;
    NodeRec *nodes;
    float *heap;              // [chunks][kHeap] boxes
    float *pyramid;           // chunk boxes, then each level of kPyramid-fold unions
    uint8_t *rel;             // depth of a node below its chunk-subtree root
    int32_t *sroot;           // that root
    uint8_t *base;            // depth of a chunk-subtree root (indexed by it)
    uint8_t *sub_height;      // deepest node below a chunk-subtree root (indexed by it)
    int32_t *span;            // nodes whose range crosses chunks
    uint32_t *span_count;
    int32_t *depth_out;
};

// Leaves are triangles or points, whose records are written in leaf order,
// or ready-made boxes.
enum LeafKind { LEAF_TRI, LEAF_POINT, LEAF_BOX };

template <int LEAF>
__global__ __launch_bounds__(kTreeBlock) void k_tree_chunk(TreeArrays A, const float *__restrict__ verts,
                                                           const int32_t *__restrict__ tris,
                                                           TriRec *__restrict__ trirecs,
                                                           float4 *__restrict__ points)
{
    __shared__ float bx[6][2 * kChunk];
    __shared__ uint32_t sk[kChunk + 2];       // codes of leaves c0 - 1 .. c0 + kChunk
    __shared__ int32_t par[kChunk];
    __shared__ int32_t deep[kChunk];
    __shared__ int32_t slist[kChunk];
    __shared__ uint32_t pack[kChunk];
    __shared__ uint32_t scount, sbase;
    const int tid = threadIdx.x;
    const int32_t n = A.n, c0 = (int32_t)blockIdx.x * kChunk;
    const int cn = n - c0 < kChunk ? (int)(n - c0) : kChunk;
    if (tid == 0) {
        scount = 0;
        sk[0] = c0 > 0 ? A.keys[c0 - 1] : 0u;
        sk[1 + cn] = c0 + cn < n ? A.keys[c0 + cn] : 0u;
    }
    for (int j = tid; j < kChunk; j += kTreeBlock) {
        par[j] = -1;
        deep[j] = 0;
        Box b = empty_box();
        if (j < cn) {
            const int32_t k = c0 + j;
            sk[1 + j] = A.keys[k];
            const int64_t t = A.sorted[k];
            if (LEAF == LEAF_TRI) {
                const float *p[3];
                for (int v = 0; v < 3; ++v) p[v] = verts + 3 * (int64_t)tris[3 * t + v];
                float c[3][3];
                for (int v = 0; v < 3; ++v)
                    for (int a = 0; a < 3; ++a) c[v][a] = p[v][a];
                for (int v = 0; v < 3; ++v)
                    for (int a = 0; a < 3; ++a) {
                        b.lo[a] = fminf(b.lo[a], c[v][a]);
                        b.hi[a] = fmaxf(b.hi[a], c[v][a]);
                    }
                TriRec r;
                r.a = make_float4(c[0][0], c[0][1], c[0][2], c[1][0]);
                r.b = make_float4(c[1][1], c[1][2], c[2][0], c[2][1]);
                r.c = make_float4(c[2][2], __int_as_float((int32_t)t), 0.0f, 0.0f);
                trirecs[k] = r;
            } else if (LEAF == LEAF_POINT) {
                for (int a = 0; a < 3; ++a) b.lo[a] = b.hi[a] = verts[3 * t + a];
                points[k] = make_float4(b.lo[0], b.lo[1], b.lo[2], __int_as_float((int32_t)t));
            } else {
                b = load_box(A.bounds, t);
            }
        }
        for (int a = 0; a < 3; ++a) {
            bx[a][kChunk + j] = b.lo[a];
            bx[3 + a][kChunk + j] = b.hi[a];
        }
    }
    __syncthreads();
    for (int w = kChunk / 2; w >= 1; w >>= 1) {
        for (int t = w + tid; t < 2 * w; t += kTreeBlock)
            for (int a = 0; a < 3; ++a) {
                bx[a][t] = fminf(bx[a][2 * t], bx[a][2 * t + 1]);
                bx[3 + a][t] = fmaxf(bx[3 + a][2 * t], bx[3 + a][2 * t + 1]);
            }
        __syncthreads();
    }
    for (int e = tid; e < 6 * kHeap; e += kTreeBlock)
        if (e >= 6) A.heap[(int64_t)blockIdx.x * (6 * kHeap) + e] = bx[e % 6][e / 6];
    if (tid < 6) A.pyramid[6 * (int64_t)blockIdx.x + tid] = bx[tid][1];

    // union of the boxes of local leaves l..r
    auto query = [&](int l, int r) {
        Box b = empty_box();
        auto add = [&](int t) {
            for (int a = 0; a < 3; ++a) {
                b.lo[a] = fminf(b.lo[a], bx[a][t]);
                b.hi[a] = fmaxf(b.hi[a], bx[3 + a][t]);
            }
        };
        for (l += kChunk, r += kChunk + 1; l < r; l >>= 1, r >>= 1) {
            if (l & 1) add(l++);
            if (r & 1) add(--r);
        }
        return b;
    };
    const int j = tid;
    const int32_t i = c0 + j;
    const bool node = j < cn && i < n - 1;
    bool inside = false;              // this thread's node lies in the chunk
    int32_t left = 0, right = 0;
    Box lb, rb;
    if (node) {
        const uint32_t ki = sk[1 + j];
        // prefix with local leaf q in -1..cn (halo included), -1 outside the input
        auto pre = [&](int q) {
            const int32_t g = c0 + q;
            return g < 0 || g >= n ? -1 : prefix(ki, sk[1 + q], i, g);
        };
        const int pn = pre(j + 1), pp = pre(j - 1);
        const int d = pn >= pp ? 1 : -1;
        const int dmin = d > 0 ? pp : pn;
        inside = pre(d > 0 ? cn : -1) <= dmin;
        if (!inside) {
            slist[atomicAdd(&scount, 1u)] = i;
        } else {
            // largest l <= len with pre(j + l d) > thr
            auto farthest = [&](int len, int thr) {
                int step = 1;
                while (step <= len && pre(j + step * d) > thr) step <<= 1;
                int l = step >> 1;                    // pre(j + l d) > thr, or l = 0
                int hi = step - 1 < len ? step - 1 : len;
                while (l < hi) {
                    const int mid = (l + hi + 1) >> 1;
                    if (pre(j + mid * d) > thr) l = mid; else hi = mid - 1;
                }
                return l;
            };
            // far end of the range: the last leaf with a prefix above dmin
            const int l = farthest(d > 0 ? cn - 1 - j : j, dmin);
            const int e = j + l * d;
            const int s = farthest(l - 1, pre(e));
            const int gamma = j + s * d + (d < 0 ? -1 : 0);
            const int lo = j < e ? j : e, hi = j < e ? e : j;
            left = lo == gamma ? ~(c0 + gamma) : c0 + gamma;
            right = hi == gamma + 1 ? ~(c0 + gamma + 1) : c0 + gamma + 1;
            if (left >= 0) par[gamma] = i;
            if (right >= 0) par[gamma + 1] = i;
            pack[j] = pack_children(left, right);
            lb = query(lo, gamma);
            rb = query(gamma + 1, hi);
        }
    }
    __syncthreads();
    if (tid == 0) sbase = scount ? atomicAdd(A.span_count, scount) : 0u;
    if (node) {
        if (inside) {
            A.topo[3 * (int64_t)i + 0] = left;
            A.topo[3 * (int64_t)i + 1] = right;
            A.nodes[i] = node_record(lb, rb, left, right, left >= 0 ? pack[left - c0] : 0u,
                                     right >= 0 ? pack[right - c0] : 0u);
        }
        if (par[j] >= 0) A.topo[3 * (int64_t)i + 2] = par[j];
        int d = 0, r = j;
        for (int32_t p = par[r]; p >= 0; p = par[r]) {
            r = p - c0;
            ++d;
        }
        A.rel[i] = (uint8_t)d;
        A.sroot[i] = c0 + r;
        if (d) atomicMax(&deep[r], d);
    }
    __syncthreads();
    if (node && par[j] < 0) A.sub_height[i] = (uint8_t)deep[j];
    for (uint32_t q = tid; q < scount; q += kTreeBlock) A.span[sbase + q] = slist[q];
    if (blockIdx.x == 0 && tid == 0) {
        if (n > 1 && n <= kChunk) {   // the whole tree
            A.topo[2] = -1;
            A.base[0] = 0;
        }
        A.depth_out[0] = n > 1 && n <= kChunk ? deep[0] + 1 : 0;   // else raised by span_depth
    }
}

// Levels of the pyramid over the chunk boxes, each level's boxes behind the
// one below; one block.
__device__ __forceinline__ void build_pyramid(float *__restrict__ pyr, int m)
{
    int64_t at = 0;
    while (m > 1) {
        const int up = (m + kPyramid - 1) / kPyramid;
        for (int t = threadIdx.x; t < up; t += blockDim.x) {
            Box b = empty_box();
            const int e = m - t * kPyramid < kPyramid ? m - t * kPyramid : kPyramid;
            for (int k = 0; k < e; ++k) grow(b, load_box(pyr, at + t * kPyramid + k));
            store_box(pyr, at + m + t, b);
        }
        at += m;
        m = up;
        __syncthreads();
    }
}

// One node whose range crosses chunks, by a group of kSpanLanes lanes: every
// step of its searches and box unions is a memory round trip, so the lanes
// probe and load side by side (16-way searches: three steps in place of
// nine in a chunk, and each union's pieces at once).  One lane per node took
// 82 us on 1.03M triangles and 107 us on 54k; the 16 lanes take 18 and 11 us.
constexpr int kSpanLanes = 16;

__device__ void span_node(const TreeArrays &A, int m, int32_t i)
{
    const uint32_t *__restrict__ keys = A.keys;
    const int32_t n = A.n;
    const int lane = threadIdx.x & (kSpanLanes - 1);
    const int shift = threadIdx.x & 63 & ~(kSpanLanes - 1);
    const uint32_t ki = keys[i];
    auto pre = [&](int32_t g) { return g < 0 || g >= n ? -1 : prefix(ki, keys[g], i, g); };
    const int pn = pre(i + 1), pp = pre(i - 1);
    const int d = pn >= pp ? 1 : -1;
    const int dmin = d > 0 ? pp : pn;
    // the largest x <= hi with pass(x), for a predicate that holds up to some
    // x >= 0 and not beyond
    auto last = [&](int32_t hi, auto pass) {
        int32_t lo = 0;
        while (lo < hi) {
            const int32_t step = (hi - lo + kSpanLanes - 1) / kSpanLanes;
            const int32_t x = lo + (lane + 1) * step;
            const uint64_t ok = __ballot(x <= hi && pass(x));
            lo += step * __popc((uint32_t)(ok >> shift) & ((1u << kSpanLanes) - 1u));
            hi = lo + step - 1 < hi ? lo + step - 1 : hi;
        }
        return lo;
    };
    // the leaf farthest from i in direction d with a prefix above thr (i
    // itself if there is none): over the chunks' near ends, then in a chunk
    const int32_t ci = i / kChunk;
    auto farthest = [&](int thr) {
        const int32_t near = d > 0 ? (ci + 1) * kChunk : ci * kChunk - 1;   // of the next chunk
        const int32_t x = last(d > 0 ? m - 1 - ci : ci,
                               [&](int32_t k) { return pre(near + d * (k - 1) * kChunk) > thr; });
        const int32_t from = x > 0 ? near + d * (x - 1) * kChunk : i;
        const int32_t c = from / kChunk;
        const int32_t end = d > 0 ? (c * kChunk + kChunk < n ? c * kChunk + kChunk : n) - 1 : c * kChunk;
        return from + d * last(d * (end - from),
                               [&](int32_t k) { return pre(from + d * k) > thr; });
    };
    const int32_t j = farthest(dmin);
    const int32_t s = farthest(pre(j));
    const int32_t gamma = s + (d < 0 ? -1 : 0);
    const int32_t lo = i < j ? i : j, hi = i < j ? j : i;
    const int32_t left = lo == gamma ? ~gamma : gamma;
    const int32_t right = hi == gamma + 1 ? ~(gamma + 1) : gamma + 1;
    Box b[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int32_t c = k == 0 ? left : right;
        const int32_t l = k == 0 ? lo : gamma + 1, r = k == 0 ? gamma : hi;
        const int32_t cl = l / kChunk, cr = r / kChunk;
        Box u = empty_box();
        if (c < 0) {
            u = load_box(A.bounds, A.sorted[l]);
        } else if (cl == cr) {
            // k_tree_chunk's node
            const NodeRec nd = A.nodes[c];
            u = Box{{fminf(nd.q0.x, nd.q0.z), fminf(nd.q1.x, nd.q1.z), fminf(nd.q2.x, nd.q2.z)},
                    {fmaxf(nd.q0.y, nd.q0.w), fmaxf(nd.q1.y, nd.q1.w), fmaxf(nd.q2.y, nd.q2.w)}};
        } else {
            // lanes 0..7: the end of the first chunk; 8..15: the start of the
            // last one.  Each a few leaves up to a whole group, then one heap
            // box per set bit of the number of groups.
            const int q = lane & 7;
            const bool first = lane < 8;
            const int32_t le = (l + kGroup - 1) / kGroup * kGroup, rb = (r + 1) / kGroup * kGroup;
            const int32_t leaf = first ? l + q : rb + q;
            if (first ? leaf < le : leaf <= r) u = load_box(A.bounds, A.sorted[leaf]);
            const int groups = first ? ((cl + 1) * kChunk - le) / kGroup : (rb - cr * kChunk) / kGroup;
            if (q < 7 && (groups >> q) & 1) {
                // a run of `groups` groups at either end of a chunk of 64:
                // its piece of 2^q groups
                const int before = groups >> (q + 1) << 1;   // in units of 2^q
                const int at = first ? ((kHeap / 2) >> q) - before - 1 : before;
                grow(u, load_box(A.heap + (int64_t)(first ? cl : cr) * (6 * kHeap),
                                 ((kHeap / 2) >> q) + at));
            }
            // whole chunks between them
            int x = cl + 1, y = cr, mm = m;
            if (m <= kTopChunks) {
#pragma unroll 4
                for (int t = x + lane; t < y; t += kSpanLanes) grow(u, load_box(A.pyramid, t));
            } else {
                int64_t at = 0;
                while (x < y) {
                    int xe = (x + kPyramid - 1) / kPyramid * kPyramid;
                    xe = xe < y ? xe : y;
                    int yb = y / kPyramid * kPyramid;
                    yb = yb > xe ? yb : xe;
                    const int t = first ? x + q : yb + q;
                    if (t < (first ? xe : y)) grow(u, load_box(A.pyramid, at + t));
                    at += mm;
                    mm = (mm + kPyramid - 1) / kPyramid;
                    x = xe / kPyramid;
                    y = yb / kPyramid;
                    if (xe >= yb) break;
                }
            }
            for (int a = 0; a < 3; ++a)
                for (int o = kSpanLanes / 2; o > 0; o >>= 1) {
                    u.lo[a] = fminf(u.lo[a], __shfl_xor(u.lo[a], o, kSpanLanes));
                    u.hi[a] = fmaxf(u.hi[a], __shfl_xor(u.hi[a], o, kSpanLanes));
                }
        }
        b[k] = u;
    }
    if (lane == 0) {
        A.topo[3 * (int64_t)i + 0] = left;
        A.topo[3 * (int64_t)i + 1] = right;
        if (left >= 0) A.topo[3 * (int64_t)left + 2] = i;
        if (right >= 0) A.topo[3 * (int64_t)right + 2] = i;
        if (i == 0) A.topo[2] = -1;
        A.nodes[i] = node_record(b[0], b[1], left, right, 0u, 0u);   // packs: span_depth
        A.rel[i] = 0;
        A.sroot[i] = i;
        A.sub_height[i] = kCrosses;
    }
}

// Depth of a crossing node by its ancestors (all of them cross chunks), and
// of the chunk subtrees and leaves below it; its record's names of its
// children's children.
__device__ void span_depth(const TreeArrays &A, int32_t i)
{
    int d = 0;
    for (int32_t p = A.topo[3 * (int64_t)i + 2]; p >= 0 && d <= 64; p = A.topo[3 * (int64_t)p + 2]) ++d;
    A.base[i] = (uint8_t)d;
    int deepest = 0;
    uint32_t pack[2];
    for (int k = 0; k < 2; ++k) {
        const int32_t c = A.topo[3 * (int64_t)i + k];
        pack[k] = c < 0 ? 0u : pack_children(A.topo[3 * (int64_t)c], A.topo[3 * (int64_t)c + 1]);
        if (c < 0) {
            deepest = deepest > d + 1 ? deepest : d + 1;
        } else if (A.sub_height[c] != kCrosses) {
            A.base[c] = (uint8_t)(d + 1);
            const int t = d + 1 + A.sub_height[c] + 1;
            deepest = deepest > t ? deepest : t;
        }
    }
    int2 *q3 = reinterpret_cast<int2 *>(&A.nodes[i].q3);
    q3[1] = make_int2((int32_t)pack[0], (int32_t)pack[1]);
    atomicMax(A.depth_out, deepest);
}

constexpr int kTopBlock = 1024;

__global__ __launch_bounds__(kTopBlock) void k_tree_pyramid(TreeArrays A, int m)
{
    build_pyramid(A.pyramid, m);
}

__global__ __launch_bounds__(kBlock) void k_tree_span(TreeArrays A, int m)
{
    const uint32_t cnt = *A.span_count;
    constexpr int per = kBlock / kSpanLanes;
    for (uint32_t q = blockIdx.x * per + threadIdx.x / kSpanLanes; q < cnt; q += gridDim.x * per)
        span_node(A, m, A.span[q]);
}

__global__ __launch_bounds__(64) void k_tree_depth(TreeArrays A)
{
    const uint32_t cnt = *A.span_count;
    for (uint32_t q = blockIdx.x * 64 + threadIdx.x; q < cnt; q += gridDim.x * 64)
        span_depth(A, A.span[q]);
}

// ---- quantised 4-wide nodes -------------------------------------------------
// Nodes at even depth become 4-wide nodes; their compact index is the prefix
// count of even-depth nodes: within kEvenNodes nodes in loc (with the parity
// in its top bit), over those blocks in bsum after k_scan_sums.
constexpr int kEvenNodes = 2048;
constexpr int kEvenBit = 0x8000;

__global__ __launch_bounds__(kBlock) void k_even_local(const uint8_t *__restrict__ rel,
                                                       const int32_t *__restrict__ sroot,
                                                       const uint8_t *__restrict__ base, int64_t ni,
                                                       uint16_t *__restrict__ loc,
                                                       uint32_t *__restrict__ bsum)
{
    constexpr int IT = kEvenNodes / kBlock;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t b0 = (int64_t)blockIdx.x * kEvenNodes + w * (64 * IT);
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    uint64_t even[IT];
    uint32_t sum = 0;
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int64_t i = b0 + r * 64 + lane;
        const bool e = i < ni && ((rel[i] + base[sroot[i]]) & 1) == 0;
        even[r] = __ballot(e);
        sum += (uint32_t)__popcll(even[r]);
    }
    __shared__ uint32_t wsum[kBlock / 64];
    if (lane == 0) wsum[w] = sum;
    __syncthreads();
    uint32_t at = 0, tot = 0;
    for (int ww = 0; ww < kBlock / 64; ++ww) {
        if (ww < w) at += wsum[ww];
        tot += wsum[ww];
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int64_t i = b0 + r * 64 + lane;
        if (i < ni)
            loc[i] = (uint16_t)((at + (uint32_t)__popcll(even[r] & lt)) |
                                ((even[r] >> lane) & 1ull ? kEvenBit : 0));
        at += (uint32_t)__popcll(even[r]);
    }
}

constexpr int kSumBlock = 1024;

__global__ __launch_bounds__(kSumBlock) void k_scan_sums(uint32_t *__restrict__ bsum, int nb,
                                                         uint32_t *__restrict__ total)
{
    uint32_t carry = 0;
    for (int base = 0; base < nb; base += kSumBlock) {
        const int i = base + threadIdx.x;
        const uint32_t v = i < nb ? bsum[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan<kSumBlock>(v, &tot);
        if (i < nb) bsum[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) total[0] = carry;
}

__device__ __forceinline__ void slot_box(const NodeRec &nd, int slot, float lo[3], float hi[3])
{
    if (slot == 0) {
        lo[0] = nd.q0.x; hi[0] = nd.q0.y; lo[1] = nd.q1.x; hi[1] = nd.q1.y;
        lo[2] = nd.q2.x; hi[2] = nd.q2.y;
    } else {
        lo[0] = nd.q0.z; hi[0] = nd.q0.w; lo[1] = nd.q1.z; hi[1] = nd.q1.w;
        lo[2] = nd.q2.z; hi[2] = nd.q2.w;
    }
}

// One 4-wide node per even-depth binary node: its children are the binary
// node's children, with every internal (odd-depth) child replaced by that
// child's own two children.  Boxes are quantised to 8 bits in the node's
// frame: scale_a = smallest power of two with 255 * scale_a >= extent_a,
// qlo = floor((lo - origin) / scale), qhi = ceil((hi - origin) / scale),
// computed in FP64 (exact here), so every decoded box contains its child.
//
// The scale's exponent and the quotients are exact without a logarithm or a
// division by the scale: ext / 255 rounds to at most 2^e exactly when
// ext <= 255 * 2^e, and scaling by a power of two is exact.
__global__ __launch_bounds__(kBlock) void k_collapse4(const NodeRec *__restrict__ nodes,
                                                      const uint16_t *__restrict__ loc,
                                                      const uint32_t *__restrict__ bsum,
                                                      int64_t ni, NodeRec *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ni || !(loc[i] & kEvenBit)) return;
    auto index4 = [&](int32_t g) {
        return bsum[g / kEvenNodes] + (uint32_t)(loc[g] & (kEvenBit - 1));
    };
    const NodeRec nd = nodes[i];
    // up to two entries for each child: itself when a leaf, else its children
    int32_t e[2][2];
    float elo[2][2][3], ehi[2][2][3];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int32_t c = s == 0 ? nd.q3.x : nd.q3.y;
        if (c < 0) {
            slot_box(nd, s, elo[s][0], ehi[s][0]);
            e[s][0] = c;
            e[s][1] = kEmptyChild;
            for (int a = 0; a < 3; ++a) {
                elo[s][1][a] = INFINITY;
                ehi[s][1][a] = -INFINITY;
            }
        } else {
            const NodeRec cd = nodes[c];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int32_t g = t == 0 ? cd.q3.x : cd.q3.y;
                slot_box(cd, t, elo[s][t], ehi[s][t]);
                e[s][t] = g < 0 ? g : (int32_t)index4(g);
            }
        }
    }
    // in order, without gaps: a lone left entry moves the right ones up
    const bool lone = e[0][1] == kEmptyChild;
    const int32_t ref[4] = {e[0][0], lone ? e[1][0] : e[0][1], lone ? e[1][1] : e[1][0],
                            lone ? kEmptyChild : e[1][1]};
    float olo[3], ohi[3], scale[3];
    uint32_t qlo[3] = {0u, 0u, 0u}, qhi[3] = {0u, 0u, 0u};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float clo[4] = {elo[0][0][a], lone ? elo[1][0][a] : elo[0][1][a],
                              lone ? elo[1][1][a] : elo[1][0][a], lone ? INFINITY : elo[1][1][a]};
        const float chi[4] = {ehi[0][0][a], lone ? ehi[1][0][a] : ehi[0][1][a],
                              lone ? ehi[1][1][a] : ehi[1][0][a], lone ? -INFINITY : ehi[1][1][a]};
        olo[a] = fminf(fminf(clo[0], clo[1]), fminf(clo[2], clo[3]));
        ohi[a] = fmaxf(fmaxf(chi[0], chi[1]), fmaxf(chi[2], chi[3]));
        const double ext = (double)ohi[a] - (double)olo[a];
        double sc = 0.0, rsc = 0.0;
        if (ext > 0.0) {
            int x;
            if (frexp(ext / 255.0, &x) == 0.5) --x;   // smallest x with 2^x >= ext / 255
            if (x < -100) x = -100;
            while (255.0 * ldexp(1.0, x) < ext) ++x;
            sc = ldexp(1.0, x);
            rsc = ldexp(1.0, -x);
        }
        scale[a] = (float)sc;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double lo = floor(((double)clo[k] - (double)olo[a]) * rsc);
            const double hi = ceil(((double)chi[k] - (double)olo[a]) * rsc);
            const bool used = ref[k] != kEmptyChild;
            qlo[a] |= used ? (uint32_t)fmin(fmax(lo, 0.0), 255.0) << (8 * k) : 0u;
            qhi[a] |= used ? (uint32_t)fmin(fmax(hi, 0.0), 255.0) << (8 * k) : 0u;
        }
    }
    NodeRec r;
    r.q0 = make_float4(olo[0], olo[1], olo[2], scale[0]);
    r.q1 = make_float4(scale[1], scale[2], __uint_as_float(qlo[0]), __uint_as_float(qhi[0]));
    r.q2 = make_float4(__uint_as_float(qlo[1]), __uint_as_float(qhi[1]), __uint_as_float(qlo[2]),
                       __uint_as_float(qhi[2]));
    r.q3 = make_int4(ref[0], ref[1], ref[2], ref[3]);
    out[index4((int32_t)i)] = r;
}

__global__ __launch_bounds__(kBlock) void k_validate(const float *__restrict__ verts, int64_t nv,
                                                     const int32_t *__restrict__ tris, int64_t nt,
                                                     int32_t *flags)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int f = 0;
    if (i < nt) {
        for (int k = 0; k < 3; ++k) {
            int32_t v = tris[3 * i + k];
            if (v < 0 || v >= nv) f |= 1;
        }
    }
    if (i < nv) {
        for (int a = 0; a < 3; ++a)
            if (!isfinite(verts[3 * i + a])) f |= 2;
    }
    if (f) atomicOr(flags, f);
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

namespace {

// tiles and digit counts of a sort of n keys
struct SortShape {
    bool small;
    int tiles, bits;
    size_t hist_bytes() const { return sizeof(uint32_t) * ((size_t)tiles << bits); }
};

SortShape sort_shape(int64_t n)
{
    SortShape s;
    s.small = n <= (int64_t)kSmallTiles * kSmallTile;
    const int64_t tile = s.small ? kSmallTile : kLargeTile;
    s.tiles = (int)((n + tile - 1) / tile);
    if (s.tiles < 1) s.tiles = 1;
    s.bits = s.small ? kSmallBits : kLargeBits;
    return s;
}

constexpr size_t kDigitTotBytes = sizeof(uint32_t) << kLargeBits;

int bound_blocks(int64_t n)
{
    const unsigned g = grid_for(n, kBlock);
    return (int)(g < (unsigned)kBoundBlocks ? g : (unsigned)kBoundBlocks);
}

// Build workspace: one carve-up for its size and its pointers.
struct BuildWs {
    float *bounds, *partial, *heap, *pyramid;
    uint32_t *keys[2], *vals[2], *hist, *digit_tot, *bsum, *span_count;
    int32_t *sroot, *span;
    uint16_t *loc;
    uint8_t *rel, *base, *sub_height;
    size_t bytes;
};

BuildWs carve_ws(char *w, int64_t n)
{
    BuildWs b;
    char *const w0 = w;
    auto take = [&](auto **p, size_t bytes) {
        *p = reinterpret_cast<std::remove_reference_t<decltype(**p)> *>(w);
        w += align_up(bytes);
    };
    const size_t nn = (size_t)n, chunks = (nn + kChunk - 1) / kChunk;
    take(&b.bounds, sizeof(float) * 6 * nn);
    for (int k = 0; k < 2; ++k) take(&b.keys[k], sizeof(uint32_t) * nn);
    for (int k = 0; k < 2; ++k) take(&b.vals[k], sizeof(uint32_t) * nn);
    take(&b.hist, sort_shape(n).hist_bytes());
    take(&b.digit_tot, kDigitTotBytes);
    take(&b.partial, sizeof(float) * 6 * (size_t)bound_blocks(n));
    take(&b.heap, sizeof(float) * 6 * kHeap * chunks);
    take(&b.pyramid, sizeof(float) * 6 * (chunks + chunks / (kPyramid - 1) + 24));
    take(&b.rel, nn);
    take(&b.base, nn);
    take(&b.sub_height, nn);
    take(&b.sroot, sizeof(int32_t) * nn);
    take(&b.span, sizeof(int32_t) * nn);
    take(&b.span_count, sizeof(uint32_t));
    take(&b.loc, sizeof(uint16_t) * nn);
    take(&b.bsum, sizeof(uint32_t) * (nn / kEvenNodes + 2));
    b.bytes = (size_t)(w - w0);
    return b;
}

}  // namespace

size_t lbvh_workspace_bytes(int64_t nt) { return carve_ws(nullptr, nt > 0 ? nt : 1).bytes; }

hipError_t validate_mesh_launch(const float *verts, int64_t nv, const int32_t *tris, int64_t nt,
                                int32_t *flags, hipStream_t s)
{
    int64_t n = nv > nt ? nv : nt;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_validate, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, verts, nv, tris,
                       nt, flags);
    return hipGetLastError();
}

namespace {

template <int B, int IT, int RB, bool SMALL>
hipError_t sort_pass(bool first, bool have_hist, const uint32_t *kin, const uint32_t *vin,
                     uint32_t *kout, uint32_t *vout, int64_t n, int shift, uint32_t *hist,
                     uint32_t *digit_tot, int tiles, hipStream_t s)
{
    const dim3 g((unsigned)tiles), b(B);
    if (!have_hist)
        hipLaunchKernelGGL((k_hist<B, IT, RB, SMALL>), g, b, 0, s, kin, n, shift, hist, tiles);
    if (!SMALL)
        hipLaunchKernelGGL(k_scan_digits, dim3(1 << RB), dim3(kBlock), 0, s, hist, tiles, digit_tot);
    if (first)
        hipLaunchKernelGGL((k_scatter<B, IT, RB, SMALL, true>), g, b, 0, s, kin, vin, kout, vout, n,
                           shift, hist, digit_tot, tiles);
    else
        hipLaunchKernelGGL((k_scatter<B, IT, RB, SMALL, false>), g, b, 0, s, kin, vin, kout, vout,
                           n, shift, hist, digit_tot, tiles);
    return hipGetLastError();
}

// One pass of the shape that n takes.  first: values are the key indices.
hipError_t sort_pass(const SortShape &sh, bool first, bool have_hist, const uint32_t *kin,
                     const uint32_t *vin, uint32_t *kout, uint32_t *vout, int64_t n, int shift,
                     uint32_t *hist, uint32_t *digit_tot, hipStream_t s)
{
    if (sh.small)
        return sort_pass<kSmallBlock, kSmallItems, kSmallBits, true>(
            first, have_hist, kin, vin, kout, vout, n, shift, hist, digit_tot, sh.tiles, s);
    return sort_pass<kLargeBlock, kLargeItems, kLargeBits, false>(
        first, have_hist, kin, vin, kout, vout, n, shift, hist, digit_tot, sh.tiles, s);
}

hipError_t lbvh_build_any(const BuildBuffers &b, const float *prim_boxes, float4 *out_pts,
                          hipStream_t s)
{
    const int64_t n = b.nt;
    if (n <= 0) return hipSuccess;
    BuildWs w = carve_ws(static_cast<char *>(b.ws), n);
    if (w.bytes > b.ws_bytes) return hipErrorInvalidValue;
    const float *bounds = prim_boxes ? prim_boxes : w.bounds;
    const int bgrid = bound_blocks(n);
    if (prim_boxes)
        hipLaunchKernelGGL(k_box_union, dim3((unsigned)bgrid), dim3(kBlock), 0, s, prim_boxes, n,
                           w.partial);
    else if (out_pts)
        hipLaunchKernelGGL(k_point_bounds, dim3((unsigned)bgrid), dim3(kBlock), 0, s, b.verts, n,
                           w.bounds, w.partial);
    else
        hipLaunchKernelGGL(k_tri_bounds, dim3((unsigned)bgrid), dim3(kBlock), 0, s, b.verts, b.tris,
                           n, w.bounds, w.partial);
    const SortShape sh = sort_shape(n);
    if (sh.small)
        hipLaunchKernelGGL((k_morton_hist<kSmallBlock, kSmallItems, kSmallBits, true>),
                           dim3((unsigned)sh.tiles), dim3(kSmallBlock), 0, s, bounds, w.partial,
                           bgrid, b.scene_box, n, b.morton_bits, b.morton, w.hist, sh.tiles,
                           w.span_count);
    else
        hipLaunchKernelGGL((k_morton_hist<kLargeBlock, kLargeItems, kLargeBits, false>),
                           dim3((unsigned)sh.tiles), dim3(kLargeBlock), 0, s, bounds, w.partial,
                           bgrid, b.scene_box, n, b.morton_bits, b.morton, w.hist, sh.tiles,
                           w.span_count);
    // the first pass reads the codes in input order, the last one writes
    // the leaf order to its place
    const uint32_t *kin = b.morton, *vin = nullptr;
    const int passes = (3 * b.morton_bits + sh.bits - 1) / sh.bits;
    for (int p = 0; p < passes; ++p) {
        uint32_t *kout = w.keys[p & 1], *vout = p == passes - 1 ? b.sorted : w.vals[p & 1];
        hipError_t e = sort_pass(sh, p == 0, p == 0, kin, vin, kout, vout, n, p * sh.bits, w.hist,
                                 w.digit_tot, s);
        if (e != hipSuccess) return e;
        kin = kout;
        vin = vout;
    }
    const int m = (int)((n + kChunk - 1) / kChunk);
    TreeArrays A;
    A.keys = kin;
    A.sorted = b.sorted;
    A.n = (int32_t)n;
    A.bounds = bounds;
    A.topo = b.topo;
    A.nodes = b.nodes;
    A.heap = w.heap;
    A.pyramid = w.pyramid;
    A.rel = w.rel;
    A.sroot = w.sroot;
    A.base = w.base;
    A.sub_height = w.sub_height;
    A.span = w.span;
    A.span_count = w.span_count;
    A.depth_out = b.depth_out;
    if (out_pts)
        hipLaunchKernelGGL(k_tree_chunk<LEAF_POINT>, dim3((unsigned)m), dim3(kTreeBlock), 0, s, A,
                           b.verts, nullptr, nullptr, out_pts);
    else if (b.trirecs)
        hipLaunchKernelGGL(k_tree_chunk<LEAF_TRI>, dim3((unsigned)m), dim3(kTreeBlock), 0, s, A,
                           b.verts, b.tris, b.trirecs, nullptr);
    else
        hipLaunchKernelGGL(k_tree_chunk<LEAF_BOX>, dim3((unsigned)m), dim3(kTreeBlock), 0, s, A,
                           nullptr, nullptr, nullptr, nullptr);
    if (m > 1) {
        if (m > kTopChunks) hipLaunchKernelGGL(k_tree_pyramid, dim3(1), dim3(kTopBlock), 0, s, A, m);
        // about 10 crossing nodes a chunk
        hipLaunchKernelGGL(k_tree_span, dim3((unsigned)m), dim3(kBlock), 0, s, A, m);
        hipLaunchKernelGGL(k_tree_depth, dim3((unsigned)((m + 3) / 4)), dim3(64), 0, s, A);
    }
    if (b.q8nodes && n > 1) {
        const int64_t ni = n - 1;
        const unsigned g = grid_for(ni, kEvenNodes);
        hipLaunchKernelGGL(k_even_local, dim3(g), dim3(kBlock), 0, s, w.rel, w.sroot, w.base, ni,
                           w.loc, w.bsum);
        hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kSumBlock), 0, s, w.bsum, (int)g, b.q8_count);
        hipLaunchKernelGGL(k_collapse4, dim3(grid_for(ni, kBlock)), dim3(kBlock), 0, s, b.nodes,
                           w.loc, w.bsum, ni, b.q8nodes);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t lbvh_build_launch(const BuildBuffers &b, hipStream_t s)
{
    return lbvh_build_any(b, nullptr, nullptr, s);
}

hipError_t lbvh_build_points_launch(const BuildBuffers &b, float4 *out_pts, hipStream_t s)
{
    if (b.trirecs || !out_pts) return hipErrorInvalidValue;
    return lbvh_build_any(b, nullptr, out_pts, s);
}

hipError_t lbvh_build_boxes_launch(const BuildBuffers &b, const float *boxes, hipStream_t s)
{
    if (b.trirecs) return hipErrorInvalidValue;
    return lbvh_build_any(b, boxes, nullptr, s);
}

size_t radix_sort_ws_bytes(int64_t n)
{
    return align_up(sort_shape(n).hist_bytes()) + align_up(kDigitTotBytes);
}

hipError_t radix_sort_launch(uint32_t *keys, uint32_t *vals, uint32_t *keys_tmp, uint32_t *vals_tmp,
                             int64_t n, int key_bits, void *ws, hipStream_t s, int *in_tmp)
{
    *in_tmp = 0;
    if (n <= 0) return hipSuccess;
    const SortShape sh = sort_shape(n);
    uint32_t *hist = static_cast<uint32_t *>(ws);
    uint32_t *digit_tot =
        reinterpret_cast<uint32_t *>(static_cast<char *>(ws) + align_up(sh.hist_bytes()));
    uint32_t *kin = keys, *kout = keys_tmp, *vin = vals, *vout = vals_tmp;
    for (int shift = 0; shift < key_bits; shift += sh.bits) {
        hipError_t e = sort_pass(sh, false, false, kin, vin, kout, vout, n, shift, hist, digit_tot,
                                 s);
        if (e != hipSuccess) return e;
        uint32_t *t = kin; kin = kout; kout = t;
        t = vin; vin = vout; vout = t;
        *in_tmp ^= 1;
    }
    return hipSuccess;
}
