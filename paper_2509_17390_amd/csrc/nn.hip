// nn.hip -- exact nearest neighbours between point clouds and the fidelity
// metrics of FGGS-LiDAR Sec. V (symmetric Chamfer distance, F-score at a
// distance threshold), gfx950.
//
// The reference cloud gets an LBVH (the shared build kernels over degenerate
// point boxes), and every query walks it nearest child first.  Distances to
// points are evaluated in FP64 from the float32 coordinates; boxes are pruned
// by a float32 bound with a margin above its rounding, so no point that could
// win or tie is lost, and the result is the FP64 minimum.  Ties go to the
// lowest reference index.  The sums of the metrics are reduced in a fixed
// order (per-block partials, then one block), so results repeat exactly.
#include "mesh_internal.h"

#include <math.h>

namespace {

constexpr int kBlock = 256;
constexpr int kStack = 64;   // the Karras tree depth is at most 62

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

__device__ __forceinline__ double axis_gap(double q, float lo, float hi)
{
    const double a = (double)lo - q, b = q - (double)hi;
    return a > 0.0 ? a : (b > 0.0 ? b : 0.0);
}

__device__ __forceinline__ double box_d2(double qx, double qy, double qz, float lx, float hx,
                                         float ly, float hy, float lz, float hz)
{
    const double dx = axis_gap(qx, lx, hx), dy = axis_gap(qy, ly, hy), dz = axis_gap(qz, lz, hz);
    return (dx * dx + dy * dy) + dz * dz;
}

__device__ __forceinline__ void leaf_test(const float4 &p, double qx, double qy, double qz,
                                          double &best, int32_t &best_i)
{
    const double dx = (double)p.x - qx, dy = (double)p.y - qy, dz = (double)p.z - qz;
    const double d2 = (dx * dx + dy * dy) + dz * dz;
    const int32_t id = __float_as_int(p.w);
    if (d2 < best || (d2 == best && id < best_i)) {
        best = d2;
        best_i = id;
    }
}

// One node a visit, box distances in FP64 with the rounded operations of the
// distance to a point inside, so that they never exceed it: exact for every
// input, infinities and NaN included.
// (Returned by value: variables whose address a caller passed would live in
// scratch memory all through its loop.)
struct Nearest {
    double d2;
    int32_t i;
};

__device__ __noinline__ Nearest search_binary(const NodeRec *__restrict__ nodes,
                                              const float4 *__restrict__ pts, double qx, double qy,
                                              double qz)
{
    double best = INFINITY;
    int32_t best_i = 0x7fffffff;
    int32_t stk[kStack];
    int sp = 0;
    stk[sp++] = 0;
    while (sp > 0) {
        const int32_t node = stk[--sp];
        const NodeRec nr = nodes[node];
        const double dl = box_d2(qx, qy, qz, nr.q0.x, nr.q0.y, nr.q1.x, nr.q1.y, nr.q2.x, nr.q2.y);
        const double dr = box_d2(qx, qy, qz, nr.q0.z, nr.q0.w, nr.q1.z, nr.q1.w, nr.q2.z, nr.q2.w);
        const int32_t cl = nr.q3.x, cr = nr.q3.y;
        // children within the best distance (ties kept: an equally near
        // point with a lower index may lie inside)
        const bool vl = dl <= best, vr = dr <= best;
        if (vl && cl < 0) leaf_test(pts[~cl], qx, qy, qz, best, best_i);
        if (vr && cr < 0) leaf_test(pts[~cr], qx, qy, qz, best, best_i);
        const bool il = vl && cl >= 0, ir = vr && cr >= 0;
        if (il && ir) {
            // the nearer child is taken next
            const bool lfirst = dl <= dr;
            if (sp + 2 <= kStack) {
                stk[sp++] = lfirst ? cr : cl;
                stk[sp++] = lfirst ? cl : cr;
            }
        } else if (il) {
            if (sp < kStack) stk[sp++] = cl;
        } else if (ir) {
            if (sp < kStack) stk[sp++] = cr;
        }
    }
    // (a node pushed before the best improved has its children tested
    // against the improved best when it is popped)
    return Nearest{best, best_i};
}

// One thread a query: launches that fill the chip, a single or no reference
// point, and references beyond pack_children.
__global__ __launch_bounds__(kBlock) void k_nearest(const NodeRec *__restrict__ nodes,
                                                    const float4 *__restrict__ pts, int64_t n_ref,
                                                    const float *__restrict__ q, int64_t n_q,
                                                    double *__restrict__ out_d,
                                                    int32_t *__restrict__ out_i)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= n_q) return;
    const double qx = q[3 * t], qy = q[3 * t + 1], qz = q[3 * t + 2];
    double best = INFINITY;
    int32_t best_i = 0x7fffffff;
    if (n_ref == 1) leaf_test(pts[0], qx, qy, qz, best, best_i);
    else if (n_ref > 1) {
        const Nearest r = search_binary(nodes, pts, qx, qy, qz);
        best = r.d2;
        best_i = r.i;
    }
    out_d[t] = n_ref > 0 ? sqrt(best) : INFINITY;
    out_i[t] = n_ref > 0 ? best_i : -1;
}

// ---------------------------------------------------------------------------
// Bounds of the shared search.  gap2 is the squared distance to a box in
// float32, off by less than 2^-21 of itself (one rounding each in the
// differences, squares and sums) or an underflow.  A box is dropped when it exceeds limit(best) =
// best (1 + 2^-19) + 1e-37, which also covers the sort key's two low bits.
// Where the best is beyond 1e38 float32 squares overflow (or nothing was
// found: infinite or NaN coordinates), and the query goes to search_binary.
constexpr int kQuadLds = 24;                 // stack entries a query in LDS (G = 4)
constexpr int kWideStack = 96;               // three pushes per two levels of 62
constexpr uint32_t kNoKey = 0x7f800000u;     // keys from here on (+inf): no candidate
constexpr int kXor1 = 0xb1, kXor2 = 0x4e, kXor3 = 0x1b;   // quad_perm controls

template <int CTRL>
__device__ __forceinline__ uint32_t quad_perm(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}

__device__ __forceinline__ float gap2(const float q[3], float lx, float hx, float ly, float hy,
                                      float lz, float hz)
{
    const float dx = fmaxf(fmaxf(lx - q[0], q[0] - hx), 0.0f);
    const float dy = fmaxf(fmaxf(ly - q[1], q[1] - hy), 0.0f);
    const float dz = fmaxf(fmaxf(lz - q[2], q[2] - hz), 0.0f);
    return fmaf(dx, dx, fmaf(dy, dy, dz * dz));
}

__device__ __forceinline__ float limit(double best)
{
    return fmaf((float)best, 1.0f + 1.9073486328125e-06f, 1e-37f);
}

template <int CTRL>
__device__ __forceinline__ void merge_best(double &best, int32_t &best_i)
{
    const uint64_t w = (uint64_t)__double_as_longlong(best);
    const uint64_t o = (uint64_t)quad_perm<CTRL>((uint32_t)w) |
                       ((uint64_t)quad_perm<CTRL>((uint32_t)(w >> 32)) << 32);
    const double d = __longlong_as_double((long long)o);
    const int32_t i = (int32_t)quad_perm<CTRL>((uint32_t)best_i);
    const bool b = d < best || (d == best && i < best_i);
    best = b ? d : best;
    best_i = b ? i : best_i;
}

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Workgroups are dealt to the 8 XCDs in turn (workgroup b on XCD b % 8): give
// each XCD one contiguous run of the queries, so that queries near each other
// (a scan's, beam by beam) share the records in an L2.  gridDim.x is a
// multiple of 8.
__device__ __forceinline__ int64_t xcd_block()
{
    return (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
}

inline unsigned xcd_grid(int64_t n, int per_block) { return (grid_for(n, per_block) + 7) / 8 * 8; }

// Four lanes a query, two levels a visit (see pack_children): the two records
// that name's children are fetched at once and each lane takes one of their
// four boxes; a child that is a point itself is measured at once.  A search is
// a chain of dependent fetches (12 such visits on average, 77 the longest, on
// scans of a room), so a launch that does not fill the chip ends with its
// longest query: 5,000 / 50,000 / 131,072 queries on 250,001 points take some
// 35 / 55 / 85 us where one thread a query takes 70 / 80 / 104.  Beyond
// quad_queries (400,000: 215 against 190) the shared queries' extra instructions
// cost more.
__global__ __launch_bounds__(64) void k_nearest_quad(const NodeRec *__restrict__ nodes,
                                                     const float4 *__restrict__ pts,
                                                     const float *__restrict__ q, int64_t n_q,
                                                     double *__restrict__ out_d,
                                                     int32_t *__restrict__ out_i)
{
    __shared__ uint64_t s_stk[kQuadLds][16];
    const int lane = threadIdx.x, j = lane & 3;
    const int64_t t = xcd_block() * 16 + (lane >> 2);
    if (t >= n_q) return;
    uint64_t *stk = &s_stk[0][lane >> 2];
    uint64_t deep[kWideStack - kQuadLds];
    const float qf[3] = {q[3 * t], q[3 * t + 1], q[3 * t + 2]};
    const double qx = qf[0], qy = qf[1], qz = qf[2];
    double best = INFINITY;
    int32_t best_i = 0x7fffffff;
    float lim = INFINITY;
    int sp = 0;
    const int which = j >> 1, slot = j & 1;
    uint32_t name = pack_children(nodes[0].q3.x, nodes[0].q3.y);
    // this lane's record of a node's children (a point's place: the root's,
    // not used)
    auto fetch = [&](uint32_t w) {
        return nodes[(w >> which) & 1u ? 0 : (int32_t)(w >> 2) + which];
    };
    NodeRec nr = fetch(name);
    bool more = true;
    while (more) {
        const bool point = (name >> which) & 1u;
        const float dl = gap2(qf, nr.q0.x, nr.q0.y, nr.q1.x, nr.q1.y, nr.q2.x, nr.q2.y);
        const float dr = gap2(qf, nr.q0.z, nr.q0.w, nr.q1.z, nr.q1.w, nr.q2.z, nr.q2.w);
        const float d = point ? (slot ? INFINITY : 0.0f) : (slot ? dr : dl);
        const int32_t ref = point ? ~((int32_t)(name >> 2) + which) : (slot ? nr.q3.y : nr.q3.x);
        const uint32_t sub = (uint32_t)(slot ? nr.q3.w : nr.q3.z);
        // the point first, then the next node, so that both fetches overlap;
        // the next node is chosen before the points have lowered the limit
        const bool pt = ref < 0 && d <= lim && d < INFINITY;
        const float4 pv = pts[pt ? ~ref : 0];
        const bool in = ref >= 0 && d <= fminf(lim, 3.402823466e38f);
        const uint32_t key = ((in ? __float_as_uint(d) : kNoKey) & ~3u) | (uint32_t)j;
        uint32_t nh = in ? 1u : 0u;
        const uint32_t k1 = quad_perm<kXor1>(key), k2 = quad_perm<kXor2>(key),
                       k3 = quad_perm<kXor3>(key);
        const int rank = (k1 < key) + (k2 < key) + (k3 < key);
        nh += quad_perm<kXor1>(nh);
        nh += quad_perm<kXor2>(nh);
        const int top = sp + (int)nh - 1, at = top - rank;   // farthest lowest
        if (in && rank > 0 && at < kQuadLds) stk[16 * at] = (uint64_t)sub | ((uint64_t)key << 32);
        if (top > kQuadLds)
            for (int o = 0; o < 4; ++o) {   // every lane keeps candidate o
                const int src = lane - j + o;
                const uint32_t k = (uint32_t)__shfl((int)key, src, 64);
                const uint32_t e = (uint32_t)__shfl((int)sub, src, 64);
                const int r = __shfl(rank, src, 64);
                if (k < kNoKey && r > 0 && top - r >= kQuadLds && top - r < kWideStack)
                    deep[top - r - kQuadLds] = (uint64_t)e | ((uint64_t)k << 32);
            }
        wave_sync();   // a lane's entries are read by the quad's others
        uint32_t next = in && rank == 0 ? sub : 0u;
        next |= quad_perm<kXor1>(next);
        next |= quad_perm<kXor2>(next);
        more = nh > 0;
        name = next;
        sp = more ? top : sp;
        while (!more && sp > 0) {
            --sp;
            uint64_t w;
            if (sp < kQuadLds) w = stk[16 * sp];
            else w = deep[sp - kQuadLds];
            more = __uint_as_float((uint32_t)(w >> 32)) <= lim;
            name = (uint32_t)w;
        }
        nr = fetch(more ? name : 3u);
        if (__ballot(pt)) {
            if (pt) leaf_test(pv, qx, qy, qz, best, best_i);
            merge_best<kXor1>(best, best_i);
            merge_best<kXor2>(best, best_i);
            lim = limit(best);
        }
        wave_sync();
    }
    if (j == 0) {
        if (!(best <= 1e38)) {
            const Nearest r = search_binary(nodes, pts, qx, qy, qz);
            best = r.d2;
            best_i = r.i;
        }
        out_d[t] = sqrt(best);
        out_i[t] = best_i;
    }
}

// per-block partial sums of d and of [d <= tau], fixed order
__global__ __launch_bounds__(kBlock) void k_metric_partials(const double *__restrict__ d,
                                                            int64_t n, double tau,
                                                            double *__restrict__ sum_out,
                                                            unsigned long long *__restrict__ cnt_out)
{
    __shared__ double ss[kBlock];
    __shared__ unsigned long long sc[kBlock];
    double s = 0.0;
    unsigned long long c = 0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        s += d[i];
        c += d[i] <= tau ? 1ull : 0ull;
    }
    ss[threadIdx.x] = s;
    sc[threadIdx.x] = c;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            ss[threadIdx.x] += ss[threadIdx.x + w];
            sc[threadIdx.x] += sc[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sum_out[blockIdx.x] = ss[0];
        cnt_out[blockIdx.x] = sc[0];
    }
}

// The partials added one after another, in block order, from LDS: from global
// memory the chain of 1,024 loads took 79 us, this takes 8.
constexpr int kMetricBlocks = 1024;

__global__ __launch_bounds__(kBlock) void k_metric_final(const double *__restrict__ sums,
                                                         const unsigned long long *__restrict__ cnts,
                                                         int nb, double *__restrict__ out_sum,
                                                         unsigned long long *__restrict__ out_cnt)
{
    __shared__ double ss[kMetricBlocks];
    __shared__ unsigned long long sc[kMetricBlocks];
    for (int b = threadIdx.x; b < nb; b += kBlock) {
        ss[b] = sums[b];
        sc[b] = cnts[b];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll 16
        for (int b = 0; b < nb; ++b) s += ss[b];
        *out_sum = s;
    } else if (threadIdx.x == 64) {
        unsigned long long c = 0;
#pragma unroll 16
        for (int b = 0; b < nb; ++b) c += sc[b];
        *out_cnt = c;
    }
}

}  // namespace

// Queries up to which four lanes share one: more for larger clouds, whose
// chains of fetches are longer.  us a call (build and search), four lanes / one,
// queries ordered by azimuth (random order likewise):
//     queries    1,000 points   5,000       50,000      250,001     1,000,000
//      65,536     115 / 130
//     100,000     124 / 135    146 / 159   172 / 201   224 / 282   315 / 386
//     150,000                  165 / 165   198 / 209   252 / 288   337 / 422
//     200,000                  177 / 173   214 / 218   268 / 314   359 / 425
//     230,000                  190 / 174   225 / 226   283 / 328   391 / 442
//     262,144                  198 / 177   236 / 231   297 / 346   402 / 457
//     300,000                  211 / 188   251 / 244   312 / 352   432 / 478
//     350,000                  225 / 202   267 / 253   333 / 357   449 / 484
static int64_t quad_queries(int64_t n_ref)
{
    int bits = 0;
    while (bits < 19 && (n_ref >> (bits + 1)) > 0) ++bits;
    return (int64_t)(bits < 11 ? 3 : bits - 8) << 15;
}

size_t nn_scratch_bytes(int64_t n_ref)
{
    const int64_t ni = n_ref > 1 ? n_ref - 1 : 1;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    return 2 * al(4 * (size_t)n_ref) + al(12 * (size_t)ni) +
           al(sizeof(NodeRec) * (size_t)ni) + al(16 * (size_t)n_ref) + al(64) +
           al(sizeof(double) * kMetricBlocks) + al(8 * kMetricBlocks) + al(16);
}

size_t nn_workspace_bytes(int64_t n_ref) { return lbvh_workspace_bytes(n_ref > 0 ? n_ref : 1); }

hipError_t nearest_launch(const float *ref, int64_t n_ref, const float *query, int64_t n_q,
                          double *out_d, int32_t *out_i, void *scratch, void *ws, size_t ws_bytes,
                          hipStream_t s)
{
    const int64_t ni = n_ref > 1 ? n_ref - 1 : 1;
    char *w = static_cast<char *>(scratch);
    auto take = [&](size_t bytes) {
        char *p = w;
        w += (bytes + 255) & ~(size_t)255;
        return p;
    };
    uint32_t *morton = reinterpret_cast<uint32_t *>(take(4 * (size_t)n_ref));
    uint32_t *sorted = reinterpret_cast<uint32_t *>(take(4 * (size_t)n_ref));
    int32_t *topo = reinterpret_cast<int32_t *>(take(12 * (size_t)ni));
    NodeRec *nodes = reinterpret_cast<NodeRec *>(take(sizeof(NodeRec) * (size_t)ni));
    float4 *pts = reinterpret_cast<float4 *>(take(16 * (size_t)n_ref));
    float *box_dev = reinterpret_cast<float *>(take(64));
    if (n_ref > 0) {
        BuildBuffers b;
        b.verts = ref;
        b.tris = nullptr;
        b.nv = 0;
        b.nt = n_ref;
        b.morton_bits = 10;
        b.ws = ws;
        b.ws_bytes = ws_bytes;
        b.morton = morton;
        b.sorted = sorted;
        b.topo = topo;
        b.nodes = nodes;
        b.trirecs = nullptr;
        b.scene_box = box_dev;
        b.depth_out = reinterpret_cast<int32_t *>(box_dev + 6);
        b.q8nodes = nullptr;
        b.q8_count = nullptr;
        hipError_t e = lbvh_build_points_launch(b, pts, s);
        if (e != hipSuccess) return e;
    }
    if (n_q > 0 && n_q <= quad_queries(n_ref) && n_ref > 1 && n_ref <= kPackMaxTris) {
        hipLaunchKernelGGL(k_nearest_quad, dim3(xcd_grid(n_q, 16)), dim3(64), 0, s, nodes, pts,
                           query, n_q, out_d, out_i);
    } else if (n_q > 0)
        hipLaunchKernelGGL(k_nearest, dim3(grid_for(n_q, kBlock)), dim3(kBlock), 0, s, nodes, pts,
                           n_ref, query, n_q, out_d, out_i);
    return hipGetLastError();
}

hipError_t metric_sums_launch(const double *d, int64_t n, double tau, void *scratch, size_t off,
                              double *out_sum, unsigned long long *out_cnt, hipStream_t s)
{
    char *w = static_cast<char *>(scratch) + off;
    double *sums = reinterpret_cast<double *>(w);
    unsigned long long *cnts =
        reinterpret_cast<unsigned long long *>(w + ((sizeof(double) * kMetricBlocks + 255) & ~(size_t)255));
    const int nb = (int)(grid_for(n, kBlock) < (unsigned)kMetricBlocks ? grid_for(n, kBlock)
                                                                       : (unsigned)kMetricBlocks);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(k_metric_partials, dim3(nb), dim3(kBlock), 0, s, d, n, tau, sums, cnts);
    hipLaunchKernelGGL(k_metric_final, dim3(1), dim3(kBlock), 0, s, sums, cnts, nb, out_sum, out_cnt);
    return hipGetLastError();
}

size_t nn_metric_offset(int64_t n_ref)
{
    const int64_t ni = n_ref > 1 ? n_ref - 1 : 1;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    return 2 * al(4 * (size_t)n_ref) + al(12 * (size_t)ni) +
           al(sizeof(NodeRec) * (size_t)ni) + al(16 * (size_t)n_ref) + al(64);
}
