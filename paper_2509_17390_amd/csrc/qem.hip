// qem.hip -- quadric-error decimation by rounds of parallel edge
// contraction on gfx950 (FGGS-LiDAR Sec. IV-B "Mesh optimization":
// quadric-error decimation to a face ratio; Sec. V: ratio 0.1, three
// rounds, boundary protected).
//
// The quadric error metric is Garland and Heckbert's (1997): a vertex
// carries the sum of the squared-distance quadrics of its faces' planes, an
// edge (u, v) contracts to the point x* minimising x^T (Q_u + Q_v) x at that
// minimum's cost, cheapest first.  One contraction at a time is sequential;
// here a step contracts an independent set of locally cheapest edges at
// once, so the work of a step is data-parallel over vertices, edges and
// faces:
//
//   round k = 1..R runs until at most ceil(F0 ratio^(k/R)) faces remain (or
//   nothing can contract); at its start the plane quadrics are summed anew
//   and the vertices on a boundary or non-manifold edge (an edge not on
//   exactly two faces) are protected for the round.  One step:
//   1. incidence from the live faces: each vertex's faces (ascending) and
//      its distinct neighbours (ascending); edges (u < v) numbered in
//      lexicographic order by a scan of the neighbour counts above u;
//   2. candidates: edges on exactly two faces, both ends unprotected,
//      exactly two common neighbours (the link condition, so a closed
//      manifold stays closed and manifold); x* is A^-1 b by Cramer's rule
//      when A (the 3x3 block of Q_u + Q_v) is well conditioned and x* lies
//      near the edge, else the cheapest of the ends and the midpoint; an
//      edge whose contraction would flip a face is dropped; key = (float32
//      cost, pi(edge number)) with pi a fixed bijection of 32-bit integers,
//      so exactly equal costs (flat regions) are ordered pseudo-randomly
//      and the locally cheapest edges are many, not one per flat region;
//   3. the ceil((F - T) / 2) smallest keys are eligible (a radix select of
//      the threshold key; an interior contraction removes two faces);
//   4. an eligible edge contracts when no eligible edge at any vertex of
//      its two closed one-rings has a smaller key (per-vertex 64-bit atomic
//      minima); no end of such an edge is an end or a neighbour of an end
//      of another, so their contractions touch disjoint faces and run in
//      place;
//   5. faces are renamed through the contraction map; the two faces of
//      each contracted edge degenerate and are dropped.
// A step changes the mesh only inside the closed one-rings of the edges it
// contracts: the next step rebuilds the incidence and evaluates the edges
// of those ("dirty") vertices alone, and every other edge keeps its cost
// and point under its new number.
// The steps run without the host: the state of the loop (faces, target, edge
// counts, whether the round is over) is on the device, every launch of a step
// after a round's end returns at once, and the host reads the state once per
// batch of steps.
// Positions, quadrics and costs are FP64 throughout, each operation in a
// fixed order (compiled with -ffp-contract=off), so a run is deterministic
// and matches a plain CPU evaluation of the same steps; positions are
// rounded to float32 once, at the end.
#include "mesh_internal.h"

#include <float.h>
#include <math.h>
#include <stddef.h>

namespace {

constexpr int kBlock = 256;
constexpr uint64_t kNone = ~0ull;

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

// Adds v of every thread of the block to *dst with one atomic: a
// shuffle-reduction per wave, then the waves' sums through LDS (a counter
// that every thread of a large launch hit directly serialised the launch).
// Every thread of the block must call it.
__device__ __forceinline__ void block_add(uint32_t v, uint32_t *dst)
{
    __shared__ uint32_t part[kBlock / 64];
    __syncthreads();   // an earlier call's sum is read before part is reused
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < kBlock / 64; ++w) t += part[w];
        if (t) atomicAdd(dst, t);
    }
}

// Radix select state: keys whose bits under `mask` equal `prefix` hold the
// rank-th smallest.
struct SelState {
    unsigned long long prefix, mask;
    unsigned long long rank;
    uint32_t done;        // prefix is the selected key, or an equal bound
    uint32_t ticket;      // blocks of the running pass that have finished
};
static_assert(offsetof(SelState, prefix) == 0, "the selected key is read at offset 0");

struct QemState {
    SelState sel;
    QemLoop loop;
    uint32_t flags;       // 1: too many faces at a vertex, 2: too many neighbours
    uint32_t n_old;       // edges of the step before
};

// Counters of a step: kQemSlots lines of (candidates, contracted, faces
// dropped), a block adding to the line of its number.  (One address for all
// blocks takes 4.5 ns an addition: 12 us at 2,700 blocks.)
struct QemSlot {
    uint32_t cand, chosen, killed, pad[13];
};
__device__ __forceinline__ QemSlot *slot_of(QemSlot *slots, int nslots)
{
    return slots + (blockIdx.x & (unsigned)(nslots - 1));
}

// This thread's value to be added up over a group of G lanes, by all of them
template <int G>
__device__ __forceinline__ uint32_t group_sum(uint32_t v)
{
#pragma unroll
    for (int o = 1; o < G; o <<= 1) v += (uint32_t)__shfl_xor((int)v, o, G);
    return v;
}

// the group's lanes for which c holds
template <int G>
__device__ __forceinline__ uint32_t group_ballot(bool c)
{
    return (uint32_t)(__ballot(c) >> (threadIdx.x & 63 & ~(unsigned)(G - 1))) & ((1u << G) - 1u);
}

// LDS written by this wave is read by it next
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The threads of the block with c listed in LDS, in no order: their numbers
// into list, returns how many.  Every thread of the block must call it.
__device__ __forceinline__ uint32_t block_list(bool c, uint16_t *list, uint32_t *count)
{
    if (threadIdx.x == 0) *count = 0;
    __syncthreads();
    const uint64_t m = __ballot(c);
    const int lane = (int)(threadIdx.x & 63);
    uint32_t base = 0;
    if (lane == 0 && m) base = atomicAdd(count, (uint32_t)__popcll(m));
    base = (uint32_t)__shfl((int)base, 0, 64);
    if (c) list[base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)threadIdx.x;
    __syncthreads();
    return *count;
}

// Exclusive offsets of the block's values, and its total to sums[blockIdx.x].
__device__ __forceinline__ uint32_t block_offsets(uint32_t v, uint32_t *__restrict__ sums)
{
    __shared__ uint32_t part[kBlock / 64];
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) part[w] = x;
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (int k = 0; k < kBlock / 64; ++k) {
        if (k < w) before += part[k];
        tot += part[k];
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
    return before + x - v;
}

// pi: "lowbias32" of C. Wellons' hash prospector (xorshift-multiply rounds,
// each invertible mod 2^32, so pi is a bijection and keys stay unique)
__device__ __forceinline__ uint32_t perm32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

__device__ __forceinline__ void cross3(const double a[3], const double b[3], double r[3])
{
    r[0] = a[1] * b[2] - a[2] * b[1];
    r[1] = a[2] * b[0] - a[0] * b[2];
    r[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ __forceinline__ double dot3(const double a[3], const double b[3])
{
    return (a[0] * b[0] + a[1] * b[1]) + a[2] * b[2];
}

// n = (b - a) x (c - a)
__device__ __forceinline__ void face_normal(const double a[3], const double b[3],
                                            const double c[3], double n[3])
{
    const double e1[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
    const double e2[3] = {c[0] - a[0], c[1] - a[1], c[2] - a[2]};
    cross3(e1, e2, n);
}

__device__ __forceinline__ void load3(const double *__restrict__ P, int i, double r[3])
{
    r[0] = P[3 * (int64_t)i];
    r[1] = P[3 * (int64_t)i + 1];
    r[2] = P[3 * (int64_t)i + 2];
}

// Plane quadric K = q q^T / (n.n) of a face, q = (n, -n.a), upper triangle
// row by row: (00 01 02 03 11 12 13 22 23 33); zero for a degenerate face.
__device__ void plane_quadric(const double a[3], const double b[3], const double c[3],
                              double K[10])
{
    double n[3];
    face_normal(a, b, c, n);
    const double nn = dot3(n, n);
    if (nn == 0.0) {
        for (int i = 0; i < 10; ++i) K[i] = 0.0;
        return;
    }
    const double q[4] = {n[0], n[1], n[2], -dot3(n, a)};
    int k = 0;
    for (int i = 0; i < 4; ++i)
        for (int j = i; j < 4; ++j) K[k++] = (q[i] * q[j]) / nn;
}

// [x 1] Q [x 1]^T
__device__ __forceinline__ double quadric_cost(const double Q[10], const double x[3])
{
    const double r0 = ((Q[0] * x[0] + Q[1] * x[1]) + Q[2] * x[2]) + Q[3];
    const double r1 = ((Q[1] * x[0] + Q[4] * x[1]) + Q[5] * x[2]) + Q[6];
    const double r2 = ((Q[2] * x[0] + Q[5] * x[1]) + Q[7] * x[2]) + Q[8];
    const double r3 = ((Q[3] * x[0] + Q[6] * x[1]) + Q[8] * x[2]) + Q[9];
    return ((x[0] * r0 + x[1] * r1) + x[2] * r2) + r3;
}

// x* = A^-1 b by Cramer's rule (cofactors along the first row) when
// trace(A) > 0 and |det A| > 1e-6 (trace / 3)^3; false otherwise.
__device__ bool minimiser(const double Q[10], double x[3])
{
    const double a00 = Q[0], a01 = Q[1], a02 = Q[2], b0 = -Q[3];
    const double a11 = Q[4], a12 = Q[5], b1 = -Q[6];
    const double a22 = Q[7], b2 = -Q[8];
    const double det = (a00 * (a11 * a22 - a12 * a12) - a01 * (a01 * a22 - a12 * a02)) +
                       a02 * (a01 * a12 - a11 * a02);
    const double tr = (a00 + a11) + a22;
    const double t3 = tr / 3.0;
    if (!(tr > 0.0 && fabs(det) > 1e-6 * ((t3 * t3) * t3))) return false;
    x[0] = ((b0 * (a11 * a22 - a12 * a12) - a01 * (b1 * a22 - a12 * b2)) +
            a02 * (b1 * a12 - a11 * b2)) / det;
    x[1] = ((a00 * (b1 * a22 - a12 * b2) - b0 * (a01 * a22 - a12 * a02)) +
            a02 * (a01 * b2 - b1 * a02)) / det;
    x[2] = ((a00 * (a11 * b2 - b1 * a12) - a01 * (a01 * b2 - b1 * a02)) +
            b0 * (a01 * a12 - a11 * a02)) / det;
    return true;
}

// Placement of an edge's contraction and its cost: x* when it lies within
// twice the edge length of the midpoint m, else the cheapest of pu, pv, m
// (the first on a tie).
__device__ double placement(const double Q[10], const double pu[3], const double pv[3],
                            double x[3])
{
    const double m[3] = {0.5 * (pu[0] + pv[0]), 0.5 * (pu[1] + pv[1]), 0.5 * (pu[2] + pv[2])};
    bool ok = minimiser(Q, x);
    if (ok) {
        const double dx[3] = {x[0] - m[0], x[1] - m[1], x[2] - m[2]};
        const double e[3] = {pv[0] - pu[0], pv[1] - pu[1], pv[2] - pu[2]};
        ok = dot3(dx, dx) <= 4.0 * dot3(e, e);
    }
    if (!ok) {
        // the cheapest of pu, pv, m; the first on a tie
        const double cu = quadric_cost(Q, pu), cv = quadric_cost(Q, pv), cm = quadric_cost(Q, m);
        const bool tv = cv < cu;
        const double cb = tv ? cv : cu;
        const bool tm = cm < cb;
        for (int i = 0; i < 3; ++i) x[i] = tm ? m[i] : (tv ? pv[i] : pu[i]);
    }
    return quadric_cost(Q, x);
}

__global__ __launch_bounds__(kBlock) void k_qem_init(const float *__restrict__ verts, int64_t nv,
                                                     const int32_t *__restrict__ tris, int64_t nt,
                                                     double *__restrict__ P,
                                                     int32_t *__restrict__ F)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < nv)
        for (int k = 0; k < 3; ++k) P[3 * i + k] = (double)verts[3 * i + k];
    if (i < nt) {
        const int32_t a = tris[3 * i], b = tris[3 * i + 1], c = tris[3 * i + 2];
        // a face with a repeated corner is no triangle: dropped at once
        const bool dead = a == b || b == c || a == c;
        F[3 * i] = dead ? -1 : a;
        F[3 * i + 1] = b;
        F[3 * i + 2] = c;
    }
}

__global__ __launch_bounds__(kBlock) void k_qem_fill_faces(const int32_t *__restrict__ F,
                                                           int64_t nt, uint32_t *__restrict__ fcnt,
                                                           int32_t *__restrict__ fl,
                                                           uint32_t *__restrict__ flags)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= nt || F[3 * t] < 0) return;
    for (int k = 0; k < 3; ++k) {
        const int32_t v = F[3 * t + k];
        const uint32_t s = atomicAdd(&fcnt[v], 1u);
        if (s < (uint32_t)kQemFaces) fl[(int64_t)v * kQemFaces + s] = (int32_t)t;
        else atomicOr(&flags[0], 1u);
    }
}

__device__ __forceinline__ bool face_has(const int32_t *__restrict__ F, int32_t t, int32_t w)
{
    return F[3 * (int64_t)t] == w || F[3 * (int64_t)t + 1] == w || F[3 * (int64_t)t + 2] == w;
}

// The distinct neighbours of v (ascending) from its n faces f into b;
// returns their number (at most kQemNbrs, else flags[0] |= 2).
__device__ int build_ring(const int32_t *__restrict__ F, const int32_t *f, int n, int64_t v,
                          int32_t *b, uint32_t *__restrict__ flags)
{
    int m = 0;
    for (int k = 0; k < n; ++k)
        for (int c = 0; c < 3; ++c) {
            const int32_t w = F[3 * (int64_t)f[k] + c];
            if (w == (int32_t)v) continue;
            int j = m;
            while (j > 0 && b[j - 1] > w) --j;
            if (j > 0 && b[j - 1] == w) continue;
            if (m == kQemNbrs) {
                atomicOr(&flags[0], 2u);
                continue;
            }
            for (int i = m; i > j; --i) b[i] = b[i - 1];
            b[j] = w;
            ++m;
        }
    return m;
}

// Per vertex: sort its faces, collect its distinct neighbours (ascending),
// count those above it, sum its faces' plane quadrics (ascending face order)
// and protect it when an edge at it is not on exactly two faces.  (A round's
// start.)  One thread, any number of faces.
__device__ void vertex_serial(const double *__restrict__ P, const int32_t *__restrict__ F,
                              int64_t v, int n, int32_t *__restrict__ fl,
                              int32_t *__restrict__ fdeg, int32_t *__restrict__ nb,
                              int32_t *__restrict__ ndeg, uint32_t *__restrict__ nlarge,
                              double *__restrict__ Q, uint8_t *__restrict__ prot,
                              uint32_t *__restrict__ flags)
{
    int32_t *f = fl + v * kQemFaces;
    for (int k = 1; k < n; ++k) {
        const int32_t x = f[k];
        int j = k;
        while (j > 0 && f[j - 1] > x) {
            f[j] = f[j - 1];
            --j;
        }
        f[j] = x;
    }
    fdeg[v] = n;
    int32_t *b = nb + v * kQemNbrs;
    const int m = build_ring(F, f, n, v, b, flags);
    ndeg[v] = m;
    uint32_t above = 0;
    for (int k = 0; k < m; ++k) above += b[k] > (int32_t)v ? 1u : 0u;
    nlarge[v] = above;
    double acc[10];
    for (int i = 0; i < 10; ++i) acc[i] = 0.0;
    for (int k = 0; k < n; ++k) {
        const int64_t t = f[k];
        double pa[3], pb[3], pc[3], K[10];
        load3(P, F[3 * t], pa);
        load3(P, F[3 * t + 1], pb);
        load3(P, F[3 * t + 2], pc);
        plane_quadric(pa, pb, pc, K);
        for (int i = 0; i < 10; ++i) acc[i] = acc[i] + K[i];
    }
    for (int i = 0; i < 10; ++i) Q[10 * v + i] = acc[i];
    uint8_t p = 0;
    for (int k = 0; k < m && !p; ++k) {
        int cnt = 0;
        for (int i = 0; i < n; ++i) cnt += face_has(F, f[i], b[k]) ? 1 : 0;
        p = cnt != 2 ? 1 : 0;
    }
    prot[v] = p;
}

// Between a round's steps, per dirty vertex: its live faces are those of
// its previous list still alive (a contraction renames faces, it never
// adds a face to a vertex it did not touch), plus, for the u of a
// contracted edge (u, v), the live faces of v's list, merged in ascending
// order; then its neighbours anew.  v itself is left to u's lanes, which
// empty v's lists after reading them.  One thread; returns the neighbours
// above v.
__device__ uint32_t vertex_update_serial(const int32_t *__restrict__ F, int64_t v,
                                         int32_t *__restrict__ absorbed, int32_t *fl, int32_t *fdeg,
                                         int32_t *__restrict__ nb, int32_t *__restrict__ ndeg,
                                         uint32_t *__restrict__ flags)
{
    int32_t *f = fl + v * kQemFaces;
    const int n0 = fdeg[v];
    int a = 0;
    for (int k = 0; k < n0; ++k) {
        const int32_t t = f[k];
        if (F[3 * (int64_t)t] >= 0) f[a++] = t;
    }
    int n = a;
    const int32_t w = absorbed[v];
    if (w >= 0) {
        absorbed[v] = -1;
        const int32_t *g = fl + (int64_t)w * kQemFaces;
        const int m0 = fdeg[w];
        int nb_live = 0;
        for (int k = 0; k < m0; ++k) nb_live += F[3 * (int64_t)g[k]] >= 0 ? 1 : 0;
        if (a + nb_live > kQemFaces) {
            atomicOr(&flags[0], 1u);
        } else {
            // merge from the top: v's own list sits at the front of the
            // destination, so no entry is overwritten before it is read
            int i = a - 1, j = m0 - 1;
            for (int o = a + nb_live - 1; o > i; --o) {
                while (F[3 * (int64_t)g[j]] < 0) --j;
                if (i < 0 || g[j] > f[i]) f[o] = g[j--];
                else f[o] = f[i--];
            }
            n = a + nb_live;
        }
        fdeg[w] = 0;
        ndeg[w] = 0;
    }
    fdeg[v] = n;
    int32_t *b = nb + v * kQemNbrs;
    const int m = build_ring(F, f, n, v, b, flags);
    ndeg[v] = m;
    uint32_t above = 0;
    for (int k = 0; k < m; ++k) above += b[k] > (int32_t)v ? 1u : 0u;
    return above;
}

constexpr int kUpLanes = 8, kUpList = 32, kUpEach = kUpList / kUpLanes;
constexpr int32_t kGone = 0x7fffffff;

// The lists of a vertex v from the faces t and their corners besides v, x, of
// its 8 lanes (row q: faces 8 q on, kGone where there is none), which s_face
// and s_ring hold in the same order: a face's place is the number of faces
// below it, a neighbour's the number of distinct ones below it.  m and above:
// this lane's neighbours, and those above v.  START: leaves s_face in order and
// returns whether one of this lane's neighbours is not on exactly two faces.
template <int ROWS, bool START>
__device__ __forceinline__ bool group_lists(int gl, int64_t v, int4 *s_face,
                                            int4 *s_ring, const int32_t (&t)[kUpEach],
                                            int32_t (&x)[kUpEach][2], int32_t *fl,
                                            int32_t *__restrict__ nb, uint32_t &m, uint32_t &above)
{
    constexpr int kUnroll = ROWS > 1 ? 1 : 4;
    int32_t *faces = reinterpret_cast<int32_t *>(s_face);
    int32_t *ring = reinterpret_cast<int32_t *>(s_ring);
    int place[ROWS] = {}, met[ROWS][2] = {};
    bool again[ROWS][2] = {};      // met before: the first of a value stays
#pragma unroll(kUnroll)
    for (int i = 0; i < 2 * ROWS; ++i) {
        const int4 f = s_face[i];
#pragma unroll
        for (int q = 0; q < ROWS; ++q)
            place[q] += (f.x < t[q]) + (f.y < t[q]) + (f.z < t[q]) + (f.w < t[q]);
    }
#pragma unroll(kUnroll)
    for (int i = 0; i < 4 * ROWS; ++i) {
        const int4 r = s_ring[i];
#pragma unroll
        for (int q = 0; q < ROWS; ++q)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int e = 2 * (q * kUpLanes + gl) + k - 4 * i, y = x[q][k];
                again[q][k] |= (e > 0 && r.x == y) || (e > 1 && r.y == y) ||
                               (e > 2 && r.z == y) || (e > 3 && r.w == y);
                if (START) met[q][k] += (r.x == y) + (r.y == y) + (r.z == y) + (r.w == y);
            }
    }
    wave_lds_fence();
#pragma unroll
    for (int q = 0; q < ROWS; ++q) {
        if (t[q] != kGone) {
            fl[v * kQemFaces + place[q]] = t[q];
            if (START) faces[place[q]] = t[q];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (again[q][k]) x[q][k] = ring[2 * (q * kUpLanes + gl) + k] = kGone;
    }
    wave_lds_fence();
    int spot[ROWS][2] = {};
#pragma unroll(kUnroll)
    for (int i = 0; i < 4 * ROWS; ++i) {
        const int4 r = s_ring[i];
#pragma unroll
        for (int q = 0; q < ROWS; ++q)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int y = x[q][k];
                spot[q][k] += (r.x < y) + (r.y < y) + (r.z < y) + (r.w < y);
            }
    }
    m = above = 0;
    bool odd = false;
#pragma unroll
    for (int q = 0; q < ROWS; ++q) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (x[q][k] != kGone) {
                nb[v * kQemNbrs + spot[q][k]] = x[q][k];
                ++m;
                above += x[q][k] > (int32_t)v ? 1u : 0u;
                odd |= met[q][k] != 2;
            }
    }
    return START && odd;
}

// By the wave's longest list: vertices have 6 faces and up to two rows when one
// was contracted into them.  (One form for any number of rows: 79 and 22.7 us
// for the two kernels where this takes 62 and 19.5, means of a decimation from
// 262,000 vertices.)
template <bool START>
__device__ __forceinline__ bool wave_lists(int rows, int gl, int64_t v, int4 *s_face, int4 *s_ring,
                                           const int32_t (&t)[kUpEach], int32_t (&x)[kUpEach][2],
                                           int32_t *fl, int32_t *__restrict__ nb, uint32_t &m,
                                           uint32_t &above)
{
    if (rows == 1) return group_lists<1, START>(gl, v, s_face, s_ring, t, x, fl, nb, m, above);
    if (rows == 2) return group_lists<2, START>(gl, v, s_face, s_ring, t, x, fl, nb, m, above);
    return group_lists<kUpEach, START>(gl, v, s_face, s_ring, t, x, fl, nb, m, above);
}

// rows of 8 faces for n faces here, 1, 2 or 4 for the whole wave
__device__ __forceinline__ int wave_rows(int n)
{
    return __any(n > 2 * kUpLanes) ? kUpEach : (__any(n > kUpLanes) ? 2 : 1);
}

// A round's start by 8 lanes a vertex, for up to kUpList faces: its lists, then
// its quadric, the faces of a row of 8 a lane each and their sums, a component
// a lane, in ascending order.  (A thread a vertex sorted its lists in place in
// memory, a chain of dependent reads and writes: 220 us on 262,000 vertices,
// mean of three rounds, now 62.)
__global__ __launch_bounds__(kBlock) void k_qem_vertex(const double *__restrict__ P,
                                                       const int32_t *__restrict__ F, int64_t nv,
                                                       const uint32_t *__restrict__ fcnt,
                                                       int32_t *fl, int32_t *__restrict__ fdeg,
                                                       int32_t *__restrict__ nb,
                                                       int32_t *__restrict__ ndeg,
                                                       uint32_t *__restrict__ nlarge,
                                                       double *__restrict__ Q,
                                                       uint8_t *__restrict__ prot,
                                                       int32_t *__restrict__ absorbed,
                                                       uint32_t *__restrict__ flags)
{
    constexpr int kGroups = kBlock / kUpLanes;
    __shared__ int4 s_face[kGroups][kUpList / 4], s_ring[kGroups][kUpList / 2];
    __shared__ double s_k[kGroups][kUpLanes][10];
    const int gl = (int)threadIdx.x % kUpLanes, grp = (int)threadIdx.x / kUpLanes;
    const int64_t v = (int64_t)blockIdx.x * kGroups + grp;
    if (v >= nv) return;
    const int n = fcnt[v] < (uint32_t)kQemFaces ? (int)fcnt[v] : kQemFaces;
    if (gl == 0) absorbed[v] = -1;
    if (n > kUpList) {
        if (gl == 0)
            vertex_serial(P, F, v, n, fl, fdeg, nb, ndeg, nlarge, Q, prot, flags);
        return;
    }
    int32_t *faces = reinterpret_cast<int32_t *>(s_face[grp]);
    int32_t *ring = reinterpret_cast<int32_t *>(s_ring[grp]);
    const int rows = wave_rows(n);
    int32_t t[kUpEach], x[kUpEach][2];
#pragma unroll
    for (int q = 0; q < kUpEach; ++q) {
        const int i = q * kUpLanes + gl;
        t[q] = i < n ? fl[v * kQemFaces + i] : kGone;
    }
#pragma unroll
    for (int q = 0; q < kUpEach; ++q) {
        if (q >= rows) break;
        const int i = q * kUpLanes + gl;
        const int64_t f = i < n ? t[q] : 0;
        const int32_t c0 = F[3 * f], c1 = F[3 * f + 1], c2 = F[3 * f + 2];
        const bool a = c0 == (int32_t)v, b = c1 == (int32_t)v;
        x[q][0] = i < n ? (a ? c1 : c0) : kGone;
        x[q][1] = i < n ? (a || b ? c2 : c1) : kGone;
        faces[i] = t[q];
        ring[2 * i] = x[q][0];
        ring[2 * i + 1] = x[q][1];
    }
    wave_lds_fence();
    uint32_t m, above;
    const bool odd = wave_lists<true>(rows, gl, v, s_face[grp], s_ring[grp], t, x,
                                       fl, nb, m, above);
    const uint32_t both = group_sum<kUpLanes>(m | (above << 16));
    const uint32_t odds = group_ballot<kUpLanes>(odd);
    if (gl == 0) {
        fdeg[v] = n;
        ndeg[v] = (int32_t)(both & 0xffffu);
        nlarge[v] = both >> 16;
        prot[v] = odds ? 1 : 0;
    }
    double acc[2] = {0.0, 0.0};
    for (int r = 0; r < n; r += kUpLanes) {
        if (r + gl < n) {
            const int64_t f = faces[r + gl];
            double pa[3], pb[3], pc[3];
            load3(P, F[3 * f], pa);
            load3(P, F[3 * f + 1], pb);
            load3(P, F[3 * f + 2], pc);
            plane_quadric(pa, pb, pc, s_k[grp][gl]);
        }
        wave_lds_fence();
        for (int k = 0; k < kUpLanes && r + k < n; ++k) {
            acc[0] = acc[0] + s_k[grp][k][gl];
            if (gl < 2) acc[1] = acc[1] + s_k[grp][k][8 + gl];
        }
        wave_lds_fence();
    }
    Q[10 * v + gl] = acc[0];
    if (gl < 2) Q[10 * v + 8 + gl] = acc[1];
}

// Between a round's steps by 8 lanes a vertex, for lists of at most kUpList
// faces together (a thread a vertex, its lists merged and its ring sorted in
// place in memory: 66 us a step on 262,000 vertices, now 38).  Every vertex's
// first edge number within its block, and the block's number of edges, follow.
__global__ __launch_bounds__(kBlock) void k_qem_vertex_update(
    const int32_t *__restrict__ F, int64_t nv, const uint8_t *__restrict__ dirty,
    const int32_t *__restrict__ remap, int32_t *__restrict__ absorbed, int32_t *fl, int32_t *fdeg,
    int32_t *__restrict__ nb, int32_t *__restrict__ ndeg, uint32_t *__restrict__ nlarge,
    uint32_t *__restrict__ eoff, uint32_t *__restrict__ ebase, QemState *__restrict__ st)
{
    if (st->loop.done) return;
    constexpr int kGroups = kBlock / kUpLanes, kEach = kUpEach;
    __shared__ uint16_t list[kBlock];
    __shared__ uint32_t count, s_above[kBlock];
    __shared__ int4 s_face[kGroups][kUpList / 4], s_ring[kGroups][kUpList / 2];
    const int64_t v0 = (int64_t)blockIdx.x * kBlock, mine = v0 + threadIdx.x;
    const bool in = mine < nv, gone = in && remap[mine] >= 0, work = in && !gone && dirty[mine];
    const uint32_t n_work = block_list(work, list, &count);
    const int gl = (int)threadIdx.x % kUpLanes, grp = (int)threadIdx.x / kUpLanes;
    for (uint32_t j = (uint32_t)grp; j < n_work; j += kGroups) {
        const int64_t v = v0 + list[j];
        const int32_t w = absorbed[v];
        const int n0 = fdeg[v], m0 = w >= 0 ? fdeg[w] : 0, tot = n0 + m0;
        if (tot > kUpList) {
            if (gl == 0) {
                const uint32_t above = vertex_update_serial(F, v, absorbed, fl, fdeg, nb, ndeg,
                                                            &st->flags);
                nlarge[v] = above;
                s_above[list[j]] = above;
            }
            continue;
        }
        int32_t t[kEach], c[kEach][3];
#pragma unroll
        for (int q = 0; q < kEach; ++q) {
            const int i = q * kUpLanes + gl;
            t[q] = i < n0 ? fl[v * kQemFaces + i]
                          : (i < tot ? fl[(int64_t)w * kQemFaces + i - n0] : kGone);
        }
#pragma unroll
        for (int q = 0; q < kEach; ++q) {
            const int64_t f = q * kUpLanes + gl < tot ? t[q] : 0;
            for (int k = 0; k < 3; ++k) c[q][k] = F[3 * f + k];
        }
        // the lane's faces and ring entries stay in registers; all of them, in
        // whole rows of 8 faces, go to LDS to be compared with four at a time
        int32_t *faces = reinterpret_cast<int32_t *>(s_face[grp]);
        int32_t *ring = reinterpret_cast<int32_t *>(s_ring[grp]);
        const int rows = wave_rows(tot);
        int32_t x[kEach][2];
        uint32_t n = 0;
#pragma unroll
        for (int q = 0; q < kEach; ++q) {
            if (q >= rows) break;
            const int i = q * kUpLanes + gl;
            const bool live = i < tot && c[q][0] >= 0;
            const bool a = c[q][0] == (int32_t)v, b = c[q][1] == (int32_t)v;
            if (!live) t[q] = kGone;
            x[q][0] = live ? (a ? c[q][1] : c[q][0]) : kGone;
            x[q][1] = live ? (a || b ? c[q][2] : c[q][1]) : kGone;
            n += live ? 1u : 0u;
            faces[i] = t[q];
            ring[2 * i] = x[q][0];
            ring[2 * i + 1] = x[q][1];
        }
        n = group_sum<kUpLanes>(n);
        wave_lds_fence();
        uint32_t m, above;
        wave_lists<false>(rows, gl, v, s_face[grp], s_ring[grp], t, x,
                           fl, nb, m, above);
        const uint32_t both = group_sum<kUpLanes>(m | (above << 16));
        if (gl == 0) {
            fdeg[v] = (int32_t)n;
            ndeg[v] = (int32_t)(both & 0xffffu);
            nlarge[v] = both >> 16;
            s_above[list[j]] = both >> 16;
            if (w >= 0) {
                absorbed[v] = -1;
                fdeg[w] = 0;
                ndeg[w] = 0;
            }
        }
        wave_lds_fence();
    }
    __syncthreads();
    if (gone) nlarge[mine] = 0;       // contracted into another: no edges
    const uint32_t own = !in || gone ? 0u : work ? s_above[threadIdx.x] : nlarge[mine];
    const uint32_t off = block_offsets(own, ebase);
    if (in) eoff[mine] = off;
}

// The offsets of k_qem_vertex_update at a round's start.
__global__ __launch_bounds__(kBlock) void k_qem_first_edge(const uint32_t *__restrict__ nlarge,
                                                           int64_t nv, uint32_t *__restrict__ eoff,
                                                           uint32_t *__restrict__ ebase,
                                                           const QemState *__restrict__ st)
{
    if (st->loop.done) return;
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const uint32_t off = block_offsets(v < nv ? nlarge[v] : 0u, ebase);
    if (v < nv) eoff[v] = off;
}

// The blocks' first edge numbers (in place), and the step's number of edges.
// One block.
constexpr int kOffBlock = 1024;

__global__ __launch_bounds__(kOffBlock) void k_qem_offsets(uint32_t *__restrict__ ebase, int64_t nb,
                                                           QemState *__restrict__ st)
{
    if (st->loop.done) return;
    __shared__ uint32_t part[kOffBlock / 64];
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    uint32_t carry = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += 4 * kOffBlock) {
        const int64_t i0 = c0 + 4 * (int64_t)threadIdx.x;
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = i0 + k < nb ? ebase[i0 + k] : 0u;
            sum += v[k];
        }
        uint32_t x = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) part[w] = x;
        __syncthreads();
        uint32_t at = carry + x - sum;
        for (int k = 0; k < kOffBlock / 64; ++k) {
            if (k < w) at += part[k];
            carry += part[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < nb) ebase[i0 + k] = at;
            at += v[k];
        }
    }
    if (threadIdx.x == 0) {
        st->n_old = st->loop.n_edges;
        st->loop.n_edges = carry;
    }
}

// Does face (c0, c1, c2) with corners p flip when its corner at u or v moves to x?
__device__ __forceinline__ bool face_flips(const int32_t c[3], const double p[3][3], int32_t u,
                                           int32_t v, const double x[3])
{
    const bool hu = c[0] == u || c[1] == u || c[2] == u;
    const bool hv = c[0] == v || c[1] == v || c[2] == v;
    if (hu && hv) return false;          // drops out
    double n0[3], n1[3], a[3], b[3], d[3];
    face_normal(p[0], p[1], p[2], n0);
    // selects, not a pointer, so the corners stay in registers
    const bool m0 = c[0] == u || c[0] == v;
    const bool m1 = !m0 && (c[1] == u || c[1] == v);
    const bool m2 = !m0 && !m1;
    for (int q = 0; q < 3; ++q) {
        a[q] = m0 ? x[q] : p[0][q];
        b[q] = m1 ? x[q] : p[1][q];
        d[q] = m2 ? x[q] : p[2][q];
    }
    face_normal(a, b, d, n1);
    return dot3(n0, n0) > 0.0 && !(dot3(n0, n1) > 0.0);
}

// Candidate test of the edge (u, v) by G lanes: true (in all of them) with the
// contraction point x and the float32 cost bits when the edge may contract
// (readings of the header comment).  The lanes share the faces and neighbours
// of the ends; the point is every lane's.  A lane's first kAhead faces (12 of
// both ends together, more than most edges have) are read, corners and all,
// before the tests: the chain is then lists - faces - corners.
template <int G>
__device__ bool edge_candidate(const double *__restrict__ P, const int32_t *__restrict__ F,
                               const int32_t *__restrict__ fl, const int32_t *__restrict__ fdeg,
                               const int32_t *__restrict__ nb, const int32_t *__restrict__ ndeg,
                               const double *__restrict__ Q, const uint8_t *__restrict__ prot,
                               int32_t u, int32_t v, int gl, double x[3], uint32_t *cbits)
{
    constexpr int kAhead = 3;
    const int nu = ndeg[u], nvv = ndeg[v], fu = fdeg[u], fv = fdeg[v];
    const int32_t *bu = nb + (int64_t)u * kQemNbrs, *bv = nb + (int64_t)v * kQemNbrs;
    const int32_t *lu = fl + (int64_t)u * kQemFaces, *lv = fl + (int64_t)v * kQemFaces;
    if (prot[u] || prot[v]) return false;
    int32_t t[kAhead], c[kAhead][3];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
        const int i = k * G + gl;
        t[k] = i < fu ? lu[i] : (i < fu + fv ? lv[i - fu] : -1);
    }
    const int32_t a0 = gl < nu ? bu[gl] : -1, a1 = G + gl < nu ? bu[G + gl] : -1;
    const int32_t b0 = gl < nvv ? bv[gl] : -2, b1 = G + gl < nvv ? bv[G + gl] : -2;
    double Qe[10], pu[3], pv[3];
#pragma unroll
    for (int q = 0; q < 10; ++q) Qe[q] = Q[10 * (int64_t)u + q] + Q[10 * (int64_t)v + q];
    load3(P, u, pu);
    load3(P, v, pv);
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
        for (int q = 0; q < 3; ++q) c[k][q] = t[k] >= 0 ? F[3 * (int64_t)t[k] + q] : 0;
    // link condition: exactly two common neighbours (each list holds a
    // vertex once)
    bool h0 = false, h1 = false;
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const int32_t y0 = __shfl(b0, q, G), y1 = __shfl(b1, q, G);
        h0 |= y0 == a0 || y1 == a0;
        h1 |= y0 == a1 || y1 == a1;
    }
    for (int j = 2 * G; j < nvv; ++j) {
        const int32_t y = bv[j];
        h0 |= y == a0;
        h1 |= y == a1;
    }
    int common = __popc(group_ballot<G>(h0)) + __popc(group_ballot<G>(h1));
    for (int i = 2 * G; i < nu; i += G) {
        const int32_t a = i + gl < nu ? bu[i + gl] : -1;
        bool hit = false;
        for (int j = 0; j < nvv; ++j) hit |= bv[j] == a;
        common += __popc(group_ballot<G>(hit));
    }
    if (common != 2) return false;
    // faces of u with v: exactly two
    int fc = 0;
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
        fc += __popc(group_ballot<G>(k * G + gl < fu && (c[k][0] == v || c[k][1] == v || c[k][2] == v)));
    for (int i = kAhead * G; i < fu; i += G)
        fc += __popc(group_ballot<G>(i + gl < fu && face_has(F, lu[i + gl], v)));
    if (fc != 2) return false;
    double p[kAhead][3][3];
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
        for (int q = 0; q < 3; ++q) load3(P, c[k][q], p[k][q]);
    const double cost = placement(Qe, pu, pv, x);
    // no face of u or v (other than the two on the edge) may flip
    bool flips = false;
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
        if (k * G < fu + fv) flips |= t[k] >= 0 && face_flips(c[k], p[k], u, v, x);
    if (group_ballot<G>(flips)) return false;
    for (int i = kAhead * G; i < fu + fv; i += G) {
        if (i + gl < fu + fv) {
            const int64_t f = i + gl < fu ? lu[i + gl] : lv[i + gl - fu];
            const int32_t d[3] = {F[3 * f], F[3 * f + 1], F[3 * f + 2]};
            double e[3][3];
            for (int q = 0; q < 3; ++q) load3(P, d[q], e[q]);
            flips = face_flips(d, e, u, v, x);
        }
        if (group_ballot<G>(flips)) return false;
    }
    // cost clamped at 0 (a NaN stays) and rounded to float32; -0 and +0
    // share one key
    const double cl = 0.0 > cost ? 0.0 : cost;
    float c32 = (float)cl;
    if (c32 == 0.0f) c32 = 0.0f;
    *cbits = __float_as_uint(c32);
    return true;
}

// The step's edges, by the first `carry_blocks` blocks and the rest.
//
// The rest, per vertex u with a dirty end role (every vertex at a round's
// start, else the dirty ones): every edge (u, v > u) in ascending v, numbered
// from u's first edge, is marked for k_qem_eval (cand = 2); and what the
// contraction marks of a vertex is cleared.
//
// The first, one thread per edge of the previous step whose lower end u is
// clean: u's edges are the same, in the same order, so the edge keeps its
// place behind u's first.  With v clean too its result is unchanged (its
// ends, their faces, neighbours, positions and quadrics are all as before)
// and only the key's low word becomes pi of the new number; with v dirty it
// is marked for k_qem_eval.
__global__ __launch_bounds__(kBlock) void k_qem_renumber(QemBuffers b, int64_t nv, int full,
                                                         uint32_t carry_blocks, int nslots)
{
    const QemState *st = reinterpret_cast<const QemState *>(b.sel);
    if (st->loop.done) return;
    if (blockIdx.x >= carry_blocks) {
        const int64_t u = (int64_t)(blockIdx.x - carry_blocks) * kBlock + threadIdx.x;
        if (u >= nv) return;
        b.best[u] = ~0ull;
        b.remap[u] = -1;
        b.dirty_next[u] = 0;
        if (!(full || b.dirty[u])) return;
        const int nu = b.ndeg[u];
        const int32_t *bu = b.nb + u * kQemNbrs;
        uint32_t e = b.eoff[u] + b.ebase[u / kBlock];
        for (int k = 0; k < nu; ++k) {
            const int32_t v = bu[k];
            if (v <= (int32_t)u) continue;
            b.eu[e] = (int32_t)u;
            b.ev[e] = v;
            b.cand[e] = 2;
            ++e;
        }
        return;
    }
    const int64_t eo = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    uint32_t found = 0;
    if (eo < (int64_t)st->n_old) {
        const int32_t u = b.eu_old[eo], v = b.ev_old[eo];
        if (!b.dirty[u]) {
            const uint32_t e = (uint32_t)eo - (b.eoff_old[u] + b.ebase_old[u / kBlock]) +
                               (b.eoff[u] + b.ebase[u / kBlock]);
            b.eu[e] = u;
            b.ev[e] = v;
            if (b.dirty[v]) {
                b.cand[e] = 2;
            } else if (b.cand_old[eo]) {
                for (int q = 0; q < 3; ++q) b.X[3 * (int64_t)e + q] = b.X_old[3 * eo + q];
                b.key[e] = (b.key_old[eo] & 0xffffffff00000000ull) | perm32(e);
                b.cand[e] = 1;
                found = 1;
            } else {
                b.key[e] = kNone;
                b.cand[e] = 0;
            }
        }
    }
    block_add(found, &slot_of(reinterpret_cast<QemSlot *>(b.slots), nslots)->cand);
}

// The edges marked by k_qem_renumber, kEvalLanes lanes each: the candidate
// test, the key (float32 cost bits, pi(e)) or "none", and the point.  A block
// lists the marked ones of its 256 edges first: a thread an edge left the
// lanes of unmarked edges idle and walked a dozen faces one after another,
// each three dependent reads (110 us a step on 682,000 edges and 47 us on
// 111,000, now 87 and 24).
constexpr int kEvalLanes = 4;
// Up to this many edges a block lists 64, so that every group has at most one
// and the launch is one chain long; beyond, 256, and no lane idles.  256 / 64:
// 17 / 13 us at 79,000 edges, 31 / 31 at 146,000, 31 / 39 at 206,000, 87 / 120
// at 682,000.
constexpr int64_t kEvalMany = 1 << 17;

template <int EDGES>          // of a block
__global__ __launch_bounds__(kBlock) void k_qem_eval(QemBuffers b, int nslots)
{
    static_assert(EDGES <= kBlock && EDGES * kEvalLanes >= kBlock, "every group an edge or more");
    const QemState *st = reinterpret_cast<const QemState *>(b.sel);
    if (st->loop.done) return;
    __shared__ uint16_t list[kBlock];
    __shared__ uint32_t count;
    const int64_t e0 = (int64_t)blockIdx.x * EDGES, n = st->loop.n_edges;
    if (e0 >= n) return;
    const uint32_t marked = block_list((int)threadIdx.x < EDGES && e0 + threadIdx.x < n &&
                                           b.cand[e0 + threadIdx.x] == 2, list, &count);
    const int gl = (int)threadIdx.x % kEvalLanes;
    uint32_t found = 0;
    for (uint32_t j = threadIdx.x / kEvalLanes; j < marked; j += kBlock / kEvalLanes) {
        const int64_t e = e0 + list[j];
        double x[3];
        uint32_t cbits = 0;
        const bool c = edge_candidate<kEvalLanes>(b.P, b.F, b.fl, b.fdeg, b.nb, b.ndeg, b.Q, b.prot,
                                                  b.eu[e], b.ev[e], gl, x, &cbits);
        if (gl == 0) {
            if (c) {
                for (int q = 0; q < 3; ++q) b.X[3 * e + q] = x[q];
                ++found;
            }
            b.key[e] = c ? ((uint64_t)cbits << 32) | perm32((uint32_t)e) : kNone;
            b.cand[e] = c ? 1 : 0;
        }
    }
    block_add(found, &slot_of(reinterpret_cast<QemSlot *>(b.slots), nslots)->cand);
}

// Radix select, one digit of `width` bits a pass from the top.  The last block
// to finish a pass picks the digit that holds the rank-th key and clears the
// counts for the next: a launch of its own for the pick took as long as the
// pass.  Equal digits of a wave's keys are counted with one addition for
// the two commonest, the rest one by one: most costs share their exponents
// (25 and 53 us for the first two passes over 682,000 keys, now 10 and 9.5).
// QEM: the need smallest keys are eligible, every candidate's if need is at
// least their number (decided in the first pass), and a digit all of whose
// keys are among them ends the select: prefix, filled up with ones, separates
// the same keys.
constexpr int kSelBlock = 1024, kSelBits = 11;

template <bool QEM>
__global__ __launch_bounds__(kSelBlock) void k_select_pass(const uint64_t *__restrict__ key,
                                                           int64_t n_keys, SelState *st, int shift,
                                                           int width, int first,
                                                           const QemSlot *__restrict__ slots,
                                                           int nslots, uint32_t *hist)
{
    if (QEM && reinterpret_cast<const QemState *>(st)->loop.done) return;
    if (st->done) return;
    __shared__ uint32_t h[1 << kSelBits];
    __shared__ uint32_t last, s_cand, wsum[kSelBlock / 64];
    const int lane = (int)(threadIdx.x & 63), bins = 1 << width;
    const int64_t n = QEM ? (int64_t)reinterpret_cast<const QemState *>(st)->loop.n_edges : n_keys;
    const unsigned long long rank = st->rank;
    for (int i = threadIdx.x; i < bins; i += kSelBlock) h[i] = 0;
    if (QEM && first && threadIdx.x < 64) {
        uint32_t c = lane < nslots ? slots[lane].cand : 0u;
        for (int o = 32; o > 0; o >>= 1) c += (uint32_t)__shfl_xor((int)c, o, 64);
        if (lane == 0) s_cand = c;
    }
    __syncthreads();
    const bool all = QEM && first && rank >= (unsigned long long)s_cand;
    const uint64_t prefix = st->prefix, mask = st->mask;
    const int64_t stride = (int64_t)gridDim.x * kSelBlock;
    for (int64_t i0 = (int64_t)blockIdx.x * kSelBlock; i0 < n && !all; i0 += stride) {
        const int64_t i = i0 + threadIdx.x;
        const uint64_t k = i < n ? key[i] : kNone;
        const bool in = i < n && (!QEM || k != kNone) && (k & mask) == prefix;
        const uint32_t d = (uint32_t)(k >> shift) & (uint32_t)(bins - 1);
        uint64_t todo = __ballot(in);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (!todo) break;
            const int f = __builtin_ctzll(todo);
            const uint32_t df = (uint32_t)__builtin_amdgcn_readlane((int)d, f);
            const uint64_t same = __ballot(in && d == df) & todo;
            if (lane == f) atomicAdd(&h[df], (uint32_t)__popcll(same));
            todo &= ~same;
        }
        if ((todo >> lane) & 1ull) atomicAdd(&h[d], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < bins; i += kSelBlock)
        if (h[i]) __hip_atomic_fetch_add(&hist[i], h[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // each wave's additions are done and the barrier orders them before thread
    // 0's ticket, whose release hands them on; the last block's acquire takes all
    // of them over.  A release by one thread a block writes back the XCD's L2
    // once (by every wave it made a pass 70 us; see sel_grid).
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        last = __hip_atomic_fetch_add(&st->ticket, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT) ==
               gridDim.x - 1;
        if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    if (!last) return;
    // bins 2 t and 2 t + 1 of thread t
    uint32_t c[2], sum = 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = 2 * (int)threadIdx.x + q;
        c[q] = i < bins ? __hip_atomic_load(&hist[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        sum += c[q];
    }
    uint32_t x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[threadIdx.x >> 6] = x;
    __syncthreads();
    uint32_t before = x - sum, tot = 0;
    for (int k = 0; k < kSelBlock / 64; ++k) {
        if (k < (int)(threadIdx.x >> 6)) before += wsum[k];
        tot += wsum[k];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = 2 * (int)threadIdx.x + q;
        if (i >= bins) break;
        hist[i] = 0;
        // the first digit whose inclusive count reaches the rank
        if (!all && before < rank && (before + c[q] >= rank)) {
            const unsigned long long m = mask | ((unsigned long long)(bins - 1) << shift);
            unsigned long long p = prefix | ((unsigned long long)i << shift);
            if (QEM && before + c[q] == rank) {
                p |= ~m;
                st->done = 1;
            }
            st->prefix = p;
            st->mask = m;
            st->rank = rank - before;
            if (shift == 0) st->done = 1;
        }
        before += c[q];
    }
    if (threadIdx.x == 0) {
        st->ticket = 0;
        if (all) {
            st->prefix = kNone;           // every candidate
            st->done = 1;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_qem_best(QemBuffers b)
{
    const QemState *st = reinterpret_cast<const QemState *>(b.sel);
    if (st->loop.done) return;
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= (int64_t)st->loop.n_edges) return;
    const uint64_t k = b.key[e];
    if (k == kNone || k > st->sel.prefix) return;
    atomicMin(&b.best[b.eu[e]], (unsigned long long)k);
    atomicMin(&b.best[b.ev[e]], (unsigned long long)k);
}

// Contracts the eligible edges that no eligible edge at a vertex of their two
// closed one-rings undercuts.  A block lists those of its edges that are the
// least at both ends, and 8 lanes take one: its neighbours' minima, its faces
// and marks side by side (a thread an edge: 82 us a step on 682,000 edges and
// 20 us on 111,000, now 17 and 9).
__global__ __launch_bounds__(kBlock) void k_qem_choose(QemBuffers b, int nslots)
{
    const QemState *st = reinterpret_cast<const QemState *>(b.sel);
    if (st->loop.done) return;
    constexpr int G = 8;
    __shared__ uint16_t list[kBlock];
    __shared__ uint32_t count;
    const int64_t e0 = (int64_t)blockIdx.x * kBlock, n = st->loop.n_edges;
    if (e0 >= n) return;
    bool ok = false;
    if (e0 + threadIdx.x < n) {
        const uint64_t k = b.key[e0 + threadIdx.x];
        if (k != kNone && k <= st->sel.prefix)
            ok = b.best[b.eu[e0 + threadIdx.x]] >= k && b.best[b.ev[e0 + threadIdx.x]] >= k;
    }
    const uint32_t some = block_list(ok, list, &count);
    const int gl = (int)threadIdx.x % G;
    uint32_t sums = 0;        // contracted, dropped << 16
    for (uint32_t j = threadIdx.x / G; j < some; j += kBlock / G) {
        const int64_t e = e0 + list[j];
        const uint64_t k = b.key[e];
        const int32_t u = b.eu[e], v = b.ev[e];
        const int nu = b.ndeg[u], nn = nu + b.ndeg[v];
        bool least = true;
        for (int i = gl; i < nn; i += G) {
            const int32_t q = i < nu ? b.nb[(int64_t)u * kQemNbrs + i]
                                     : b.nb[(int64_t)v * kQemNbrs + i - nu];
            least = least && b.best[q] >= k;
        }
        if (group_ballot<G>(!least)) continue;
        // no end of an edge chosen in this step is an end or a neighbour of
        // an end of another: each updates its own u in place
        for (int i = gl; i < 10; i += G)
            b.Q[10 * (int64_t)u + i] = b.Q[10 * (int64_t)u + i] + b.Q[10 * (int64_t)v + i];
        if (gl < 3) b.P[3 * (int64_t)u + gl] = b.X[3 * e + gl];
        if (gl == 0) {
            b.remap[v] = u;
            b.absorbed[u] = v;
            b.dirty_next[u] = 1;
            b.dirty_next[v] = 1;
            sums += 1;
        }
        // v's faces: the two on the edge degenerate and are dropped, the
        // others take u for v (no face has ends of two chosen edges)
        const int fv = b.fdeg[v];
        for (int i = gl; i < fv; i += G) {
            const int64_t t = b.fl[(int64_t)v * kQemFaces + i];
            const int32_t c0 = b.F[3 * t], c1 = b.F[3 * t + 1], c2 = b.F[3 * t + 2];
            if (c0 == u || c1 == u || c2 == u) {
                b.F[3 * t] = -1;
                sums += 1u << 16;
            } else {
                b.F[3 * t + (c0 == v ? 0 : (c1 == v ? 1 : 2))] = u;
            }
        }
        // the closed one-rings change: their vertices are evaluated anew
        // in the next step (two rings may share a vertex: equal stores)
        for (int i = gl; i < nn; i += G)
            b.dirty_next[i < nu ? b.nb[(int64_t)u * kQemNbrs + i]
                                : b.nb[(int64_t)v * kQemNbrs + i - nu]] = 1;
    }
    QemSlot *slot = slot_of(reinterpret_cast<QemSlot *>(b.slots), nslots);
    block_add(sums & 0xffffu, &slot->chosen);
    block_add(sums >> 16, &slot->killed);
}

// A round's start.
__global__ void k_qem_round(QemBuffers b, int64_t nf, int64_t target)
{
    QemState *st = reinterpret_cast<QemState *>(b.sel);
    st->loop.nf = nf;
    st->loop.target = target;
    st->loop.done = 0;
    st->sel.prefix = 0;
    st->sel.mask = 0;
    st->sel.rank = (unsigned long long)((nf - target + 1) / 2);
    st->sel.done = 0;
}

// A step's end: its counters, whether it was the round's last, and the next
// one's select.  One wave.
__global__ __launch_bounds__(64) void k_qem_end(QemBuffers b, int nslots)
{
    QemState *st = reinterpret_cast<QemState *>(b.sel);
    if (st->loop.done) return;
    QemSlot *slots = reinterpret_cast<QemSlot *>(b.slots);
    const int lane = (int)threadIdx.x;
    uint32_t cand = 0, chosen = 0, killed = 0;
    if (lane < nslots) {
        cand = slots[lane].cand;
        chosen = slots[lane].chosen;
        killed = slots[lane].killed;
        slots[lane].cand = slots[lane].chosen = slots[lane].killed = 0;
    }
    cand = group_sum<64>(cand);
    chosen = group_sum<64>(chosen);
    killed = group_sum<64>(killed);
    if (lane != 0) return;
    QemLoop &l = st->loop;
    if (st->flags) {
        l.error = st->flags & 1u ? kQemManyFaces : kQemManyNbrs;
    } else if (cand != 0) {
        ++l.steps;
        l.removed = killed;
        // a contraction drops exactly the two faces on its edge
        if (chosen == 0) l.error = kQemStuck;
        else if (killed != 2 * chosen) l.error = kQemMismatch;
        l.nf -= killed;
    }
    l.done = l.error || cand == 0 || l.nf <= l.target ? 1u : 0u;
    st->sel.prefix = 0;
    st->sel.mask = 0;
    st->sel.rank = l.nf > l.target ? (unsigned long long)((l.nf - l.target + 1) / 2) : 0ull;
    st->sel.done = 0;
}

__global__ __launch_bounds__(kBlock) void k_qem_live(const int32_t *__restrict__ F, int64_t nt,
                                                     QemSlot *__restrict__ slots, int nslots)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    block_add(t < nt && F[3 * t] >= 0 ? 1u : 0u, &slot_of(slots, nslots)->killed);
}

// the live faces of k_qem_live; the state and counters start from 0
__global__ __launch_bounds__(64) void k_qem_start(QemBuffers b, int nslots)
{
    QemSlot *slots = reinterpret_cast<QemSlot *>(b.slots);
    uint32_t live = 0;
    if ((int)threadIdx.x < nslots) {
        live = slots[threadIdx.x].killed;
        slots[threadIdx.x].killed = 0;
    }
    live = group_sum<64>(live);
    if (threadIdx.x == 0) reinterpret_cast<QemState *>(b.sel)->loop.nf = live;
}

__global__ __launch_bounds__(kBlock) void k_qem_used(const int32_t *__restrict__ F, int64_t nt,
                                                     uint32_t *__restrict__ used,
                                                     uint32_t *__restrict__ keep)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= nt) return;
    const bool live = F[3 * t] >= 0;
    keep[t] = live ? 1u : 0u;
    if (live)
        for (int k = 0; k < 3; ++k) used[F[3 * t + k]] = 1u;
}

__global__ __launch_bounds__(kBlock) void k_qem_emit(const double *__restrict__ P, int64_t nv,
                                                     const uint32_t *__restrict__ used,
                                                     const uint32_t *__restrict__ newid,
                                                     const int32_t *__restrict__ F, int64_t nt,
                                                     const uint32_t *__restrict__ keep,
                                                     const uint32_t *__restrict__ tpos,
                                                     float *__restrict__ out_verts,
                                                     int32_t *__restrict__ out_tris)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < nv && used[i])
        for (int k = 0; k < 3; ++k) out_verts[3 * (int64_t)newid[i] + k] = (float)P[3 * i + k];
    if (i < nt && keep[i])
        for (int k = 0; k < 3; ++k)
            out_tris[3 * (int64_t)tpos[i] + k] = (int32_t)newid[F[3 * i + k]];
}

__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t *p, int64_t n, uint32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_sel_init(SelState *st, unsigned long long rank, uint32_t *hist)
{
    if (threadIdx.x == 0) {
        st->prefix = 0;
        st->mask = 0;
        st->rank = rank;
        st->done = 0;
        st->ticket = 0;
    }
    if (threadIdx.x < 256) hist[threadIdx.x] = 0;
}

// The state, then the counts of a digit, then the counters.  Meshes of fewer
// than 2^16 edge places take 8-bit digits and one line of counters.
bool wide_select(int64_t ne_cap) { return ne_cap >= (1 << 16); }
int sel_bins(int64_t ne_cap) { return wide_select(ne_cap) ? 1 << kSelBits : 256; }
constexpr int kQemSlots = 64;
int qem_slots(int64_t ne_cap) { return wide_select(ne_cap) ? kQemSlots : 1; }

// Blocks of a pass.  Each pays for its release (see k_select_pass), which up to
// 2^20 keys costs more than the keys: 256 / 128 / 64 blocks take 173 / 166 / 170
// us a coarse quantile reconstruction (350,200 keys) and 11.18 / 11.05 / 11.04
// ms a decimation (682,000 keys at first); beyond, the keys count: 566 / 613 /
// 711 us a reconstruction of 17.6M voxels.
unsigned sel_grid(int64_t n)
{
    const unsigned g = grid_for(n, kSelBlock), most = n <= (1 << 20) ? 128 : 256;
    return g < 1 ? 1 : (g > most ? most : g);
}

}  // namespace

size_t qem_sel_bytes(int64_t ne_cap)
{
    return sizeof(QemState) + sizeof(uint32_t) * sel_bins(ne_cap) +
           sizeof(QemSlot) * qem_slots(ne_cap);
}
size_t qem_sel_slots(int64_t ne_cap) { return sizeof(QemState) + sizeof(uint32_t) * sel_bins(ne_cap); }
size_t qem_sel_loop() { return offsetof(QemState, loop); }
size_t radix_select_state_bytes() { return sizeof(SelState) + 256 * sizeof(uint32_t); }

hipError_t qem_init_launch(const float *verts, int64_t nv, const int32_t *tris, int64_t nt,
                           double *P, int32_t *F, hipStream_t s)
{
    const int64_t n = nv > nt ? nv : nt;
    hipLaunchKernelGGL(k_qem_init, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, verts, nv, tris,
                       nt, P, F);
    return hipGetLastError();
}

hipError_t qem_live_launch(const QemBuffers &b, int64_t nt, hipStream_t s)
{
    const int ns = qem_slots(3 * nt);
    hipLaunchKernelGGL(k_qem_live, dim3(grid_for(nt, kBlock)), dim3(kBlock), 0, s, b.F, nt,
                       reinterpret_cast<QemSlot *>(b.slots), ns);
    hipLaunchKernelGGL(k_qem_start, dim3(1), dim3(64), 0, s, b, ns);
    return hipGetLastError();
}

hipError_t qem_round_launch(const QemBuffers &b, int64_t nv, int64_t nt, int64_t nf, int64_t target,
                            hipStream_t s)
{
    QemState *st = reinterpret_cast<QemState *>(b.sel);
    hipLaunchKernelGGL(k_qem_round, dim3(1), dim3(1), 0, s, b, nf, target);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nv, kBlock)), dim3(kBlock), 0, s, b.fcnt, nv, 0u);
    hipLaunchKernelGGL(k_qem_fill_faces, dim3(grid_for(nt, kBlock)), dim3(kBlock), 0, s, b.F, nt,
                       b.fcnt, b.fl, &st->flags);
    hipLaunchKernelGGL(k_qem_vertex, dim3(grid_for(nv, kBlock / kUpLanes)), dim3(kBlock), 0, s, b.P,
                       b.F, nv, b.fcnt, b.fl, b.fdeg, b.nb, b.ndeg, b.nlarge, b.Q, b.prot,
                       b.absorbed, &st->flags);
    return hipGetLastError();
}

// A vertex with more faces or neighbours than its lists hold is reported by
// k_qem_end: until then the step runs on lists cut to their length.  Every entry
// is a face or vertex of the mesh and the edges are among the faces' (at most
// 3 nt), so all indices stay in range, and the caller discards the result.
hipError_t qem_step_launch(const QemBuffers &b, int64_t nv, int64_t nt, int64_t max_edges,
                           int round_start, hipStream_t s)
{
    QemState *st = reinterpret_cast<QemState *>(b.sel);
    const int64_t cap = 3 * nt;
    const int ns = qem_slots(cap);
    const unsigned gv = grid_for(nv, kBlock), ge = grid_for(max_edges > 0 ? max_edges : 1, kBlock);
    if (round_start)
        hipLaunchKernelGGL(k_qem_first_edge, dim3(gv), dim3(kBlock), 0, s, b.nlarge, nv, b.eoff,
                           b.ebase, st);
    else
        hipLaunchKernelGGL(k_qem_vertex_update, dim3(gv), dim3(kBlock), 0, s, b.F, nv, b.dirty,
                           b.remap, b.absorbed, b.fl, b.fdeg, b.nb, b.ndeg, b.nlarge, b.eoff,
                           b.ebase, st);
    hipLaunchKernelGGL(k_qem_offsets, dim3(1), dim3(kOffBlock), 0, s, b.ebase, (int64_t)gv, st);
    const unsigned gc = round_start ? 0u : ge;
    hipLaunchKernelGGL(k_qem_renumber, dim3(gc + gv), dim3(kBlock), 0, s, b, nv, round_start, gc, ns);
    if (max_edges > kEvalMany)
        hipLaunchKernelGGL(k_qem_eval<256>, dim3(ge), dim3(kBlock), 0, s, b, ns);
    else
        hipLaunchKernelGGL(k_qem_eval<64>, dim3(grid_for(max_edges > 0 ? max_edges : 1, 64)),
                           dim3(kBlock), 0, s, b, ns);
    uint32_t *hist = reinterpret_cast<uint32_t *>(b.sel + sizeof(QemState));
    const QemSlot *slots = reinterpret_cast<const QemSlot *>(b.slots);
    // 32 bits of cost, then 32 of pi(edge)
    const int bits = wide_select(cap) ? kSelBits : 8;
    for (int word = 1; word >= 0; --word)
        for (int top = 32; top > 0; top -= bits) {
            const int width = top < bits ? top : bits;
            hipLaunchKernelGGL(k_select_pass<true>, dim3(sel_grid(max_edges)), dim3(kSelBlock), 0, s,
                               b.key, (int64_t)0, &st->sel, 32 * word + top - width, width,
                               word == 1 && top == 32 ? 1 : 0, slots, ns, hist);
        }
    hipLaunchKernelGGL(k_qem_best, dim3(ge), dim3(kBlock), 0, s, b);
    hipLaunchKernelGGL(k_qem_choose, dim3(ge), dim3(kBlock), 0, s, b, ns);
    hipLaunchKernelGGL(k_qem_end, dim3(1), dim3(64), 0, s, b, ns);
    return hipGetLastError();
}

hipError_t radix_select_u64_launch(const uint64_t *keys, int64_t n, uint64_t rank, int bits,
                                   char *state, hipStream_t s)
{
    SelState *st = reinterpret_cast<SelState *>(state);
    uint32_t *hist = reinterpret_cast<uint32_t *>(state + sizeof(SelState));
    hipLaunchKernelGGL(k_sel_init, dim3(1), dim3(256), 0, s, st, (unsigned long long)rank, hist);
    for (int shift = (bits - 1) / 8 * 8; shift >= 0; shift -= 8)
        hipLaunchKernelGGL(k_select_pass<false>, dim3(sel_grid(n)), dim3(kSelBlock), 0, s, keys, n,
                           st, shift, 8, 0, (const QemSlot *)nullptr, 0, hist);
    return hipGetLastError();
}

const uint64_t *radix_select_value(const char *state)
{
    return reinterpret_cast<const uint64_t *>(state);   // SelState::prefix
}

hipError_t qem_used_launch(const int32_t *F, int64_t nt, uint32_t *used, uint32_t *keep,
                           hipStream_t s)
{
    hipLaunchKernelGGL(k_qem_used, dim3(grid_for(nt, kBlock)), dim3(kBlock), 0, s, F, nt, used,
                       keep);
    return hipGetLastError();
}

hipError_t qem_emit_launch(const double *P, int64_t nv, const uint32_t *used,
                           const uint32_t *newid, const int32_t *F, int64_t nt,
                           const uint32_t *keep, const uint32_t *tpos, float *out_verts,
                           int32_t *out_tris, hipStream_t s)
{
    const int64_t n = nv > nt ? nv : nt;
    hipLaunchKernelGGL(k_qem_emit, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, P, nv, used,
                       newid, F, nt, keep, tpos, out_verts, out_tris);
    return hipGetLastError();
}
