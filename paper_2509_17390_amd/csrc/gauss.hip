// gauss.hip -- Gaussian-to-occupancy conversion on gfx950.
//
// FGGS-LiDAR Sec. IV-A ("Grid query and occupancy evaluation") on the
// Gaussian model of Sec. III-A:
//   b_i     box of the k-sigma ellipsoid of G_i: mu +- k sqrt(diag Sigma),
//           Sigma = R S S^T R^T
//   C_tile  the Gaussians whose box meets the box of a tile of 8^3 voxels,
//           found by querying the LBVH built over the b_i (build.hip)
//   D(v)    sum over C_tile of exp(-1/2 (v - mu)^T Sigma^-1 (v - mu)) alpha^2
//   V_occ   D > theta;  Surf = V_occ and not (all six face neighbours occupied)
//
// Kernels:
//   k_gauss_pack      the uploaded arrays interleaved, 48 bytes per Gaussian
//   k_gauss_validate  input checks at upload
//   k_gauss_boxes     b_i: FP64 in one fixed operation order (the library is
//                     built without contraction), each end rounded to the
//                     nearest float32, so that membership in C_tile is an
//                     exact float32 comparison
//   k_gauss_records   64-byte evaluation records in leaf order: mu, the
//                     whitening matrix M = c0 S^-1 R^T and alpha^2 * 2^31
//   k_voxelize        one wave per tile, or four.  Query: 64 nodes off an LDS
//                     stack at a time; culling-set members go to an LDS ring.
//                     Every 64 members the wave stages their
//                     records in LDS (in the tile's voxel-unit frame) and each
//                     lane evaluates one 8-voxel column of the tile against
//                     them.
//   k_surface         6-neighbour test on the occupancy bytes
//
// The density is accumulated in 64-bit fixed point (units of 2^-31 per
// term), so the result does not depend on the order in which the query
// returns culling-set members: it is deterministic and needs no sorting.
// A term with w alpha^2 2^31 < 1/4 rounds to zero, so voxels where the
// exponent exceeds 33 skip the exponential exactly.
#include "gauss_internal.h"

#include <math.h>

namespace {

constexpr int kBlock = 256;
// per wave of a tile: the ring holds what is pending after a step (< 64 + 128)
// and what the last flush may still be read from (64)
constexpr int kRing = 256;        // LDS ring of culling-set members
constexpr int kStack = 320;       // LDS stack of a wave's pending nodes
constexpr int kDepth = 64;        // the tree depth is at most 62
// Tiles up to which four waves share one: a launch that leaves the chip's 1,024
// SIMDs idle or with one tile each.  One wave / four, us: 87 / 40 at 192
// tiles, 111 / 89 at 1,768, 155 / 172 at 5,700, 248 / 333 at 11,550.
constexpr int64_t kSharedTiles = 3072;
constexpr int kSkipRun = 2;       // voxels of a column that are left out together
constexpr float kQSkip = 33.0f;   // exp2(-q) * 2^31 < 1/4 beyond this
constexpr double kC0 = 0.8493218002880191;   // sqrt(log2(e) / 2)
constexpr double kFix = 2147483648.0;        // 2^31: fixed-point unit of one term

// R of q / |q| for q = (w, x, y, z); every step one FP64 operation, in the
// order the Gaussian boxes are defined with.
__device__ __forceinline__ void rotation64(const float4 q4, double R[3][3])
{
    const double w = q4.x, x = q4.y, y = q4.z, z = q4.w;
    const double n = ((w * w + x * x) + y * y) + z * z;
    const double s = 2.0 / n;
    R[0][0] = 1.0 - s * (y * y + z * z);
    R[0][1] = s * (x * y - w * z);
    R[0][2] = s * (x * z + w * y);
    R[1][0] = s * (x * y + w * z);
    R[1][1] = 1.0 - s * (x * x + z * z);
    R[1][2] = s * (y * z - w * x);
    R[2][0] = s * (x * z - w * y);
    R[2][1] = s * (y * z + w * x);
    R[2][2] = 1.0 - s * (x * x + y * y);
}

__global__ __launch_bounds__(kBlock) void k_gauss_pack(GaussArrays a, float4 *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n) return;
    out[3 * i + 0] = make_float4(a.mean[3 * i], a.mean[3 * i + 1], a.mean[3 * i + 2], a.opacity[i]);
    out[3 * i + 1] = make_float4(a.quat[4 * i], a.quat[4 * i + 1], a.quat[4 * i + 2], a.quat[4 * i + 3]);
    out[3 * i + 2] = make_float4(a.scale[3 * i], a.scale[3 * i + 1], a.scale[3 * i + 2], 0.0f);
}

__global__ __launch_bounds__(kBlock) void k_gauss_validate(GaussParams p, int32_t *flags)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.n) return;
    const float4 m = p.g[3 * i], q = p.g[3 * i + 1], s = p.g[3 * i + 2];
    int f = 0;
    const float v[11] = {m.x, m.y, m.z, m.w, q.x, q.y, q.z, q.w, s.x, s.y, s.z};
    for (int k = 0; k < 11; ++k)
        if (!isfinite(v[k])) f |= 1;
    const double qn = (double)q.x * q.x + (double)q.y * q.y + (double)q.z * q.z + (double)q.w * q.w;
    if (!(qn > 0.0)) f |= 4;
    if (!(s.x > 0.0f) || !(s.y > 0.0f) || !(s.z > 0.0f)) f |= 2;
    if (isfinite(m.w) && (m.w < 0.0f || m.w > 1.0f)) f |= 8;
    if (f) atomicOr(flags, f);
}

__global__ __launch_bounds__(kBlock) void k_gauss_boxes(GaussParams p, double k,
                                                        float *__restrict__ boxes)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.n) return;
    const float4 m = p.g[3 * i], sc = p.g[3 * i + 2];
    double R[3][3];
    rotation64(p.g[3 * i + 1], R);
    const double s0 = sc.x, s1 = sc.y, s2 = sc.z;
    const double mu[3] = {m.x, m.y, m.z};
    for (int a = 0; a < 3; ++a) {
        const double c0 = R[a][0] * s0, c1 = R[a][1] * s1, c2 = R[a][2] * s2;
        const double saa = (c0 * c0 + c1 * c1) + c2 * c2;
        const double e = k * sqrt(saa);
        boxes[6 * i + a] = (float)(mu[a] - e);
        boxes[6 * i + 3 + a] = (float)(mu[a] + e);
    }
}

__global__ __launch_bounds__(kBlock) void k_gauss_records(GaussParams p,
                                                          const uint32_t *__restrict__ sorted,
                                                          GaussRec *__restrict__ recs)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= p.n) return;
    const int64_t i = sorted[k];
    const float4 m = p.g[3 * i], sc = p.g[3 * i + 2];
    double R[3][3];
    rotation64(p.g[3 * i + 1], R);
    const double inv[3] = {kC0 / (double)sc.x, kC0 / (double)sc.y, kC0 / (double)sc.z};
    float M[9];
    for (int r = 0; r < 3; ++r)
        for (int j = 0; j < 3; ++j) M[3 * r + j] = (float)(R[j][r] * inv[r]);   // (S^-1 R^T)_rj
    const double al = m.w;
    GaussRec g;
    g.r0 = make_float4(m.x, m.y, m.z, (float)(al * al * kFix));
    g.r1 = make_float4(M[0], M[1], M[2], M[3]);
    g.r2 = make_float4(M[4], M[5], M[6], M[7]);
    g.r3 = make_float4(M[8], __int_as_float((int32_t)i), 0.0f, 0.0f);
    recs[k] = g;
}

__device__ __forceinline__ bool meets(float lx, float hx, float ly, float hy, float lz, float hz,
                                      const float tb[6])
{
    return lx <= tb[3] && hx >= tb[0] && ly <= tb[4] && hy >= tb[1] && lz <= tb[5] &&
           hz >= tb[2];
}

__device__ __forceinline__ uint32_t below(uint64_t m, int lane)
{
    return (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
}

// Test both children of internal node `node` against the tile box.
__device__ __forceinline__ void test_children(const NodeRec *__restrict__ nodes, int32_t node,
                                              const float tb[6], int32_t &cl, int32_t &cr,
                                              bool &hl, bool &hr)
{
    const NodeRec nr = nodes[node];
    cl = nr.q3.x;
    cr = nr.q3.y;
    hl = meets(nr.q0.x, nr.q0.y, nr.q1.x, nr.q1.y, nr.q2.x, nr.q2.y, tb);
    hr = meets(nr.q0.z, nr.q0.w, nr.q1.z, nr.q1.w, nr.q2.z, nr.q2.w, tb);
}

// v's integer part, 0 if v is no number (a Gaussian thinner than float32's
// reciprocals go has terms inf - inf).  The instruction saturates; a cast of
// such a value has no defined result.
__device__ __forceinline__ uint32_t floor_or_0(float v)
{
    uint32_t r;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// LDS written by this wave is read by it next
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// MODE 0: density and occupancy.  MODE 1: |C_tile| per tile only.
//
// Bound by VALU issue on a grid of many tiles, 88 instructions a member and
// wave, eight of them quarter-rate exponentials: 510 x 410 x 160 voxels and 1M
// Gaussians (4.7M members) take 882 us; 964 with a test and a branch per voxel
// and a depth-first walk per lane for the query, 926 with tests per voxel, 925
// per four, 938 with none.  (The matrix cores' 4 x 4 outer products for u give
// the same bits, but the moves to and from their registers cost more than the
// 21 multiply-adds: 1,223.)
//
// WAVES: a launch of few tiles ends with its heaviest one, so four waves share
// a tile: the stack, the ring, and a quarter of the members each; their sums
// are whole numbers and add up to the same density in any order.
template <int MODE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(6))) void
k_voxelize(const NodeRec *__restrict__ nodes,
                                                         const GaussRec *__restrict__ recs,
                                                         const float *__restrict__ boxes,
                                                         int64_t n_gauss, VoxGrid g,
                                                         float *__restrict__ density,
                                                         uint8_t *__restrict__ occ,
                                                         int32_t *__restrict__ counts)
{
    static_assert(MODE == 0 || WAVES == 1, "one wave counts a tile");
    constexpr int kThreads = 64 * WAVES, kSlots = kRing * WAVES, kNodes = kStack * WAVES;
    __shared__ int32_t ring[kSlots];
    __shared__ int32_t stack[kNodes];
    __shared__ float4 s_stage[WAVES][64 * 4];
    __shared__ uint32_t s_count[2][WAVES];      // leaves | inner nodes << 16, of a step's parity

    // Workgroups are dealt to the 8 XCDs in turn (workgroup b on XCD b % 8):
    // give each XCD one contiguous run of tiles so that neighbouring tiles,
    // which share most of their culling sets, share an L2.
    const int64_t per = (int64_t)gridDim.x / 8;
    const int64_t tile = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (tile >= g.n_tiles) return;
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    float4 *stage = s_stage[wave];
    const int ti = (int)(tile % g.tx);
    const int tj = (int)((tile / g.tx) % g.ty);
    const int tk = (int)(tile / ((int64_t)g.tx * g.ty));
    const int i0 = ti * kVoxTile, j0 = tj * kVoxTile, k0 = tk * kVoxTile;
    const int ie = min(i0 + kVoxTile, g.nx), je = min(j0 + kVoxTile, g.ny),
              ke = min(k0 + kVoxTile, g.nz);
    float tb[6];
    tb[0] = (float)(g.o[0] + (double)i0 * g.h);
    tb[1] = (float)(g.o[1] + (double)j0 * g.h);
    tb[2] = (float)(g.o[2] + (double)k0 * g.h);
    tb[3] = (float)(g.o[0] + (double)ie * g.h);
    tb[4] = (float)(g.o[1] + (double)je * g.h);
    tb[5] = (float)(g.o[2] + (double)ke * g.h);

    // evaluation frame: voxel units, origin at the tile's first voxel centre
    const double v0x = g.o[0] + ((double)i0 + 0.5) * g.h;
    const double v0y = g.o[1] + ((double)j0 + 0.5) * g.h;
    const double v0z = g.o[2] + ((double)k0 + 0.5) * g.h;
    const double inv_h = 1.0 / g.h;
    const float hf = (float)g.h;
    const int cy = lane & 7, cz = lane >> 3;   // this lane's column of 8 voxels along x
    const float py = (float)cy, pz = (float)cz;

    uint64_t acc[kVoxTile];
#pragma unroll
    for (int x = 0; x < kVoxTile; ++x) acc[x] = 0;
    uint32_t head = 0, tail = 0;   // ring positions (wave-uniform)
    int64_t total = 0;

    // Evaluate the next m (<= kThreads) members of the ring against this lane's
    // column, each wave its share, and drop them from the ring.
    auto flush = [&](uint32_t all) {
        if (MODE == 1) {
            total += all;
            head += all;
            return;
        }
        const uint32_t share = (all + WAVES - 1) / WAVES, from = share * (uint32_t)wave;
        const uint32_t m = all > from ? min(share, all - from) : 0u;
        if ((uint32_t)lane < m) {
            const GaussRec r = recs[ring[(head + from + lane) & (kSlots - 1)]];
            const float M[9] = {r.r1.x * hf, r.r1.y * hf, r.r1.z * hf, r.r1.w * hf, r.r2.x * hf,
                                r.r2.y * hf, r.r2.z * hf, r.r2.w * hf, r.r3.x * hf};
            const double c0 = ((double)r.r0.x - v0x) * inv_h;
            const double c1 = ((double)r.r0.y - v0y) * inv_h;
            const double c2 = ((double)r.r0.z - v0z) * inv_h;
            float a[3];
            for (int k = 0; k < 3; ++k)
                a[k] = (float)(((double)M[3 * k] * c0 + (double)M[3 * k + 1] * c1) +
                               (double)M[3 * k + 2] * c2);
            stage[4 * lane + 0] = make_float4(M[0], M[1], M[2], a[0]);
            stage[4 * lane + 1] = make_float4(M[3], M[4], M[5], a[1]);
            stage[4 * lane + 2] = make_float4(M[6], M[7], M[8], a[2]);
            stage[4 * lane + 3] = make_float4(r.r0.w, 0.0f, 0.0f, 0.0f);
        }
        wave_lds_fence();
        for (uint32_t r = 0; r < m; ++r) {
            const float4 s0 = stage[4 * r + 0], s1 = stage[4 * r + 1], s2 = stage[4 * r + 2];
            const float A = stage[4 * r + 3].x;
            // u = M (p - c) = M p - a with p = (x, cy, cz) in voxel units
            const float b0 = fmaf(s0.y, py, fmaf(s0.z, pz, -s0.w));
            const float b1 = fmaf(s1.y, py, fmaf(s1.z, pz, -s1.w));
            const float b2 = fmaf(s2.y, py, fmaf(s2.z, pz, -s2.w));
#pragma unroll
            for (int x0 = 0; x0 < kVoxTile; x0 += kSkipRun) {
                float q[kSkipRun], least = INFINITY;
#pragma unroll
                for (int k = 0; k < kSkipRun; ++k) {
                    const int x = x0 + k;
                    const float u0 = x ? fmaf(s0.x, (float)x, b0) : b0;
                    const float u1 = x ? fmaf(s1.x, (float)x, b1) : b1;
                    const float u2 = x ? fmaf(s2.x, (float)x, b2) : b2;
                    q[k] = fmaf(u0, u0, fmaf(u1, u1, u2 * u2));
                    least = fminf(least, q[k]);
                }
                // terms with q > 33 (or no number) round to 0: left out where
                // that holds in every lane (of a launch that VALU issue
                // bounds), added elsewhere
                if (WAVES > 1 || __ballot(least <= kQSkip)) {
#pragma unroll
                    for (int k = 0; k < kSkipRun; ++k)
                        acc[x0 + k] += floor_or_0(fmaf(__builtin_amdgcn_exp2f(-q[k]), A, 0.5f));
                }
            }
        }
        wave_lds_fence();
        head += all;
    };

    auto sync = [&]() {
        if (WAVES > 1) __syncthreads();
        else wave_lds_fence();
    };
    if (n_gauss == 1) {
        if (meets(boxes[0], boxes[3], boxes[1], boxes[4], boxes[2], boxes[5], tb)) {
            if (threadIdx.x == 0) ring[0] = 0;
            tail = 1;
        }
        sync();
    } else if (n_gauss > 1) {
        // as many nodes as threads off the top of the stack at a time; near its
        // end fewer, down to one, which never needs more than the tree's depth
        // beyond what is there
        int top = 1, step = 0;
        if (threadIdx.x == 0) stack[0] = 0;
        sync();
        while (top > 0) {
            const int room = kNodes - kDepth - top;
            const int k = min(min(kThreads, top), max(1, room));
            const int32_t node = (int)threadIdx.x < k ? stack[top - 1 - (int)threadIdx.x] : -1;
            top -= k;
            int32_t cl = 0, cr = 0;
            bool hl = false, hr = false;
            if (node >= 0) test_children(nodes, node, tb, cl, cr, hl, hr);
            // children that are leaves go to the ring, the others to the stack
            // (ballot compaction; the order within a step is irrelevant)
            const bool ll = hl && cl < 0, lr = hr && cr < 0, il = hl && cl >= 0, ir = hr && cr >= 0;
            const uint64_t bll = __ballot(ll), blr = __ballot(lr);
            const uint64_t bil = __ballot(il), bir = __ballot(ir);
            const uint32_t nl = (uint32_t)(__popcll(bll) + __popcll(blr));
            const uint32_t ni = (uint32_t)(__popcll(bil) + __popcll(bir));
            uint32_t l0 = tail, i0w = (uint32_t)top, nl_all = nl, ni_all = ni;
            if (WAVES > 1) {
                if (lane == 0) s_count[step & 1][wave] = nl | (ni << 16);
                __syncthreads();               // and every node of the step is read
                nl_all = ni_all = 0;
                for (int w = 0; w < WAVES; ++w) {
                    const uint32_t c = s_count[step & 1][w];
                    if (w < wave) {
                        l0 += c & 0xffffu;
                        i0w += c >> 16;
                    }
                    nl_all += c & 0xffffu;
                    ni_all += c >> 16;
                }
            } else {
                wave_lds_fence();
            }
            if (ll) ring[(l0 + below(bll, lane)) & (kSlots - 1)] = ~cl;
            if (lr) ring[(l0 + (uint32_t)__popcll(bll) + below(blr, lane)) & (kSlots - 1)] = ~cr;
            if (il) stack[i0w + below(bil, lane)] = cl;
            if (ir) stack[i0w + (uint32_t)__popcll(bil) + below(bir, lane)] = cr;
            tail += nl_all;
            top += (int)ni_all;
            ++step;
            sync();
            while (tail - head >= (uint32_t)kThreads) flush(kThreads);
        }
    }
    if (tail > head) flush(tail - head);

    if (MODE == 1) {
        if (lane == 0) counts[tile] = (int32_t)total;
        return;
    }
    if (WAVES > 1) {
        // each wave adds up and writes its share of the columns' voxels
        uint64_t *sums = reinterpret_cast<uint64_t *>(stage);
        static_assert(sizeof s_stage[0] == 8 * 64 * sizeof(uint64_t), "a wave's sums fit its stage");
#pragma unroll
        for (int k = 0; k < 8; ++k) sums[64 * k + lane] = acc[k];
        __syncthreads();
    }
    const uint64_t *all = reinterpret_cast<const uint64_t *>(s_stage);
    const int y = j0 + cy, z = k0 + cz;
    if (y >= je || z >= ke) return;
    const int64_t row = ((int64_t)z * g.ny + y) * g.nx;
#pragma unroll
    for (int x = 0; x < kVoxTile; ++x) {
        if (WAVES > 1 && x % WAVES != wave) continue;
        uint64_t sum = acc[x];
        if (WAVES > 1) {
            sum = 0;
            for (int w = 0; w < WAVES; ++w) sum += all[8 * 64 * w + 64 * x + lane];
        }
        if (i0 + x < ie) {
            const float d = (float)((double)sum * (1.0 / kFix));
            if (density) density[row + i0 + x] = d;
            if (occ) occ[row + i0 + x] = d > g.theta ? 1 : 0;
        }
    }
}

__device__ __forceinline__ uint32_t udiv32(uint32_t n, UDiv d)
{
    const uint32_t t = __umulhi(n, d.m);
    return (t + ((n - t) >> (d.sh & 0xffu))) >> (d.sh >> 8);
}

// Four consecutive voxels of a row per thread; rows are (z, y) pairs.
__global__ __launch_bounds__(kBlock) void k_surface(const uint8_t *__restrict__ occ,
                                                    uint8_t *__restrict__ surf, int nx, int ny,
                                                    int nz, uint32_t n_threads, int quads,
                                                    UDiv div_quads, UDiv div_ny)
{
    const uint32_t t = blockIdx.x * (uint32_t)kBlock + threadIdx.x;
    if (t >= n_threads) return;
    const uint32_t row = udiv32(t, div_quads);
    const int x0 = 4 * (int)(t - row * (uint32_t)quads);
    const uint32_t zz = udiv32(row, div_ny);
    const int y = (int)(row - zz * (uint32_t)ny), z = (int)zz;
    const int64_t sxy = (int64_t)nx * ny;
    const int64_t base = (int64_t)row * nx;
    const bool ym = y > 0, yp = y < ny - 1, zm = z > 0, zp = z < nz - 1;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int x = x0 + k;
        if (x >= nx) break;
        const int64_t i = base + x;
        uint8_t s = 0;
        if (occ[i]) {
            const bool interior = x > 0 && x < nx - 1 && ym && yp && zm && zp && occ[i - 1] &&
                                  occ[i + 1] && occ[i - nx] && occ[i + nx] && occ[i - sxy] &&
                                  occ[i + sxy];
            s = interior ? 0 : 1;
        }
        surf[i] = s;
    }
}

// The same for rows of 16 voxels and more, 16 per thread: the five rows' bytes
// (0 or 1) as four words each, the x neighbours by byte shifts, one store.  A
// row's last thread takes its last 16 voxels, some of them its neighbour's too
// (equal stores).  Bound by memory: 23 us on 33.5M voxels; four voxels a
// thread, seven byte reads each, took 83 us.
__global__ __launch_bounds__(kBlock) void k_surface16(const uint8_t *__restrict__ occ,
                                                      uint8_t *__restrict__ surf, int nx, int ny,
                                                      int nz, uint32_t n_threads, int runs,
                                                      UDiv div_runs, UDiv div_ny)
{
    const uint32_t t = blockIdx.x * (uint32_t)kBlock + threadIdx.x;
    if (t >= n_threads) return;
    const uint32_t row = udiv32(t, div_runs);
    int x0 = 16 * (int)(t - row * (uint32_t)runs);
    if (x0 > nx - 16) x0 = nx - 16;
    const uint32_t zz = udiv32(row, div_ny);
    const int y = (int)(row - zz * (uint32_t)ny), z = (int)zz;
    const int64_t sxy = (int64_t)nx * ny, i = (int64_t)row * nx + x0;
    // a row outside the grid is free: read the own row in its place
    const bool ym = y > 0, yp = y < ny - 1, zm = z > 0, zp = z < nz - 1;
    uint32_t c[4], n[4][4];
    __builtin_memcpy(c, occ + i, 16);
    __builtin_memcpy(n[0], occ + (ym ? i - nx : i), 16);
    __builtin_memcpy(n[1], occ + (yp ? i + nx : i), 16);
    __builtin_memcpy(n[2], occ + (zm ? i - sxy : i), 16);
    __builtin_memcpy(n[3], occ + (zp ? i + sxy : i), 16);
    const uint32_t before = x0 > 0 ? occ[i - 1] : 0u, after = x0 + 16 < nx ? occ[i + 16] : 0u;
    const uint32_t inside = ym && yp && zm && zp ? 0xffffffffu : 0u;
    uint32_t out[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t l = __builtin_amdgcn_alignbyte(c[k], k ? c[k > 0 ? k - 1 : 0] : before << 24, 3u);
        const uint32_t r = __builtin_amdgcn_alignbyte(k < 3 ? c[k < 3 ? k + 1 : 3] : after, c[k], 1u);
        out[k] = c[k] & ~(l & r & n[0][k] & n[1][k] & n[2][k] & n[3][k] & inside);
    }
    __builtin_memcpy(surf + i, out, 16);
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

hipError_t gauss_pack_launch(const GaussArrays &a, float4 *out, hipStream_t s)
{
    if (a.n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gauss_pack, dim3(grid_for(a.n, kBlock)), dim3(kBlock), 0, s, a, out);
    return hipGetLastError();
}

hipError_t gauss_validate_launch(const GaussParams &p, int32_t *flags, hipStream_t s)
{
    if (p.n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gauss_validate, dim3(grid_for(p.n, kBlock)), dim3(kBlock), 0, s, p,
                       flags);
    return hipGetLastError();
}

hipError_t gauss_boxes_launch(const GaussParams &p, float k, float *boxes, hipStream_t s)
{
    if (p.n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gauss_boxes, dim3(grid_for(p.n, kBlock)), dim3(kBlock), 0, s, p,
                       (double)k, boxes);
    return hipGetLastError();
}

hipError_t gauss_records_launch(const GaussParams &p, const uint32_t *sorted, GaussRec *recs,
                                hipStream_t s)
{
    if (p.n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gauss_records, dim3(grid_for(p.n, kBlock)), dim3(kBlock), 0, s, p,
                       sorted, recs);
    return hipGetLastError();
}

hipError_t voxelize_launch(int mode, const NodeRec *nodes, const GaussRec *recs,
                           const float *boxes, int64_t n_gauss, const VoxGrid &g,
                           float *density, uint8_t *occ, int32_t *tile_counts, hipStream_t s)
{
    if (g.n_tiles <= 0) return hipSuccess;
    const int64_t blocks = (g.n_tiles + 7) / 8 * 8;   // a multiple of the XCD count
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (mode != 0)
        hipLaunchKernelGGL((k_voxelize<1, 1>), dim3((unsigned)blocks), dim3(64), 0, s, nodes, recs,
                           boxes, n_gauss, g, density, occ, tile_counts);
    else if (g.n_tiles <= kSharedTiles)
        hipLaunchKernelGGL((k_voxelize<0, 4>), dim3((unsigned)blocks), dim3(256), 0, s, nodes, recs,
                           boxes, n_gauss, g, density, occ, tile_counts);
    else
        hipLaunchKernelGGL((k_voxelize<0, 1>), dim3((unsigned)blocks), dim3(64), 0, s, nodes, recs,
                           boxes, n_gauss, g, density, occ, tile_counts);
    return hipGetLastError();
}

hipError_t surface_launch(const uint8_t *occ, uint8_t *surf, const VoxGrid &g, hipStream_t s)
{
    const int quads = (g.nx + 3) / 4;
    const int64_t rows = (int64_t)g.ny * g.nz;
    const int64_t threads = (int64_t)quads * rows;
    if (threads <= 0) return hipSuccess;
    if (threads > 0xffffff00LL) return hipErrorInvalidValue;
    if (g.nx >= 16) {
        const int runs = (g.nx + 15) / 16;
        const int64_t n = (int64_t)runs * rows;
        hipLaunchKernelGGL(k_surface16, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, occ, surf,
                           g.nx, g.ny, g.nz, (uint32_t)n, runs, udiv_magic((uint32_t)runs),
                           udiv_magic((uint32_t)g.ny));
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_surface, dim3(grid_for(threads, kBlock)), dim3(kBlock), 0, s, occ, surf,
                       g.nx, g.ny, g.nz, (uint32_t)threads, quads, udiv_magic((uint32_t)quads),
                       udiv_magic((uint32_t)g.ny));
    return hipGetLastError();
}
