// tsdf.hip -- denoising, flood-fill sign, narrow-band TSDF and marching cubes
// on gfx950 (FGGS-LiDAR Sec. IV-B).
//
//   V'    = G * V (binomial kernel of n steps: integer weights C(2n, n+k),
//           the discrete Gaussian of variance n / 2), separable, exact in
//           64-bit integers; V~ = [V' >= tau], decided on the exact sum
//   O     = free voxels 6-connected to a free frame around the grid:
//           rounds of sweeps along x, y and z lines, spreading along whole
//           free runs, until a round changes nothing (x and y of a slice
//           in one kernel where it fits LDS)
//   S_0   = voxels with a 6-neighbour of the other V~ value (frame = free)
//   p     = shell index of a 6-neighbour expansion from S_0, up to ceil(r / h)
//           shells: for at most 4, S_0, the shells and phi in one pass on the
//           packed words of V~; else one launch each
//   phi   = clip(s p h, -r, r), s = +1 on O, -1 elsewhere
//   mesh  = marching cubes of phi at iso on the voxel-centre lattice:
//           per point, count crossed lattice edges (one vertex each) and the
//           triangles of the cell it anchors; tile scans give every vertex
//           and triangle its slot; a second pass writes them.  The case
//           table is built on the host from a walk over the cube's faces.
#include "mesh_internal.h"

#include <math.h>

#include <mutex>

namespace {

constexpr int kBlock = 256;
constexpr int kScanItems = 4;                  // per thread in the block scan
constexpr int kScanTile = kBlock * kScanItems;

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

// (x, y, z) of voxel i.  Below 2^32 voxels the divisions by nx and ny are
// multiplications (64-bit integer division is a long emulated sequence,
// and these kernels run it for every voxel).
__device__ __forceinline__ uint32_t div_by(uint32_t n, uint64_t c)
{
    return c ? (uint32_t)__umul64hi(c, (uint64_t)n) : n;
}

__device__ __forceinline__ void coords(int64_t i, const TsdfGrid &g, int &x, int &y, int &z)
{
    if (g.n <= (int64_t)0xffffffffLL) {
        const uint32_t u = (uint32_t)i;
        const uint32_t r = div_by(u, g.cx);
        x = (int)(u - r * (uint32_t)g.nx);
        const uint32_t zz = div_by(r, g.cy);
        y = (int)(r - zz * (uint32_t)g.ny);
        z = (int)zz;
        return;
    }
    x = (int)(i % g.nx);
    const int64_t r = i / g.nx;
    y = (int)(r % g.ny);
    z = (int)(r / g.ny);
}

// ---- smoothing and re-threshold ------------------------------------------
__global__ __launch_bounds__(kBlock) void k_smooth_x(const uint8_t *__restrict__ v,
                                                     uint32_t *__restrict__ out, TsdfGrid g,
                                                     Binomial w)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.n) return;
    int x, y, z;
    coords(i, g, x, y, z);
    uint32_t s = 0;
    for (int k = -w.n; k <= w.n; ++k) {
        const int xx = x + k;
        if (xx >= 0 && xx < g.nx && v[i + k]) s += w.w[k + w.n];
    }
    out[i] = s;
}

__global__ __launch_bounds__(kBlock) void k_smooth_y(const uint32_t *__restrict__ a,
                                                     uint64_t *__restrict__ out, TsdfGrid g,
                                                     Binomial w)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.n) return;
    int x, y, z;
    coords(i, g, x, y, z);
    uint64_t s = 0;
    for (int k = -w.n; k <= w.n; ++k) {
        const int yy = y + k;
        if (yy >= 0 && yy < g.ny) s += (uint64_t)w.w[k + w.n] * a[i + (int64_t)k * g.nx];
    }
    out[i] = s;
}

__global__ __launch_bounds__(kBlock) void k_smooth_z(const uint64_t *__restrict__ b,
                                                     uint8_t *__restrict__ vt, TsdfGrid g,
                                                     Binomial w, uint64_t thr)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.n) return;
    const int64_t sxy = (int64_t)g.nx * g.ny;
    int x, y, z;
    coords(i, g, x, y, z);
    uint64_t s = 0;
    for (int k = -w.n; k <= w.n; ++k) {
        const int zz = z + k;
        if (zz >= 0 && zz < g.nz) s += (uint64_t)w.w[k + w.n] * b[i + (int64_t)k * sxy];
    }
    vt[i] = s >= thr ? 1 : 0;
}

// The same z pass keeping the integer sums (for the quantile re-threshold),
// and the threshold of such sums against a value held on the device.
__global__ __launch_bounds__(kBlock) void k_smooth_z_sum(const uint64_t *__restrict__ b,
                                                         uint64_t *__restrict__ out, TsdfGrid g,
                                                         Binomial w)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.n) return;
    const int64_t sxy = (int64_t)g.nx * g.ny;
    int x, y, z;
    coords(i, g, x, y, z);
    uint64_t s = 0;
    for (int k = -w.n; k <= w.n; ++k) {
        const int zz = z + k;
        if (zz >= 0 && zz < g.nz) s += (uint64_t)w.w[k + w.n] * b[i + (int64_t)k * sxy];
    }
    out[i] = s;
}

// Tile number of a block, consecutive tiles on one XCD (workgroups go to the 8
// XCDs in turn): neighbouring tiles share lines of packed words in its L2.
// Launches of many tiles have several rows of kTileRow blocks: a tile of a thin
// grid holds few voxels, and a launch's x axis ends at 2^32 work-items.
constexpr int64_t kTileRow = 1 << 16;

__device__ __forceinline__ uint32_t xcd_tile()
{
    return blockIdx.y * gridDim.x + (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

inline dim3 xcd_tiles(int64_t n)
{
    if (n <= kTileRow) return dim3((unsigned)((n + 7) / 8 * 8));
    return dim3((unsigned)kTileRow, (unsigned)((n + kTileRow - 1) / kTileRow));
}

// lane k's value, the same in every lane; and the lane's own bit of such a word
__device__ __forceinline__ uint64_t read_lane64(uint64_t v, int k)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), k);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ bool lane_bit(uint64_t w) { return __builtin_amdgcn_inverse_ballot_w64(w); }

// Kernels of at most 3 steps run on bits, 64 voxels of a row to a word: the
// surface bytes are packed once, and the sums are held bit-sliced, one word
// per bit of the sum, so that an addition of 64 voxels is a few word
// operations per bit.  The integer sums are those of the per-voxel passes.
// (Bytes in LDS tiles, one voxel a lane, took 116 us on 34.2M voxels at n = 1:
// two LDS reads and an add per voxel, tap and axis; these take 23 + 12 us.)
//
// Packing: 16 bytes a lane, four lanes a word, kPackRun words of a lane's
// reads in flight (a byte a lane and a ballot a word: 25 us, these 23 us,
// 1.5 TB/s on a mask that no cache holds).
constexpr int kPackRun = 4;

// bit j: byte j of v is not 0
__device__ __forceinline__ uint32_t nonzero_nibble(uint32_t v)
{
    const uint32_t t = (((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u;
    return (t >> 7) * 0x10204080u >> 28;
}

template <bool FREE>    // the words of V~ = 0 and clear outside words, else of non-zero bytes
__global__ __launch_bounds__(kBlock) void k_pack_bits(const uint8_t *__restrict__ v, TsdfGrid g,
                                                      int W, uint64_t cw,
                                                      uint64_t *__restrict__ bits,
                                                      uint64_t *__restrict__ O)
{
    const int64_t nw = (int64_t)W * g.ny * g.nz;
    const int part = (int)(threadIdx.x & 3);
    const int64_t w0 = (int64_t)blockIdx.x * (kBlock / 4 * kPackRun) + (threadIdx.x >> 2);
    uint32_t d[kPackRun][4];
    int left[kPackRun];          // the row's voxels from the lane's first on
    int64_t at[kPackRun];
#pragma unroll
    for (int k = 0; k < kPackRun; ++k) {
        const int64_t w = w0 + k * (kBlock / 4);
        const int64_t row = nw <= (int64_t)0xffffffffLL ? (int64_t)div_by((uint32_t)w, cw) : w / W;
        const int x = 64 * (int)(w - row * W) + 16 * part;
        left[k] = w < nw ? g.nx - x : 0;
        at[k] = left[k] > 0 ? row * g.nx + x : 0;
    }
    // no branch between the reads (each would wait for the one before); a
    // read may reach into the next row, and the grid's last 15 bytes are
    // read one by one
    if (g.n >= 16) {
#pragma unroll
        for (int k = 0; k < kPackRun; ++k)
            __builtin_memcpy(d[k], v + (at[k] + 16 <= g.n ? at[k] : 0), 16);
    }
#pragma unroll
    for (int k = 0; k < kPackRun; ++k)
        if (at[k] + 16 > g.n) {
            d[k][0] = d[k][1] = d[k][2] = d[k][3] = 0;
            for (int j = 0; at[k] + j < g.n; ++j) d[k][j >> 2] |= (uint32_t)v[at[k] + j] << (8 * (j & 3));
        }
#pragma unroll
    for (int k = 0; k < kPackRun; ++k) {
        const int64_t w = w0 + k * (kBlock / 4);
        const uint32_t in = left[k] >= 16 ? 0xffffu : left[k] > 0 ? (1u << left[k]) - 1u : 0u;
        uint32_t m = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) m |= nonzero_nibble(d[k][j]) << (4 * j);
        m = (FREE ? ~m : m) & in;
        m <<= 16 * (part & 1);
        m |= (uint32_t)__shfl_xor((int)m, 1, 64);         // the pair's half of the word
        if ((part & 1) == 0 && w < nw) {
            reinterpret_cast<uint32_t *>(bits)[2 * w + (part >> 1)] = m;
            if (FREE) reinterpret_cast<uint32_t *>(O)[2 * w + (part >> 1)] = 0;
        }
    }
}

// V~ = [sums >= *thr] as free words (and bytes, if asked for), with clear
// outside words: a ballot a word, kPackSums words' reads in flight.  (Bytes and
// a packing launch behind them took 4 + 7 us on 350,200 voxels, this 4.)
constexpr int kPackSums = 4;

__global__ __launch_bounds__(kBlock) void k_threshold_pack(const uint64_t *__restrict__ sums,
                                                           const uint64_t *__restrict__ thr,
                                                           uint8_t *__restrict__ vt, TsdfGrid g,
                                                           int W, uint64_t *__restrict__ F,
                                                           uint64_t *__restrict__ O)
{
    const int64_t w0 = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * kPackSums;
    const int64_t nw = (int64_t)W * g.ny * g.nz;
    if (w0 >= nw) return;                                 // whole waves
    const int lane = (int)(threadIdx.x & 63);
    const uint64_t t = *thr;
    int64_t row = w0 / W, at[kPackSums];
    int wx = (int)(w0 - row * W);
    uint64_t v[kPackSums];
    bool ok[kPackSums];
#pragma unroll
    for (int k = 0; k < kPackSums; ++k) {
        const int x = 64 * wx + lane;
        ok[k] = w0 + k < nw && x < g.nx;
        at[k] = ok[k] ? row * g.nx + x : 0;
        v[k] = sums[at[k]];
        if (++wx == W) {
            wx = 0;
            ++row;
        }
    }
#pragma unroll
    for (int k = 0; k < kPackSums; ++k) {
        const bool one = v[k] >= t;
        const uint64_t f = __ballot(ok[k] && !one);
        if (vt && ok[k]) vt[at[k]] = one ? 1 : 0;
        if (lane == 0 && w0 + k < nw) {
            F[w0 + k] = f;
            O[w0 + k] = 0;
        }
    }
}

// a += b << S on bit-sliced numbers of NA and NB bits (modulo 2^NA)
template <int S, int NA, int NB>
__device__ __forceinline__ void slice_add(uint64_t (&a)[NA], const uint64_t (&b)[NB])
{
    uint64_t carry = 0;
#pragma unroll
    for (int i = S; i < NA; ++i) {
        const uint64_t x = a[i];
        if (i - S < NB) {
            const uint64_t y = x ^ b[i - S < NB ? i - S : 0];
            const uint64_t c = (x & b[i - S < NB ? i - S : 0]) | (carry & y);
            a[i] = y ^ carry;
            carry = c;
        } else {
            a[i] = x ^ carry;
            carry &= x;
        }
    }
}

constexpr uint32_t binomial(int n, int k) { return k == 0 ? 1u : binomial(n, k - 1) * (uint32_t)(n - k + 1) / (uint32_t)k; }

// a += w b
template <uint32_t WT, int S, int NA, int NB>
__device__ __forceinline__ void slice_madd(uint64_t (&a)[NA], const uint64_t (&b)[NB])
{
    if constexpr (WT != 0) {
        if constexpr ((WT & 1u) != 0) slice_add<S>(a, b);
        slice_madd<(WT >> 1), S + 1>(a, b);
    }
}

// out = the weighted sum over the 2N + 1 taps get(k, number), k = -N .. N
template <int N, int K, int NA, int NB, class Get>
__device__ __forceinline__ void slice_taps(uint64_t (&out)[NA], const Get &get, const uint64_t (&)[NB])
{
    if constexpr (K <= N) {
        uint64_t t[NB + 1], u[NB];
        get(K, u);
#pragma unroll
        for (int i = 0; i < NB; ++i) t[i] = u[i];
        t[NB] = 0;
        if constexpr (K > 0) {
            get(-K, u);
            slice_add<0>(t, u);
        }
        slice_madd<binomial(2 * N, N + K), 0>(out, t);
        slice_taps<N, K + 1>(out, get, u);
    }
}

constexpr int kSmY = 16, kSmZ = 16;

// A block owns one word by kSmY x kSmZ rows: the x sums of its rows and a halo
// of N, the x-y sums, and the full sums, which are compared with the
// threshold bit by bit.  Writes V~ (if asked for), the free words and clear
// outside words.
template <int N>
__global__ __launch_bounds__(kBlock) void k_smooth_bits(const uint64_t *__restrict__ bits,
                                                        uint8_t *__restrict__ vt, TsdfGrid g,
                                                        uint64_t thr, int W,
                                                        uint64_t *__restrict__ F,
                                                        uint64_t *__restrict__ O)
{
    constexpr int PX = 2 * N + 1, PY = 4 * N + 1, PZ = 6 * N + 1;   // bits of sums up to 2^(2N axes)
    constexpr int LY = kSmY + 2 * N, LZ = kSmZ + 2 * N;
    static_assert(kSmY * kSmZ == kBlock && kSmY == 16, "a row a thread");
    __shared__ uint64_t X[PX][LZ * LY];
    __shared__ uint64_t Y[PY][LZ * kSmY];
    const uint32_t tile = xcd_tile(), ty = (uint32_t)(g.ny + kSmY - 1) / kSmY;
    const int bx = (int)(tile % (uint32_t)W), by = (int)(tile / (uint32_t)W % ty) * kSmY;
    const int bz = (int)(tile / (uint32_t)W / ty) * kSmZ;
    if (bz >= g.nz) return;
    for (int q = threadIdx.x; q < LY * LZ; q += kBlock) {
        const int gy = by - N + q % LY, gz = bz - N + q / LY;
        uint64_t l = 0, c = 0, r = 0;
        if (gy >= 0 && gy < g.ny && gz >= 0 && gz < g.nz) {
            const uint64_t *p = bits + ((int64_t)gz * g.ny + gy) * W + bx;
            c = p[0];
            if (bx > 0) l = p[-1];
            if (bx + 1 < W) r = p[1];
        }
        uint64_t out[PX] = {};
        const uint64_t one[1] = {0};
        slice_taps<N, 0>(out, [&](int k, uint64_t (&u)[1]) {
            u[0] = k == 0 ? c : k < 0 ? (c << -k) | (l >> (64 + k)) : (c >> k) | (r << (64 - k));
        }, one);
#pragma unroll
        for (int i = 0; i < PX; ++i) X[i][q] = out[i];
    }
    __syncthreads();
    for (int q = threadIdx.x; q < kSmY * LZ; q += kBlock) {
        const int at = (q / kSmY) * LY + q % kSmY + N;
        uint64_t out[PY] = {};
        const uint64_t one[PX] = {0};
        slice_taps<N, 0>(out, [&](int k, uint64_t (&u)[PX]) {
#pragma unroll
            for (int i = 0; i < PX; ++i) u[i] = X[i][at + k];
        }, one);
#pragma unroll
        for (int i = 0; i < PY; ++i) Y[i][q] = out[i];
    }
    __syncthreads();
    uint64_t sum[PZ] = {};
    {
        const int at = (int)threadIdx.x + N * kSmY;
        const uint64_t one[PY] = {0};
        slice_taps<N, 0>(sum, [&](int k, uint64_t (&u)[PY]) {
#pragma unroll
            for (int i = 0; i < PY; ++i) u[i] = Y[i][at + k * kSmY];
        }, one);
    }
    uint64_t ge = ~0ull;                  // sum >= thr on the bits so far
#pragma unroll
    for (int i = 0; i < PZ; ++i) ge = (thr >> i) & 1ull ? sum[i] & ge : sum[i] | ge;
    if (thr >> PZ) ge = 0;
    const int gy = by + (int)threadIdx.x % kSmY, gz = bz + (int)threadIdx.x / kSmY;
    const uint64_t valid = bx == W - 1 ? ~0ull >> (63 - ((g.nx - 1) & 63)) : ~0ull;
    if (gy < g.ny && gz < g.nz) {
        const int64_t w = ((int64_t)gz * g.ny + gy) * W + bx;
        F[w] = valid & ~ge;
        O[w] = 0;
    }
    if (!vt) return;
    // a row at a time, lane x
    const int lane = (int)threadIdx.x & 63, gx = 64 * bx + lane;
    for (int k = 0; k < 64; ++k) {
        const int t = ((int)threadIdx.x & ~63) + k, y = by + t % kSmY, z = bz + t / kSmY;
        const bool one = lane_bit(read_lane64(ge, k));
        if (gx < g.nx && y < g.ny && z < g.nz)
            vt[((int64_t)z * g.ny + y) * g.nx + gx] = one ? 1 : 0;
    }
}

// ---- outside labelling -----------------------------------------------------
// Bit-packed along x: word (z, y, wx) holds voxels x = 64 wx .. 64 wx + 63
// of row (y, z); F = free (V~ = 0), O = known to be outside; bits beyond
// nx are never free.  A sweep along an axis makes every run of free voxels
// on a line that holds an outside voxel or touches the frame (beyond both
// ends of the line) outside; sweeps along x, y and z repeat until a round
// changes nothing, which is the 6-connected component joined to the frame
// (a path to the frame is a chain of axis-parallel runs).  O only grows.
//
// x: one thread per row, an occluded fill per word with a carry bit.
// y and z: 64 lines per thread (one word column), where one row step is
// R = F & (R | O).  Lines are cut into kSegRows-row segments for
// parallelism: (1) per segment, the reach out of its end and out of its
// start from its own seeds, and the lines it is free on throughout; (2) per
// column, the carries into each segment from the frame and the segments
// before and after it; (3) per segment, the walk forward from its left
// carry and backward from its right carry.
constexpr int kSegRows = 16;

__device__ __forceinline__ uint64_t fill_up(uint64_t gen, uint64_t pro)
{
    gen |= pro & (gen << 1);
    pro &= pro << 1;
    gen |= pro & (gen << 2);
    pro &= pro << 2;
    gen |= pro & (gen << 4);
    pro &= pro << 4;
    gen |= pro & (gen << 8);
    pro &= pro << 8;
    gen |= pro & (gen << 16);
    pro &= pro << 16;
    gen |= pro & (gen << 32);
    return gen;
}

__device__ __forceinline__ uint64_t fill_down(uint64_t gen, uint64_t pro)
{
    gen |= pro & (gen >> 1);
    pro &= pro >> 1;
    gen |= pro & (gen >> 2);
    pro &= pro >> 2;
    gen |= pro & (gen >> 4);
    pro &= pro >> 4;
    gen |= pro & (gen >> 8);
    pro &= pro >> 8;
    gen |= pro & (gen >> 16);
    pro &= pro >> 16;
    gen |= pro & (gen >> 32);
    return gen;
}

__global__ __launch_bounds__(kBlock) void k_sweep_x(const uint64_t *__restrict__ F,
                                                    uint64_t *__restrict__ O, TsdfGrid g, int W,
                                                    int32_t *__restrict__ changed,
                                                    const int32_t *__restrict__ skip)
{
    // a round enqueued after the labelling settled does nothing
    if (skip && *skip == 0) return;

    const int64_t row = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (row >= (int64_t)g.ny * g.nz) return;
    const uint64_t *f = F + row * W;
    uint64_t *o = O + row * W;
    const int top = (g.nx - 1) & 63;                      // last voxel's bit in the last word
    bool any = false;
    uint64_t carry = 1;                                   // the frame before x = 0
    for (int wx = 0; wx < W; ++wx) {
        const uint64_t fw = f[wx], ow = o[wx];
        const uint64_t gen = fill_up(ow | (fw & carry), fw);
        if (gen != ow) {
            o[wx] = gen;
            any = true;
        }
        carry = gen >> 63;
    }
    carry = 1;                                            // the frame after x = nx - 1
    for (int wx = W - 1; wx >= 0; --wx) {
        const uint64_t fw = f[wx], ow = o[wx];
        const uint64_t seed = carry ? (fw & (1ull << (wx == W - 1 ? top : 63))) : 0ull;
        const uint64_t gen = fill_down(ow | seed, fw);
        if (gen != ow) {
            o[wx] = gen;
            any = true;
        }
        carry = gen & 1ull;
    }
    if (any && *changed == 0) *changed = 1;
}

// The x and y sweeps of a whole z-slice in one launch, one block per slice: a
// thread reads its rows' words, sweeps them in registers and leaves them in
// LDS; then a wave takes a word column and each lane consecutive rows of it,
// carries between lanes being a scan of (reach, free throughout) pairs.  F and
// O are read once (apart: 16 us a round on 512 x 412 x 162 voxels, now
// 11 us; bound by the chain load - sweep - scan - sweep of a block).  WORDS: a
// slice's place in LDS.  Slices of up to kSliceSmall words run four blocks a
// CU, where one at a time leaves most of its waves to the chain (512 x 256 x
// 2,048 voxels, noise: 3,073 us a TSDF call with one, 2,715 with four).
// Repeating both sweeps in LDS until the slice settled took 75 us in the first
// round and saved two rounds of seven: what blocks a slice's fill is passed
// in z.
//
// A row's fill upwards is an addition: in f + seeds a seed's carry runs
// through the free bits above it and clears them ((f + s) ^ f) & f, apart
// from the seeds it meets); downwards the same on reversed words.
constexpr int kSliceWords = 9216;     // 2 x 72 KB of LDS
constexpr int kSliceSmall = 2304;     // 2 x 18 KB
constexpr int kSliceBlock = 512;

__device__ __forceinline__ uint64_t row_fill_up(uint64_t f, uint64_t s)
{
    return (((f + s) ^ f) & f) | s;
}

// rows of a slice are an odd number of words apart, and a lane's rows an odd
// number: lanes hit different banks
inline __host__ __device__ int slice_pitch(int W) { return W | 1; }

template <int WORDS>
__global__ __launch_bounds__(kSliceBlock) void k_sweep_slice(const uint64_t *__restrict__ Fg,
                                                             uint64_t *__restrict__ Og, TsdfGrid g,
                                                             int W, int32_t *__restrict__ changed,
                                                             const int32_t *__restrict__ skip)
{
    // a round enqueued after the labelling settled does nothing
    if (skip && *skip == 0) return;
    constexpr int kRun = 8, kRows = 9;    // words of a row, rows of a column, read together
    __shared__ uint64_t F[WORDS], O[WORDS];
    const int P = slice_pitch(W);
    const int64_t base = (int64_t)blockIdx.x * g.ny * W;
    const int top = (g.nx - 1) & 63;                      // last voxel's bit in the last word
    bool any = false;
    for (int y = threadIdx.x; y < g.ny; y += kSliceBlock) {
        uint64_t f[kRun], o[kRun], was[kRun], carry = 1;  // the frame before x = 0
        auto down = [&](int n) {
#pragma unroll
            for (int k = kRun - 1; k >= 0; --k)
                if (k < n) {
                    const uint64_t fr = __brevll(f[k]);
                    const uint64_t gen = row_fill_up(fr, __brevll(o[k]) | (fr & carry));
                    o[k] = __brevll(gen);
                    carry = gen >> 63;
                }
        };
        for (int c0 = 0; c0 < W; c0 += kRun) {
            const int n = W - c0 < kRun ? W - c0 : kRun;
            const uint64_t *fp = Fg + base + (int64_t)y * W + c0, *op = Og + base + (int64_t)y * W + c0;
#pragma unroll
            for (int k = 0; k < kRun; ++k)
                if (k < n) {
                    f[k] = fp[k];
                    o[k] = was[k] = op[k];
                }
#pragma unroll
            for (int k = 0; k < kRun; ++k)
                if (k < n) {
                    o[k] = row_fill_up(f[k], o[k] | (f[k] & carry));
                    carry = o[k] >> 63;
                }
            if (c0 + kRun >= W) {
                carry = 1ull << (63 - top);               // the frame after x = nx - 1
                down(n);
            }
#pragma unroll
            for (int k = 0; k < kRun; ++k)
                if (k < n) {
                    F[y * P + c0 + k] = f[k];
                    O[y * P + c0 + k] = o[k];
                    any |= o[k] != was[k];
                }
        }
        for (int c0 = (W - 1) / kRun * kRun - kRun; c0 >= 0; c0 -= kRun) {
#pragma unroll
            for (int k = 0; k < kRun; ++k) {
                f[k] = F[y * P + c0 + k];
                o[k] = was[k] = O[y * P + c0 + k];
            }
            down(kRun);
#pragma unroll
            for (int k = 0; k < kRun; ++k) {
                O[y * P + c0 + k] = o[k];
                any |= o[k] != was[k];
            }
        }
    }
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63);
    const int rs = ((g.ny + 63) / 64) | 1, r0 = lane * rs;
    const int r1 = r0 + rs < g.ny ? r0 + rs : g.ny;
    for (int c = (int)threadIdx.x >> 6; c < W; c += kSliceBlock / 64) {
        uint64_t f[kRows], o[kRows], was[kRows];
        // rows outside the lane's or the slice: free, nothing outside
        auto load = [&](int q) {
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const bool in = r0 + q + k < r1;
                f[k] = in ? F[(r0 + q + k) * P + c] : ~0ull;
                o[k] = was[k] = in ? O[(r0 + q + k) * P + c] : 0ull;
            }
        };
        auto store = [&](int q) {
#pragma unroll
            for (int k = 0; k < kRows; ++k)
                if (r0 + q + k < r1 && o[k] != was[k]) {
                    O[(r0 + q + k) * P + c] = o[k];
                    any = true;
                }
        };
        uint64_t a = 0, b = 0, t = ~0ull;                 // reach out of the end, of the start
        for (int q = 0; q < rs; q += kRows) {
            load(q);
            uint64_t bq = 0, tq = ~0ull;
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                a = f[k] & (a | o[k]);
                tq &= f[k];
            }
#pragma unroll
            for (int k = kRows - 1; k >= 0; --k) bq = f[k] & (bq | o[k]);
            b |= t & bq;
            t &= tq;
        }
        uint64_t ta = t, tb = t;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t pa = __shfl_up(a, d, 64), pt = __shfl_up(ta, d, 64);
            const uint64_t qb = __shfl_down(b, d, 64), qt = __shfl_down(tb, d, 64);
            if (lane >= d) {
                a |= ta & pa;
                ta &= pt;
            }
            if (lane + d < 64) {
                b |= tb & qb;
                tb &= qt;
            }
        }
        // the frame is outside at both ends
        uint64_t up = __shfl_up(a | ta, 1, 64), dn = __shfl_down(b | tb, 1, 64);
        if (lane == 0) up = ~0ull;
        if (lane == 63) dn = ~0ull;
        for (int q = 0; q < rs; q += kRows) {
            if (rs > kRows) load(q);
#pragma unroll
            for (int k = 0; k < kRows; ++k) o[k] = up = f[k] & (up | o[k]);
            if (rs > kRows) store(q);
        }
        for (int q = (rs - 1) / kRows * kRows; q >= 0; q -= kRows) {
            if (rs > kRows) load(q);
#pragma unroll
            for (int k = kRows - 1; k >= 0; --k) o[k] = dn = f[k] & (dn | o[k]);
            store(q);
        }
    }
    if (!__syncthreads_or(any)) return;
    for (int i = threadIdx.x; i < W * g.ny; i += kSliceBlock) Og[base + i] = O[i / W * P + i % W];
    if (threadIdx.x == 0 && *changed == 0) *changed = 1;
}

// The whole labelling of a small grid by one block, its words in LDS: rounds of
// x, y and z sweeps until y and z change nothing.  A row is a thread's; a column
// is cut into runs of kLabelRun words held in registers by neighbouring lanes,
// whose effects (what reaches the far end from the near end, and what starts
// outside within) are composed by a scan over the lanes.  Slices start at odd
// words, so that runs along z fall on different banks.  Bound by a round's chain,
// three sweeps with barriers, about 5 us: 39 us on 350,200 voxels, where a round
// in two launches takes 11 and a flag's way to the host 25.  (A column a thread's
// took 63 and lost to the launches on columns of 96 rows and more.)
constexpr int kLabelBlock = 1024, kLabelRun = 9, kLabelColumn = 64 * kLabelRun;

// Rows at + k * stride, k < n (n <= kLabelRun), of the run `part` of S lanes of
// a column: outside spreads along free words from what is outside and from the
// frame at both ends.  Rows past n are taken as free: they pass on what comes.
__device__ __forceinline__ bool sweep_run(const uint64_t *F, uint64_t *O, int at, int stride,
                                          int n, int part, int S)
{
    uint64_t f[kLabelRun], o[kLabelRun], r = 0, p = ~0ull, moved = 0;
#pragma unroll
    for (int k = 0; k < kLabelRun; ++k) {
        const int a = k < n ? at + k * stride : 0;
        const uint64_t fk = F[a], ok = O[a];
        f[k] = k < n ? fk : ~0ull;
        o[k] = k < n ? ok : 0ull;
        r = f[k] & (r | o[k]);
        p &= f[k];
    }
    for (int d = 1; d < S; d *= 2) {
        const uint64_t rb = __shfl_up(r, d, S), pb = __shfl_up(p, d, S);
        if (part >= d) {
            r |= p & rb;
            p &= pb;
        }
    }
    r = __shfl_up(r | p, 1, S);
    if (part == 0) r = ~0ull;
#pragma unroll
    for (int k = 0; k < kLabelRun; ++k) {
        r = f[k] & (r | o[k]);
        if (k < n) moved |= r ^ o[k];
        o[k] = r;
    }
    r = 0;
    p = ~0ull;
#pragma unroll
    for (int k = kLabelRun - 1; k >= 0; --k) {
        r = f[k] & (r | o[k]);
        p &= f[k];
    }
    for (int d = 1; d < S; d *= 2) {
        const uint64_t rb = __shfl_down(r, d, S), pb = __shfl_down(p, d, S);
        if (part + d < S) {
            r |= p & rb;
            p &= pb;
        }
    }
    r = __shfl_down(r | p, 1, S);
    if (part == S - 1) r = ~0ull;
#pragma unroll
    for (int k = kLabelRun - 1; k >= 0; --k) {
        r = f[k] & (r | o[k]);
        if (k < n) moved |= r ^ o[k];
        o[k] = r;
    }
    if (!moved) return false;
#pragma unroll
    for (int k = 0; k < kLabelRun; ++k)
        if (k < n) O[at + k * stride] = o[k];
    return true;
}

// lanes a column of n rows, as a shift
__host__ __device__ inline int label_lanes_log2(int n)
{
    int s = 0;
    while ((kLabelRun << s) < n) ++s;
    return s;
}

__host__ __device__ inline int label_pitch(const TsdfGrid &g, int W) { return (W * g.ny) | 1; }

__global__ __launch_bounds__(kLabelBlock) void k_label_small(const uint64_t *__restrict__ Fg,
                                                             uint64_t *__restrict__ Og, TsdfGrid g,
                                                             int W)
{
    __shared__ uint64_t F[kSliceWords], O[kSliceWords];
    const int slice = W * g.ny, pitch = label_pitch(g, W), nw = slice * g.nz, rows = g.ny * g.nz;
    for (int i = threadIdx.x; i < nw; i += kLabelBlock) {
        const int at = i + i / slice * (pitch - slice);
        F[at] = Fg[i];
        O[at] = 0;
    }
    __syncthreads();
    const uint64_t last = 1ull << (63 - ((g.nx - 1) & 63));   // the frame after x = nx - 1, reversed
    const int sy = label_lanes_log2(g.ny), sz = label_lanes_log2(g.nz);
    for (;;) {
        for (int row = threadIdx.x; row < rows; row += kLabelBlock) {
            const int z = row / g.ny, first = z * pitch + (row - z * g.ny) * W;
            uint64_t carry = 1;                               // the frame before x = 0
            for (int i = first; i < first + W; ++i) {
                const uint64_t f = F[i], o = O[i], n = row_fill_up(f, o | (f & carry));
                if (n != o) O[i] = n;
                carry = n >> 63;
            }
            carry = last;
            for (int i = first + W - 1; i >= first; --i) {
                const uint64_t f = __brevll(F[i]), o = __brevll(O[i]);
                const uint64_t n = row_fill_up(f, o | (f & carry));
                if (n != o) O[i] = __brevll(n);
                carry = n >> 63;
            }
        }
        __syncthreads();
        bool moved = false;
        for (int i = threadIdx.x; i < (W * g.nz) << sy; i += kLabelBlock) {
            const int c = i >> sy, part = i & ((1 << sy) - 1), k0 = part * kLabelRun, z = c / W;
            moved |= sweep_run(F, O, z * pitch + c - z * W + k0 * W, W, g.ny - k0, part, 1 << sy);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < slice << sz; i += kLabelBlock) {
            const int c = i >> sz, part = i & ((1 << sz) - 1), k0 = part * kLabelRun;
            moved |= sweep_run(F, O, c + k0 * pitch, pitch, g.nz - k0, part, 1 << sz);
        }
        // rows hold since their sweep if neither moved anything
        if (!__syncthreads_or(moved)) break;
    }
    for (int i = threadIdx.x; i < nw; i += kLabelBlock)
        Og[i] = O[i + i / slice * (pitch - slice)];
}

// word-column layout of a sweep along y (AXIS 1) or z (AXIS 2): column c,
// row r -> word base + r * stride; rows = ny or nz
struct Cols {
    int64_t ncols, stride;
    int rows, nseg;
};

template <int AXIS>
__device__ __forceinline__ int64_t col_base(int64_t c, const TsdfGrid &g, int W)
{
    const int64_t a = c / W, wx = c - a * W;
    return AXIS == 1 ? a * g.ny * W + wx      // a = z
                     : a * W + wx;            // a = y
}

// (1) per segment: A = reach out of its end, B = reach out of its start
// (from its own outside voxels), T = lines free on every row
template <int AXIS>
__global__ __launch_bounds__(kBlock) void k_seg_summary(const uint64_t *__restrict__ F,
                                                        const uint64_t *__restrict__ O,
                                                        TsdfGrid g, int W, Cols cl,
                                                        uint64_t *__restrict__ A,
                                                        uint64_t *__restrict__ B,
                                                        uint64_t *__restrict__ T,
                                                        const int32_t *__restrict__ skip)
{
    // a round enqueued after the labelling settled does nothing
    if (skip && *skip == 0) return;

    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= cl.ncols * cl.nseg) return;
    const int sg = (int)(t / cl.ncols);
    const int64_t c = t - (int64_t)sg * cl.ncols;
    const int64_t base = col_base<AXIS>(c, g, W);
    const int r0 = sg * kSegRows;
    const int nr = cl.rows - r0 < kSegRows ? cl.rows - r0 : kSegRows;
    uint64_t f[kSegRows], o[kSegRows];
#pragma unroll
    for (int k = 0; k < kSegRows; ++k) {
        f[k] = k < nr ? F[base + (int64_t)(r0 + k) * cl.stride] : 0ull;
        o[k] = k < nr ? O[base + (int64_t)(r0 + k) * cl.stride] : 0ull;
    }
    uint64_t r = 0, tr = ~0ull;
#pragma unroll
    for (int k = 0; k < kSegRows; ++k)
        if (k < nr) {
            r = f[k] & (r | o[k]);
            tr &= f[k];
        }
    uint64_t rb = 0;
#pragma unroll
    for (int k = kSegRows - 1; k >= 0; --k)
        if (k < nr) rb = f[k] & (rb | o[k]);
    A[t] = r;
    B[t] = rb;
    T[t] = tr;
}

// (2) per column: carries into each segment, C from the start side (the
// frame before row 0), D from the end side (the frame after the last row)
__global__ __launch_bounds__(kBlock) void k_seg_carry(const uint64_t *__restrict__ A,
                                                      const uint64_t *__restrict__ B,
                                                      const uint64_t *__restrict__ T, Cols cl,
                                                      uint64_t *__restrict__ C,
                                                      uint64_t *__restrict__ D,
                                                      const int32_t *__restrict__ skip)
{
    // a round enqueued after the labelling settled does nothing
    if (skip && *skip == 0) return;

    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c >= cl.ncols) return;
    // 8 segments' summaries are loaded together, then chained in registers
    // (one dependent load per segment left the walk latency-bound)
    constexpr int G = 8;
    uint64_t carry = ~0ull;
    for (int s0 = 0; s0 < cl.nseg; s0 += G) {
        uint64_t a[G], t[G];
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int64_t i = (int64_t)(s0 + k) * cl.ncols + c;
            a[k] = s0 + k < cl.nseg ? A[i] : 0ull;
            t[k] = s0 + k < cl.nseg ? T[i] : 0ull;
        }
#pragma unroll
        for (int k = 0; k < G; ++k)
            if (s0 + k < cl.nseg) {
                C[(int64_t)(s0 + k) * cl.ncols + c] = carry;
                carry = a[k] | (t[k] & carry);
            }
    }
    carry = ~0ull;
    for (int s1 = cl.nseg - 1; s1 >= 0; s1 -= G) {
        uint64_t b[G], t[G];
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int64_t i = (int64_t)(s1 - k) * cl.ncols + c;
            b[k] = s1 - k >= 0 ? B[i] : 0ull;
            t[k] = s1 - k >= 0 ? T[i] : 0ull;
        }
#pragma unroll
        for (int k = 0; k < G; ++k)
            if (s1 - k >= 0) {
                D[(int64_t)(s1 - k) * cl.ncols + c] = carry;
                carry = b[k] | (t[k] & carry);
            }
    }
}

// (3) per segment: forward from C, backward from D, new outside bits out
template <int AXIS>
__global__ __launch_bounds__(kBlock) void k_seg_apply(const uint64_t *__restrict__ F,
                                                      uint64_t *__restrict__ O, TsdfGrid g,
                                                      int W, Cols cl,
                                                      const uint64_t *__restrict__ C,
                                                      const uint64_t *__restrict__ D,
                                                      int32_t *__restrict__ changed,
                                                      const int32_t *__restrict__ skip)
{
    // a round enqueued after the labelling settled does nothing
    if (skip && *skip == 0) return;

    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= cl.ncols * cl.nseg) return;
    const int sg = (int)(t / cl.ncols);
    const int64_t c = t - (int64_t)sg * cl.ncols;
    const int64_t base = col_base<AXIS>(c, g, W);
    const int r0 = sg * kSegRows;
    const int nr = cl.rows - r0 < kSegRows ? cl.rows - r0 : kSegRows;
    uint64_t f[kSegRows], o[kSegRows], o0[kSegRows];
#pragma unroll
    for (int k = 0; k < kSegRows; ++k) {
        f[k] = k < nr ? F[base + (int64_t)(r0 + k) * cl.stride] : 0ull;
        o[k] = k < nr ? O[base + (int64_t)(r0 + k) * cl.stride] : 0ull;
        o0[k] = o[k];
    }
    uint64_t r = C[t];
#pragma unroll
    for (int k = 0; k < kSegRows; ++k)
        if (k < nr) {
            r = f[k] & (r | o[k]);
            o[k] = r;
        }
    r = D[t];
#pragma unroll
    for (int k = kSegRows - 1; k >= 0; --k)
        if (k < nr) {
            r = f[k] & (r | o[k]);
            o[k] = r;
        }
    bool any = false;
#pragma unroll
    for (int k = 0; k < kSegRows; ++k)
        if (k < nr && o[k] != o0[k]) {
            O[base + (int64_t)(r0 + k) * cl.stride] = o[k];
            any = true;
        }
    if (any && *changed == 0) *changed = 1;
}

// (1) to (3) in one kernel, for columns of at most kFusedSegs segments: a
// block takes cj adjacent columns (threads column-fastest, so the words of
// one row are read together; cj * nseg <= kBlock), keeps each segment's
// words in registers, and one thread per column chains the summaries
// through LDS into the carries; the same recurrences as the three kernels,
// without two launches and the summary and carry arrays.
constexpr int kFusedSegs = 32;

template <int AXIS>
__global__ __launch_bounds__(kBlock) void k_seg_fused(const uint64_t *__restrict__ F,
                                                      uint64_t *__restrict__ O, TsdfGrid g,
                                                      int W, Cols cl, int cj,
                                                      int32_t *__restrict__ changed,
                                                      const int32_t *__restrict__ skip)
{
    // a round enqueued after the labelling settled does nothing
    if (skip && *skip == 0) return;

    __shared__ uint64_t sA[kBlock], sB[kBlock], sT[kBlock];
    const int j = (int)threadIdx.x % cj, sg = (int)threadIdx.x / cj;
    const int64_t c = (int64_t)blockIdx.x * cj + j;
    const bool act = sg < cl.nseg && c < cl.ncols;
    const int64_t base = act ? col_base<AXIS>(c, g, W) : 0;
    const int r0 = sg * kSegRows;
    const int nr = !act ? 0 : (cl.rows - r0 < kSegRows ? cl.rows - r0 : kSegRows);
    uint64_t f[kSegRows], o[kSegRows], o0[kSegRows];
#pragma unroll
    for (int k = 0; k < kSegRows; ++k) {
        f[k] = k < nr ? F[base + (int64_t)(r0 + k) * cl.stride] : 0ull;
        o[k] = k < nr ? O[base + (int64_t)(r0 + k) * cl.stride] : 0ull;
        o0[k] = o[k];
    }
    // summary: reach out of the end, out of the start, free throughout
    uint64_t r = 0, tr = ~0ull;
#pragma unroll
    for (int k = 0; k < kSegRows; ++k)
        if (k < nr) {
            r = f[k] & (r | o[k]);
            tr &= f[k];
        }
    uint64_t rb = 0;
#pragma unroll
    for (int k = kSegRows - 1; k >= 0; --k)
        if (k < nr) rb = f[k] & (rb | o[k]);
    sA[threadIdx.x] = r;
    sB[threadIdx.x] = rb;
    sT[threadIdx.x] = tr;
    __syncthreads();
    // carries, in place of the summaries: threads 0 .. cj - 1 are column j
    // of segment 0
    if ((int)threadIdx.x < cj && c < cl.ncols) {
        uint64_t carry = ~0ull;                           // the frame before row 0
        for (int q = 0; q < cl.nseg; ++q) {
            const int i = q * cj + j;
            const uint64_t a = sA[i];
            sA[i] = carry;
            carry = a | (sT[i] & carry);
        }
        carry = ~0ull;                                    // the frame after the last row
        for (int q = cl.nseg - 1; q >= 0; --q) {
            const int i = q * cj + j;
            const uint64_t b = sB[i];
            sB[i] = carry;
            carry = b | (sT[i] & carry);
        }
    }
    __syncthreads();
    if (!act) return;
    r = sA[threadIdx.x];
#pragma unroll
    for (int k = 0; k < kSegRows; ++k)
        if (k < nr) {
            r = f[k] & (r | o[k]);
            o[k] = r;
        }
    r = sB[threadIdx.x];
#pragma unroll
    for (int k = kSegRows - 1; k >= 0; --k)
        if (k < nr) {
            r = f[k] & (r | o[k]);
            o[k] = r;
        }
    bool any = false;
#pragma unroll
    for (int k = 0; k < kSegRows; ++k)
        if (k < nr && o[k] != o0[k]) {
            O[base + (int64_t)(r0 + k) * cl.stride] = o[k];
            any = true;
        }
    if (any && *changed == 0) *changed = 1;
}

// the four bytes at any offset, from two aligned words
__device__ __forceinline__ uint32_t word_at(const uint8_t *__restrict__ p, int64_t idx)
{
    const int64_t a = idx & ~(int64_t)3;
    const uint32_t lo = *reinterpret_cast<const uint32_t *>(p + a);
    const int sh = (int)(idx & 3);
    if (sh == 0) return lo;
    const uint32_t hi = *reinterpret_cast<const uint32_t *>(p + a + 4);
    return __builtin_amdgcn_alignbyte(hi, lo, (uint32_t)sh);
}

__device__ __forceinline__ uint32_t byte_of(uint32_t w, int j) { return (w >> (8 * j)) & 0xffu; }

__device__ __forceinline__ void step_voxel(const TsdfGrid &g, int &x, int &y, int &z)
{
    if (++x == g.nx) {
        x = 0;
        if (++y == g.ny) {
            y = 0;
            ++z;
        }
    }
}

// ---- distance shells and phi -----------------------------------------------

// p = 0 on S_0 (a 6-neighbour with the other V~ value; outside the grid is
// 0), else 255 (not reached)
// bytes idx .. idx + 3 of p[0, n) (0 outside it), p 4-byte aligned: two
// aligned words where they lie inside the buffer, bytes near its ends
__device__ __forceinline__ uint32_t word_any(const uint8_t *__restrict__ p, int64_t idx, int64_t n)
{
    const int64_t a = idx & ~(int64_t)3;
    if (a >= 0 && a + 8 <= n) {
        const uint32_t lo = *reinterpret_cast<const uint32_t *>(p + a);
        const int sh = (int)(idx & 3);
        if (sh == 0) return lo;
        const uint32_t hi = *reinterpret_cast<const uint32_t *>(p + a + 4);
        return __builtin_amdgcn_alignbyte(hi, lo, (uint32_t)sh);
    }
    uint32_t w = 0;
    for (int j = 0; j < 4; ++j) {
        const int64_t q = idx + j;
        if (q >= 0 && q < n) w |= (uint32_t)p[q] << (8 * j);
    }
    return w;
}

// p = 0 on S_0 (a 6-neighbour with the other V~ value; outside the grid is
// 0), else 255 (not reached).  Four voxels per thread (V~ 4-byte aligned:
// word loads; p has the shell kernel's padding).
__global__ __launch_bounds__(kBlock) void k_shell0(const uint8_t *__restrict__ vt,
                                                   uint8_t *__restrict__ p, TsdfGrid g)
{
    const int64_t i0 = 4 * ((int64_t)blockIdx.x * kBlock + threadIdx.x);
    if (i0 >= g.n) return;
    const int64_t sxy = (int64_t)g.nx * g.ny;
    const uint32_t c = word_any(vt, i0, g.n);
    const uint32_t xm = word_any(vt, i0 - 1, g.n), xp = word_any(vt, i0 + 1, g.n);
    const uint32_t ym = word_any(vt, i0 - g.nx, g.n), yp = word_any(vt, i0 + g.nx, g.n);
    const uint32_t zm = word_any(vt, i0 - sxy, g.n), zp = word_any(vt, i0 + sxy, g.n);
    int x, y, z;
    coords(i0, g, x, y, z);
    uint32_t out = 0;
    for (int j = 0; j < 4; ++j) {
        const uint32_t cj = byte_of(c, j);
        const bool edge = (x > 0 ? byte_of(xm, j) : 0u) != cj ||
                          (x < g.nx - 1 ? byte_of(xp, j) : 0u) != cj ||
                          (y > 0 ? byte_of(ym, j) : 0u) != cj ||
                          (y < g.ny - 1 ? byte_of(yp, j) : 0u) != cj ||
                          (z > 0 ? byte_of(zm, j) : 0u) != cj ||
                          (z < g.nz - 1 ? byte_of(zp, j) : 0u) != cj;
        out |= (edge ? 0u : 255u) << (8 * j);
        step_voxel(g, x, y, z);
    }
    *reinterpret_cast<uint32_t *>(p + i0) = out;
}

// the same, one voxel per thread (V~ not 4-byte aligned)
__global__ __launch_bounds__(kBlock) void k_shell0_1(const uint8_t *__restrict__ vt,
                                                     uint8_t *__restrict__ p, TsdfGrid g)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.n) return;
    int x, y, z;
    coords(i, g, x, y, z);
    const int64_t sxy = (int64_t)g.nx * g.ny;
    const uint8_t c = vt[i];
    const uint8_t nb[6] = {x > 0 ? vt[i - 1] : (uint8_t)0, x < g.nx - 1 ? vt[i + 1] : (uint8_t)0,
                           y > 0 ? vt[i - g.nx] : (uint8_t)0,
                           y < g.ny - 1 ? vt[i + g.nx] : (uint8_t)0,
                           z > 0 ? vt[i - sxy] : (uint8_t)0, z < g.nz - 1 ? vt[i + sxy] : (uint8_t)0};
    bool edge = false;
    for (int k = 0; k < 6; ++k) edge |= nb[k] != c;
    p[i] = edge ? 0 : 255;
}

// Shell m: the unreached voxels (255) with a 6-neighbour in shell m - 1.
// Four voxels per thread as one aligned word: byte-wide loads, one per lane
// and neighbour, capped the one-voxel form at the rate the memory pipeline
// issues instructions.  Neighbour words at any byte offset are put together
// from two aligned words; `p` has kShellPad bytes of readable padding on
// both sides, so every load stays inside the buffer (bytes outside the grid
// are never used: the coordinate tests exclude them).  Voxels written in
// this pass go from 255 to m, neither of which is m - 1, so a neighbour
// read before or after the write gives the same answer; no two threads
// write the same word.

__global__ __launch_bounds__(kBlock) void k_shell(uint8_t *__restrict__ p, TsdfGrid g, int m)
{
    const int64_t i0 = 4 * ((int64_t)blockIdx.x * kBlock + threadIdx.x);
    if (i0 >= g.n) return;
    const uint32_t c = *reinterpret_cast<const uint32_t *>(p + i0);
    int live = 0;
    for (int j = 0; j < 4; ++j)
        if (i0 + j < g.n && byte_of(c, j) == 255u) live |= 1 << j;
    if (!live) return;
    const int64_t sxy = (int64_t)g.nx * g.ny;
    const uint32_t prev = (uint32_t)(m - 1);
    const uint32_t wl = *reinterpret_cast<const uint32_t *>(p + i0 - 4);
    const uint32_t wr = *reinterpret_cast<const uint32_t *>(p + i0 + 4);
    const uint32_t xm = __builtin_amdgcn_alignbyte(c, wl, 3u);   // bytes i0 - 1 + j
    const uint32_t xp = __builtin_amdgcn_alignbyte(wr, c, 1u);   // bytes i0 + 1 + j
    const uint32_t ym = word_at(p, i0 - g.nx), yp = word_at(p, i0 + g.nx);
    const uint32_t zm = word_at(p, i0 - sxy), zp = word_at(p, i0 + sxy);
    uint32_t out = c;
    for (int j = 0; j < 4; ++j) {
        if (!((live >> j) & 1)) continue;
        int x, y, z;
        coords(i0 + j, g, x, y, z);
        const bool hit = (x > 0 && byte_of(xm, j) == prev) ||
                         (x < g.nx - 1 && byte_of(xp, j) == prev) ||
                         (y > 0 && byte_of(ym, j) == prev) ||
                         (y < g.ny - 1 && byte_of(yp, j) == prev) ||
                         (z > 0 && byte_of(zm, j) == prev) ||
                         (z < g.nz - 1 && byte_of(zp, j) == prev);
        if (hit) out = (out & ~(0xffu << (8 * j))) | ((uint32_t)m << (8 * j));
    }
    if (out != c) *reinterpret_cast<uint32_t *>(p + i0) = out;
}

// S_0, the P <= 4 shells and phi in one pass on bits.  A block owns one word
// by 16 x 16 rows and holds it with a halo of P + 1 rows in y and z; the 32
// voxels before the word and the 32 after it share a second word (halo: bits
// 0..31 and 32..63), so a step of one voxel is two words a row.  A halo's
// outer end is wrong one voxel further in after each step, and a step leaves
// out one more row of the halo: after P + 1 steps the block's own words are
// right.  R_m, the voxels within m shells, is R_(m-1) and its neighbours; the
// shell index is the number of m <= P with the voxel outside R_m, counted
// bit-sliced, and each row's phi is chosen from its P + 2 values and their
// negatives by those words as lane masks.  phi comes from the same
// operations as k_phi's: the same bits.  Bound by phi's stores: 49 us on
// 34.2M voxels at P = 3 (bytes in LDS, four voxels a word: 220 us).
constexpr int kShY = 16, kShZ = 16;

template <int P>
__global__ __launch_bounds__(kBlock) void k_shells_phi_bits(const uint64_t *__restrict__ F,
                                                            const uint64_t *__restrict__ O,
                                                            float *__restrict__ phi, TsdfGrid g,
                                                            int W, float h, float r,
                                                            const int32_t *__restrict__ unsettled)
{
    static_assert(P >= 1 && P <= 4 && P + 1 < 31, "halo of 32 voxels in x");
    static_assert(kShY * kShZ == kBlock && kShY == 16, "a row a thread");
    constexpr int H = P + 1, LY = kShY + 2 * H, LZ = kShZ + 2 * H;
    __shared__ uint64_t C[2][LY * LZ], E[2][LY * LZ];
    const uint32_t tile = xcd_tile(), ty = (uint32_t)(g.ny + kShY - 1) / kShY;
    const int bx = (int)(tile % (uint32_t)W), by = (int)(tile / (uint32_t)W % ty) * kShY;
    const int bz = (int)(tile / (uint32_t)W / ty) * kShZ;
    if (bz >= g.nz || (unsettled && *unsettled)) return;
    const uint64_t last = ~0ull >> (63 - ((g.nx - 1) & 63));   // the last word's voxels
    const uint64_t mc = bx == W - 1 ? last : ~0ull;
    const uint64_t mr = bx + 1 < W ? (bx + 1 == W - 1 ? last : ~0ull) : 0ull;
    const uint64_t me = (bx > 0 ? 0xffffffffull : 0ull) | (mr << 32);
    for (int q = threadIdx.x; q < LY * LZ; q += kBlock) {
        const int gy = by - H + q % LY, gz = bz - H + q / LY;
        uint64_t c = 0, e = 0;                                 // V~, 0 outside the grid
        if (gy >= 0 && gy < g.ny && gz >= 0 && gz < g.nz) {
            const uint64_t *f = F + ((int64_t)gz * g.ny + gy) * W + bx;
            c = mc & ~f[0];
            e = (bx > 0 ? ~f[-1] >> 32 : 0ull) | (bx + 1 < W ? (mr & ~f[1]) << 32 : 0ull);
        }
        C[0][q] = c;
        E[0][q] = e;
    }
    const int gy = by + (int)threadIdx.x % kShY, gz = bz + (int)threadIdx.x / kShY;
    const uint64_t out = gy < g.ny && gz < g.nz ? O[((int64_t)gz * g.ny + gy) * W + bx] : 0ull;
    __syncthreads();
    uint64_t p0 = 0, p1 = 0, p2 = 0;
    const int own = ((int)threadIdx.x / kShY + H) * LY + (int)threadIdx.x % kShY + H;
#pragma unroll
    for (int m = 0; m <= P; ++m) {
        const int d = m + 1, ny = LY - 2 * d, n = ny * (LZ - 2 * d);
        const uint64_t *cs = C[m & 1], *es = E[m & 1];
        uint64_t *cd = C[(m & 1) ^ 1], *ed = E[(m & 1) ^ 1];
        for (int t = threadIdx.x; t < n; t += kBlock) {
            const int ly = d + t % ny, lz = d + t / ny, q = lz * LY + ly;
            const int y = by - H + ly, z = bz - H + lz;
            const bool in = y >= 0 && y < g.ny && z >= 0 && z < g.nz;
            const uint64_t c = cs[q], e = es[q];
            const uint64_t cm = (c << 1) | ((e >> 31) & 1ull), cp = (c >> 1) | (((e >> 32) & 1ull) << 63);
            const uint64_t em = ((e << 1) & ~(1ull << 32)) | ((c >> 63) << 32);
            const uint64_t ep = ((e >> 1) & ~(1ull << 31)) | ((c & 1ull) << 31);
            uint64_t cn, en;
            if (m == 0) {     // a 6-neighbour with the other V~
                cn = (c ^ cm) | (c ^ cp) | (c ^ cs[q - 1]) | (c ^ cs[q + 1]) | (c ^ cs[q - LY]) |
                     (c ^ cs[q + LY]);
                en = (e ^ em) | (e ^ ep) | (e ^ es[q - 1]) | (e ^ es[q + 1]) | (e ^ es[q - LY]) |
                     (e ^ es[q + LY]);
            } else {
                cn = c | cm | cp | cs[q - 1] | cs[q + 1] | cs[q - LY] | cs[q + LY];
                en = e | em | ep | es[q - 1] | es[q + 1] | es[q - LY] | es[q + LY];
            }
            cd[q] = in ? cn & mc : 0ull;
            ed[q] = in ? en & me : 0ull;
        }
        __syncthreads();
        const uint64_t add = ~cd[own], k0 = p0 & add, k1 = p1 & k0;
        p0 ^= add;
        p1 ^= k0;
        p2 |= k1;
    }
    float mag[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) mag[k] = k <= P ? fminf((float)k * h, r) : r;
    const int lane = (int)threadIdx.x & 63, w0 = (int)threadIdx.x & ~63, gx = 64 * bx + lane;
#pragma unroll 4
    for (int k = 0; k < 64; ++k) {
        const int y = by + (w0 + k) % kShY, z = bz + (w0 + k) / kShY;
        const bool b0 = lane_bit(read_lane64(p0, k)), b1 = lane_bit(read_lane64(p1, k));
        const bool b2 = lane_bit(read_lane64(p2, k)), bo = lane_bit(read_lane64(out, k));
        const float m01 = b0 ? mag[1] : mag[0], m23 = b0 ? mag[3] : mag[2];
        const float m45 = b0 ? mag[5] : mag[4];
        const float f = b2 ? m45 : b1 ? m23 : m01;
        if (y < g.ny && z < g.nz && gx < g.nx)
            phi[((int64_t)z * g.ny + y) * g.nx + gx] = bo ? f : -f;
    }
}

// phi = clip(s p h, -r, r); s = +1 where the packed outside bit is set.
// Four voxels per thread (p padded and aligned); one float4 store when phi
// is 16-byte aligned.
__global__ __launch_bounds__(kBlock) void k_phi(const uint8_t *__restrict__ p,
                                                const uint64_t *__restrict__ O,
                                                float *__restrict__ phi, TsdfGrid g, int W,
                                                float h, float r, int vec)
{
    const int64_t i0 = 4 * ((int64_t)blockIdx.x * kBlock + threadIdx.x);
    if (i0 >= g.n) return;
    const uint32_t pw = *reinterpret_cast<const uint32_t *>(p + i0);
    int x, y, z;
    coords(i0, g, x, y, z);
    float f[4];
    for (int j = 0; j < 4; ++j) {
        const uint32_t pj = byte_of(pw, j);
        bool out = false;
        if (i0 + j < g.n) out = (O[((int64_t)z * g.ny + y) * W + (x >> 6)] >> (x & 63)) & 1ull;
        const float delta = pj == 255u ? r : (float)pj * h;
        const float sg = out ? delta : -delta;
        f[j] = fminf(fmaxf(sg, -r), r);
        step_voxel(g, x, y, z);
    }
    if (vec && i0 + 4 <= g.n) {
        *reinterpret_cast<float4 *>(phi + i0) = make_float4(f[0], f[1], f[2], f[3]);
    } else {
        for (int j = 0; i0 + j < g.n && j < 4; ++j) phi[i0 + j] = f[j];
    }
}

__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t *total)
{
    __shared__ uint32_t ws[kBlock / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) ws[w] = x;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int k = 0; k < kBlock / 64; ++k) {
        if (k < w) off += ws[k];
        tot += ws[k];
    }
    __syncthreads();
    *total = tot;
    return off + x - v;
}

// ---- marching cubes --------------------------------------------------------
// Inside bits (phi < iso) packed 64 lattice points a word, in point order:
// word w holds points 64 w .. 64 w + 63, whatever rows they lie in.  A
// point's neighbours are then fixed bit offsets away (1, nx, nx ny), and
// crossed edges and active cells are word operations: the passes over the
// grid read phi once and a bit a point afterwards.  (One mask byte, one case
// byte and one 16-bit vertex offset a point, written, scanned and read again,
// took 137 + 35 + 26 us and 142 us in the emission on 34.2M points with 1.7M
// vertices; these take 26 + 21 + 8 us, the first at the rate of a copy, and
// 93 us.)
struct __align__(16) McWord {
    uint64_t e[3];    // points whose +x / +y / +z edge is crossed
    uint32_t v, t;    // vertices and triangles of the block's earlier words
};
constexpr int kMcWords = 256;   // words of a count block
constexpr uint32_t kMcGroup = 64, kMcMinWeight = 8;   // a group's weight and a word's least

// one wave a word: coalesced reads, a ballot packs; kMcInsideRun words a
// wave keep as many reads in flight
constexpr int kMcInsideRun = 8;

__global__ __launch_bounds__(kBlock) void k_mc_inside(const float *__restrict__ phi, int64_t n,
                                                      float iso, uint64_t *__restrict__ inside)
{
    const int lane = (int)(threadIdx.x & 63);
    const int64_t w0 = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * kMcInsideRun;
    float f[kMcInsideRun];
#pragma unroll
    for (int k = 0; k < kMcInsideRun; ++k) {
        const int64_t i = 64 * (w0 + k) + lane;
        f[k] = phi[i < n ? i : 0];
    }
#pragma unroll
    for (int k = 0; k < kMcInsideRun; ++k) {
        const int64_t i = 64 * (w0 + k) + lane;
        const uint64_t m = __ballot(i < n && f[k] < iso);
        if (lane == 0 && 64 * (w0 + k) < n) inside[w0 + k] = m;
    }
}

// inside bits of the points `off` beyond word w's (u), and one further (v)
__device__ __forceinline__ void corner_words(const uint64_t *__restrict__ inside, int64_t nw,
                                             int64_t w, int64_t off, uint64_t &u, uint64_t &v)
{
    const int64_t q = w + (off >> 6);
    const int sh = (int)(off & 63);
    const uint64_t lo = q < nw ? inside[q] : 0ull, hi = q + 1 < nw ? inside[q + 1] : 0ull;
    u = sh ? (lo >> sh) | (hi << (64 - sh)) : lo;
    v = (u >> 1) | (((hi >> sh) & 1ull) << 63);
}

// Points of word w that have a +x, +y, +z neighbour in the grid.
__device__ __forceinline__ void neighbour_masks(int64_t w, const TsdfGrid &g, uint64_t &mx,
                                                uint64_t &my, uint64_t &mz)
{
    const int64_t i0 = 64 * w, sxy = (int64_t)g.nx * g.ny;
    auto below = [&](int64_t end) -> uint64_t {   // points i < end
        const int64_t k = end - i0;
        return k <= 0 ? 0ull : (k >= 64 ? ~0ull : (1ull << k) - 1ull);
    };
    const uint64_t valid = below(g.n);
    mz = below(g.n - sxy) & valid;
    mx = valid;
    my = valid;
    int x, y, z;
    coords(i0, g, x, y, z);
    // row by row: the last point has no +x, the last row no +y
    for (int64_t start = i0 - x; start < i0 + 64; start += g.nx) {
        mx &= ~(below(start + g.nx) & ~below(start + g.nx - 1));
        if (y == g.ny - 1) my &= ~(below(start + g.nx) & ~below(start));
        y = y == g.ny - 1 ? 0 : y + 1;
    }
}

// Per word: its crossed edges and active cells, its vertices and triangles,
// and their offsets within the block of kMcWords words; the block's totals;
// the block's list of the words that have any.  Only listed words are written.
//
// The list falls into groups of words for the emission's waves: about 64
// vertices, at most 8 words.  (Surfaces that follow x have 64 vertices in a
// word, others 1 to 3: waves of 8 words each had from 10 to 1,500 items, and
// the last layers' waves ran long after the others, 136 us.)  A word weighs its
// vertices, but 8 to 64, and belongs to group [weight of the words before it
// / 64]: no group is empty.
__global__ __launch_bounds__(kMcWords) void k_mc_count(const uint64_t *__restrict__ inside,
                                                       TsdfGrid g, int64_t nw,
                                                       const uint8_t *__restrict__ ntri,
                                                       McWord *__restrict__ words,
                                                       uint64_t *__restrict__ cells,
                                                       uint8_t *__restrict__ list,
                                                       uint8_t *__restrict__ group,
                                                       uint32_t *__restrict__ nlist,
                                                       uint32_t *__restrict__ vsums,
                                                       uint32_t *__restrict__ tsums,
                                                       uint32_t *__restrict__ gsums)
{
    static_assert(kMcWords == kBlock, "the block scan's size, and a byte names a word");
    static_assert(kMcGroup * kMcWords < (1 << 15) && 5 * 64 * kMcWords < (1 << 17), "shared scan");
    __shared__ uint8_t nt_lds[256];
    nt_lds[threadIdx.x] = ntri[threadIdx.x];
    __syncthreads();
    const int64_t w = (int64_t)blockIdx.x * kMcWords + threadIdx.x;
    McWord m;
    m.e[0] = m.e[1] = m.e[2] = 0;
    uint64_t cell = 0;
    uint32_t nv = 0, nt = 0;
    if (w < nw) {
        uint64_t c[8], mx, my, mz;   // corner k = (k & 1, k >> 1 & 1, k >> 2 & 1)
        const int64_t sxy = (int64_t)g.nx * g.ny;
        corner_words(inside, nw, w, 0, c[0], c[1]);
        corner_words(inside, nw, w, g.nx, c[2], c[3]);
        corner_words(inside, nw, w, sxy, c[4], c[5]);
        corner_words(inside, nw, w, sxy + g.nx, c[6], c[7]);
        uint64_t any = c[0], all = c[0];
#pragma unroll
        for (int k = 1; k < 8; ++k) {
            any |= c[k];
            all &= c[k];
        }
        cell = any & ~all;
        if (cell) {                  // most words lie inside or outside
            neighbour_masks(w, g, mx, my, mz);
            m.e[0] = (c[0] ^ c[1]) & mx;
            m.e[1] = (c[0] ^ c[2]) & my;
            m.e[2] = (c[0] ^ c[4]) & mz;
            cell &= mx & my & mz;
            nv = (uint32_t)(__popcll(m.e[0]) + __popcll(m.e[1]) + __popcll(m.e[2]));
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                uint32_t todo = (uint32_t)(cell >> (32 * half));
                while (todo) {
                    const int b = __builtin_ctz(todo);
                    todo &= todo - 1;
                    uint32_t cs = 0;
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        cs |= (((uint32_t)(c[k] >> (32 * half)) >> b) & 1u) << k;
                    nt += nt_lds[cs];
                }
            }
        }
    }
    // vertices (at most 3 x 64 x 256 = 49,152 a block) and listed words
    // (at most 256) share a scan, triangles (81,920) and weights (16,384) one
    const uint32_t busy = nv + nt ? 1u : 0u;
    const uint32_t wt = !busy ? 0u : nv < kMcMinWeight ? kMcMinWeight : nv > kMcGroup ? kMcGroup : nv;
    uint32_t tv, tt;
    const uint32_t rv = block_scan_excl(nv | (busy << 16), &tv);
    const uint32_t rt = block_scan_excl(nt | (wt << 17), &tt);
    m.v = rv & 0xffffu;
    m.t = rt & 0x1ffffu;
    const uint32_t gi = (rt >> 17) / kMcGroup, li = rv >> 16;
    __shared__ uint16_t group_of[kMcWords];
    if (busy) {
        words[w] = m;
        cells[w] = cell;
        list[(int64_t)blockIdx.x * kMcWords + li] = (uint8_t)threadIdx.x;
        group_of[li] = (uint16_t)gi;
    }
    __syncthreads();
    if (busy && (li == 0 || group_of[li - 1] != gi))
        group[(int64_t)blockIdx.x * kMcWords + gi] = (uint8_t)li;      // its first word
    if (threadIdx.x == 0) {
        const uint32_t n = tv >> 16;
        vsums[blockIdx.x] = tv & 0xffffu;
        nlist[blockIdx.x] = n;
        tsums[blockIdx.x] = tt & 0x1ffffu;
        gsums[blockIdx.x] = n ? group_of[n - 1] + 1u : 0u;
    }
}

// Gradient of phi at a lattice point along one axis, phi per voxel:
// central difference halved inside, one-sided on the first and last point,
// 0 on an axis of size 1.  The two reads are split from the arithmetic and
// made unconditional (the point itself where a neighbour is missing), so
// that the twelve reads of a vertex's two gradients are all in flight
// before the first is used.
__device__ __forceinline__ void lattice_reads(const float *__restrict__ phi, int64_t i, int c,
                                              int n, int64_t step, float &a, float &b)
{
    a = phi[c < n - 1 ? i + step : i];
    b = phi[c > 0 ? i - step : i];
}

// the same operations as the three cases: phi[i+1] - phi[i] at c = 0,
// phi[i] - phi[i-1] at c = n - 1, (phi[i+1] - phi[i-1]) / 2 between
__device__ __forceinline__ float lattice_diff(float a, float b, int c, int n)
{
    const float d = __fsub_rn(a, b);
    if (n < 2) return 0.0f;
    return (c == 0 || c == n - 1) ? d : __fmul_rn(d, 0.5f);
}

// The vertex on edge `a` (0: +x, 1: +y, 2: +z) of lattice point i, into
// slot v: the crossing of iso by linear interpolation along the edge, and
// with normals the normalised interpolation of the lattice gradients at the
// edge's ends.
__device__ __forceinline__ void mc_emit_vertex(const float *__restrict__ phi, const TsdfGrid &g,
                                               float iso, float *__restrict__ verts,
                                               float *__restrict__ normals, int64_t i, int a,
                                               uint32_t v)
{
    int x, y, z;
    coords(i, g, x, y, z);
    const float c0 = (float)(g.o[0] + ((double)x + 0.5) * g.h);
    const float c1 = (float)(g.o[1] + ((double)y + 0.5) * g.h);
    const float c2 = (float)(g.o[2] + ((double)z + 0.5) * g.h);
    const int64_t sx = g.nx, sxy = (int64_t)g.nx * g.ny;
    const int64_t step = a == 0 ? 1 : (a == 1 ? sx : sxy);
    float fa, fb;
    // gradient reads at both ends of the edge, issued before any is used
    const int xb = x + (a == 0), yb = y + (a == 1), zb = z + (a == 2);
    float r[12];
    if (normals && x > 0 && x + 2 < g.nx) {
        // neighbours along x come with the same read (a lane's read costs a
        // cache lookup of its own wherever vertices are not x neighbours):
        // 5 or 8 reads for the 14 values
        const int64_t q = a == 0 ? i : i + step;
        float A[4], B[4], R[6][2];
        __builtin_memcpy(A, phi + i - 1, sizeof A);
        __builtin_memcpy(B, phi + q - 1, sizeof B);
        const int64_t yp = y < g.ny - 1 ? sx : 0, ym = y > 0 ? sx : 0;
        const int64_t zp = z < g.nz - 1 ? sxy : 0, zm = z > 0 ? sxy : 0;
        // x: i + y, i - y, i + z, i - z, both ends at once.  y (z): i - y,
        // then q + y, then +z and -z (y) at both ends; i + y is q
        const bool ez = a == 2;
        const int64_t qp = ez ? (zb < g.nz - 1 ? sxy : 0) : (yb < g.ny - 1 ? sx : 0);
        const int64_t om = ez ? zm : ym, sp = ez ? yp : zp, sm = ez ? ym : zm;
        __builtin_memcpy(R[0], phi + (a == 0 ? i + yp : q + qp), sizeof R[0]);
        __builtin_memcpy(R[1], phi + (a == 0 ? i - ym : i - om), sizeof R[1]);
        __builtin_memcpy(R[2], phi + (a == 0 ? i + zp : i + sp), sizeof R[2]);
        __builtin_memcpy(R[3], phi + (a == 0 ? i - zm : i - sm), sizeof R[3]);
        if (a != 0) {
            __builtin_memcpy(R[4], phi + q + sp, sizeof R[4]);
            __builtin_memcpy(R[5], phi + q - sm, sizeof R[5]);
        }
        fa = A[1];
        fb = a == 0 ? A[2] : B[1];
        r[0] = A[2];
        r[1] = A[0];
        r[6] = a == 0 ? A[3] : B[2];
        r[7] = a == 0 ? A[1] : B[0];
        if (a == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                r[2 + k] = R[k][0];
                r[8 + k] = R[k][1];
            }
        } else {
            const float ap = fb, am = R[1][0], bp = R[0][0], bm = fa;   // along the edge
            r[2] = ez ? R[2][0] : ap;
            r[3] = ez ? R[3][0] : am;
            r[4] = ez ? ap : R[2][0];
            r[5] = ez ? am : R[3][0];
            r[8] = ez ? R[4][0] : bp;
            r[9] = ez ? R[5][0] : bm;
            r[10] = ez ? bp : R[4][0];
            r[11] = ez ? bm : R[5][0];
        }
    } else if (normals) {
        fa = phi[i];
        fb = phi[i + step];
        lattice_reads(phi, i, x, g.nx, 1, r[0], r[1]);
        lattice_reads(phi, i, y, g.ny, sx, r[2], r[3]);
        lattice_reads(phi, i, z, g.nz, sxy, r[4], r[5]);
        lattice_reads(phi, i + step, xb, g.nx, 1, r[6], r[7]);
        lattice_reads(phi, i + step, yb, g.ny, sx, r[8], r[9]);
        lattice_reads(phi, i + step, zb, g.nz, sxy, r[10], r[11]);
    } else {
        fa = phi[i];
        fb = phi[i + step];
    }
    const float t = __fdiv_rn(iso - fa, fb - fa);
    const float pa = __fadd_rn(a == 0 ? c0 : (a == 1 ? c1 : c2), __fmul_rn(t, g.hf));
    verts[3 * (int64_t)v + 0] = a == 0 ? pa : c0;
    verts[3 * (int64_t)v + 1] = a == 1 ? pa : c1;
    verts[3 * (int64_t)v + 2] = a == 2 ? pa : c2;
    if (normals) {
        // n = (1 - t) g_a + t g_b, normalised; float32, one rounded
        // operation at a time
        const float ga[3] = {lattice_diff(r[0], r[1], x, g.nx), lattice_diff(r[2], r[3], y, g.ny),
                             lattice_diff(r[4], r[5], z, g.nz)};
        const float gb[3] = {lattice_diff(r[6], r[7], xb, g.nx),
                             lattice_diff(r[8], r[9], yb, g.ny),
                             lattice_diff(r[10], r[11], zb, g.nz)};
        const float w = __fsub_rn(1.0f, t);
        float nv[3];
        for (int k = 0; k < 3; ++k)
            nv[k] = __fadd_rn(__fmul_rn(w, ga[k]), __fmul_rn(t, gb[k]));
        const float l2 = __fadd_rn(__fadd_rn(__fmul_rn(nv[0], nv[0]), __fmul_rn(nv[1], nv[1])),
                                   __fmul_rn(nv[2], nv[2]));
        // correctly rounded float32 square root: the FP64 root rounded to
        // float32 (53 >= 2 * 24 + 2 bits, so the double rounding is exact);
        // v_sqrt_f32 alone is not exact
        const float l = (float)sqrt((double)l2);
        for (int k = 0; k < 3; ++k)
            normals[3 * (int64_t)v + k] = l > 0.0f ? __fdiv_rn(nv[k], l) : 0.0f;
    }
}

// What the triangles of a word's cells need of the words their corners lie
// in: the words at the four offsets of corner_words, two each, kept in LDS
// (read from memory per triangle corner, scattered, they took most of the
// cache's lookups).
struct McCorner {
    uint64_t e[3];
    uint32_t id;         // first vertex
};

// Triangle k of the cell at bit b of a word (case cs), into slot t: its
// corners are the vertices of the cell edges the case table names.  The
// vertex on edge `axis` of a point follows those of its word's earlier points
// and of its own earlier axes.
__device__ __forceinline__ void mc_emit_tri(const int8_t *__restrict__ tris_of,
                                            const McCorner *__restrict__ corners,
                                            const uint32_t off_bits[4],
                                            int32_t *__restrict__ tris, uint32_t b, int cs, int k,
                                            uint32_t t)
{
    int32_t id[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int edge = tris_of[cs * 15 + 3 * k + e];
        // edges are numbered (axis, lower corner): 4 per axis
        const int axis = edge >> 2, nth = edge & 3;
        // the nth corner (ascending) whose bit `axis` is clear
        const int lo = nth & ((1 << axis) - 1);
        const int corner = ((nth >> axis) << (axis + 1)) | lo;
        const int o = corner >> 1;
        const uint32_t ob = o == 0 ? off_bits[0] : o == 1 ? off_bits[1] : o == 2 ? off_bits[2]
                                                                                 : off_bits[3];
        const uint32_t at = ob + b + (uint32_t)(corner & 1);   // at most 63 + 63 + 1
        const McCorner &m = corners[2 * o + (int)(at >> 6)];
        const uint64_t bit = 1ull << (at & 63u);
        // edges before (point, axis): all of earlier points, the point's of
        // lower axes
        const uint64_t m0 = axis > 0 ? (bit << 1) - 1ull : bit - 1ull;
        const uint64_t m1 = axis > 1 ? (bit << 1) - 1ull : bit - 1ull;
        id[e] = (int32_t)(m.id + (uint32_t)(__popcll(m.e[0] & m0) + __popcll(m.e[1] & m1) +
                                            __popcll(m.e[2] & (bit - 1ull))));
    }
    __builtin_memcpy(tris + 3 * (int64_t)t, id, sizeof id);
}

// One wave per group of listed words.  Their points need different amounts of
// work (0 to 3 vertices, 0 to 5 triangles), so the wave lists its vertices, its
// active cells, and the triangles of 64 cells at a time as items in LDS, and
// each lane emits one item at a time: every lane runs the same code on every
// item, and no wave waits for another.  Bound by VALU issue and by the chain
// of a wave's reads: 93 us on 1.7M vertices and 3.4M triangles (142 us with
// blocks of 1,024 points).
constexpr int kMcEmitWords = (int)(kMcGroup / kMcMinWeight), kMcEmitWaves = kBlock / 64;
constexpr int kMcSlice = kMcEmitWords;        // points of a lane
// Blocks of the emission, each over several groups where there are more: the
// host does not know the number of groups when it enqueues them.  (1.7M
// vertices: 93 us; 1,280 blocks 100, 2,048 103.)
constexpr unsigned kMcEmitBlocks = 4096;

__device__ __forceinline__ uint32_t wave_scan_excl(uint32_t v, int lane, uint32_t &tot)
{
    uint32_t r = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(r, o, 64);
        if (lane >= o) r += y;
    }
    tot = __shfl(r, 63, 64);
    return r - v;
}

// LDS written by this wave is read by it next
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(kBlock) void k_mc_emit(const float *__restrict__ phi, TsdfGrid g,
                                                    float iso, int64_t nw, uint32_t nb,
                                                    const uint32_t *__restrict__ totals,
                                                    uint32_t cap_v, uint32_t cap_t,
                                                    const uint8_t *__restrict__ ntri,
                                                    const int8_t *__restrict__ tris_of,
                                                    const uint64_t *__restrict__ inside,
                                                    const McWord *__restrict__ words,
                                                    const uint64_t *__restrict__ cells,
                                                    const uint8_t *__restrict__ list,
                                                    const uint8_t *__restrict__ group,
                                                    const uint32_t *__restrict__ nlist,
                                                    const uint32_t *__restrict__ vbase,
                                                    const uint32_t *__restrict__ tbase,
                                                    const uint32_t *__restrict__ gbase,
                                                    float *__restrict__ verts,
                                                    int32_t *__restrict__ tris,
                                                    float *__restrict__ normals)
{
    constexpr int WL = 64 / kMcEmitWords;         // lanes of a word
    constexpr int PTS = 64 * kMcEmitWords;        // points of a wave
    static_assert(WL == 8 && WL * kMcSlice == 64, "a lane a corner word");
    static_assert(PTS <= 1024, "point in bits 0..9 of an item");
    // vertex items (point | axis << 10), then cell items (point)
    __shared__ uint16_t s_item[kMcEmitWaves][3 * PTS];
    __shared__ uint16_t s_tri[kMcEmitWaves][5 * 64];         // lane of the cell | k << 6
    __shared__ uint32_t s_cell[kMcEmitWaves][64];            // point | case << 10
    __shared__ uint64_t s_c[kMcEmitWaves][kMcEmitWords][8];  // corners of the words
    __shared__ McCorner s_k[kMcEmitWaves][kMcEmitWords][8];
    // a word's first lattice point, its first vertex's and triangle's slots
    // less their items' places, its first cell's place
    __shared__ int64_t s_base[kMcEmitWaves][kMcEmitWords];
    __shared__ uint32_t s_v[kMcEmitWaves][kMcEmitWords], s_t[kMcEmitWaves][kMcEmitWords];
    __shared__ uint8_t nt_lds[256];
    // the case table's triangle edges (256 x 15 bytes, word aligned)
    __shared__ uint32_t tri_lds[256 * 15 / 4];
    // the caller's capacity: the host reads the totals behind this launch
    const uint32_t ngroups = totals[2];
    if (totals[0] > cap_v || totals[1] > cap_t) return;
    nt_lds[threadIdx.x] = ntri[threadIdx.x];              // kBlock == 256 cases
    for (int k = threadIdx.x; k < 256 * 15 / 4; k += kBlock)
        tri_lds[k] = reinterpret_cast<const uint32_t *>(tris_of)[k];
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63), wv = (int)(threadIdx.x >> 6);
    const int wi = lane / WL, part_w = lane % WL, b0 = part_w * kMcSlice;
    const int64_t sxy = (int64_t)g.nx * g.ny;
    const uint32_t off_bits[4] = {0u, (uint32_t)g.nx & 63u, (uint32_t)(sxy & 63),
                                  (uint32_t)((sxy + g.nx) & 63)};
    for (uint32_t grp = blockIdx.x * kMcEmitWaves + wv; grp < ngroups;
         grp += gridDim.x * kMcEmitWaves) {
        // the count block: the last whose first group is not beyond grp, by a
        // search of 64 places at a time
        uint32_t blk = 0;
        for (uint32_t span = nb; span > 1;) {
            const uint32_t step = (span + 63u) / 64u, at = blk + lane * step;
            const bool le = lane * step < span && gbase[at] <= grp;
            const uint32_t top = 63u - (uint32_t)__builtin_clzll(__ballot(le));   // lane 0 always
            blk += top * step;
            span = span - top * step < step ? span - top * step : step;
        }
        const uint32_t gk = grp - gbase[blk], nl = nlist[blk];
        const uint32_t gn = blk + 1 < nb ? gbase[blk + 1] - gbase[blk] : ngroups - gbase[blk];
        const uint8_t *gs = group + (int64_t)blk * kMcWords + gk;
        const uint32_t l = gs[0] + (uint32_t)wi, lend = gk + 1 < gn ? gs[1] : nl;
        const uint32_t vb = vbase[blk], tb = tbase[blk];
        uint32_t e[3] = {0, 0, 0}, act = 0, v0 = 0, t0 = 0;
        int64_t w = 0;
        if (l < lend) {
            w = (int64_t)blk * kMcWords + list[(int64_t)blk * kMcWords + l];
            const McWord m = words[w];
            const uint32_t low = (uint32_t)((1ull << kMcSlice) - 1ull);
            v0 = vb + m.v;
            t0 = tb + m.t;
            for (int a = 0; a < 3; ++a) e[a] = (uint32_t)(m.e[a] >> b0) & low;
            act = (uint32_t)(cells[w] >> b0) & low;
            const int o = part_w >> 1;
            const int64_t off = (o & 1 ? (int64_t)g.nx : 0) + (o & 2 ? sxy : 0);
            const int64_t q = w + (off >> 6) + (part_w & 1);
            if (q < nw) {                  // a word without vertices is not named
                const McWord mq = words[q];
                McCorner &k = s_k[wv][wi][part_w];
                for (int a = 0; a < 3; ++a) k.e[a] = mq.e[a];
                k.id = vbase[q / kMcWords] + mq.v;
            }
            if ((part_w & 1) == 0) {
                uint64_t u, v;
                corner_words(inside, nw, w, off, u, v);
                s_c[wv][wi][2 * o] = u;
                s_c[wv][wi][2 * o + 1] = v;
            }
        }
        // at most 3 PTS vertices and PTS cells
        uint32_t tot;
        const uint32_t r = wave_scan_excl((uint32_t)(__popc(e[0]) + __popc(e[1]) + __popc(e[2])) |
                                              ((uint32_t)__popc(act) << 16), lane, tot);
        const uint32_t nv = tot & 0xffffu, nc = tot >> 16;
        uint32_t rv = r & 0xffffu, rc = r >> 16;
        if (part_w == 0) {
            s_base[wv][wi] = 64 * w;
            s_v[wv][wi] = v0 - rv;
        }
        uint32_t todo = e[0] | e[1] | e[2];
        while (todo) {
            const int b = __builtin_ctz(todo);
            todo &= todo - 1;
            const uint32_t pt = (uint32_t)(lane * kMcSlice + b);
#pragma unroll
            for (uint32_t a = 0; a < 3; ++a)
                if ((e[a] >> b) & 1u) s_item[wv][rv++] = (uint16_t)(pt | (a << 10));
        }
        wave_lds_fence();
        for (uint32_t j = lane; j < nv; j += 64) {
            const uint32_t it = s_item[wv][j], pt = it & 1023u;
            mc_emit_vertex(phi, g, iso, verts, normals, s_base[wv][pt >> 6] + (pt & 63u),
                           (int)(it >> 10), s_v[wv][pt >> 6] + j);
        }
        wave_lds_fence();
        const bool first = part_w == 0;
        uint32_t word_c0 = rc;      // place of the word's first cell (first lanes)
        while (act) {
            const int b = __builtin_ctz(act);
            act &= act - 1;
            s_item[wv][rc++] = (uint16_t)(lane * kMcSlice + b);
        }
        wave_lds_fence();
        uint32_t done = 0;          // triangles of earlier cells
        for (uint32_t j0 = 0; j0 < nc; j0 += 64) {
            const uint32_t j = j0 + lane;
            uint32_t n = 0;
            if (j < nc) {
                const uint32_t pt = s_item[wv][j];
                uint32_t cs = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    cs |= (uint32_t)((s_c[wv][pt >> 6][k] >> (pt & 63u)) & 1ull) << k;
                s_cell[wv][lane] = pt | (cs << 10);
                n = nt_lds[cs];
            }
            uint32_t nt;
            const uint32_t rt = wave_scan_excl(n, lane, nt);
            for (uint32_t k = 0; k < n; ++k) s_tri[wv][rt + k] = (uint16_t)(lane | (k << 6));
            // the triangles before a word's first cell, if it lies in these 64
            const uint32_t at = __shfl(rt, (int)((word_c0 - j0) & 63u), 64);
            if (first && word_c0 - j0 < 64u) s_t[wv][wi] = t0 - (done + at);
            wave_lds_fence();
            for (uint32_t q = lane; q < nt; q += 64) {
                const uint32_t it = s_tri[wv][q], cc = s_cell[wv][it & 63u], pt = cc & 1023u;
                mc_emit_tri(reinterpret_cast<const int8_t *>(tri_lds), s_k[wv][pt >> 6], off_bits, tris,
                            pt & 63u, (int)(cc >> 10), (int)(it >> 6), s_t[wv][pt >> 6] + done + q);
            }
            done += nt;
            wave_lds_fence();
        }
        wave_lds_fence();             // the next group refills the lists
    }
}

// ---- exclusive scan of uint32 (three kernels) ------------------------------

__global__ __launch_bounds__(kBlock) void k_scan_tiles(const uint32_t *__restrict__ in,
                                                       uint32_t *__restrict__ out, int64_t n,
                                                       uint32_t *__restrict__ sums)
{
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems], s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = base + k < n ? in[base + k] : 0u;
        s += v[k];
    }
    uint32_t tot;
    uint32_t run = block_scan_excl(s, &tot);
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// One 1024-thread block: exclusive scans of the vertex and the triangle
// tile totals in place, grand totals after them.
constexpr int kSums3Block = 1024;

__device__ __forceinline__ uint32_t block_scan_excl_1024(uint32_t v, uint32_t *total,
                                                         uint32_t *ws)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) ws[w] = x;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int k = 0; k < kSums3Block / 64; ++k) {
        if (k < w) off += ws[k];
        tot += ws[k];
    }
    __syncthreads();
    *total = tot;
    return off + x - v;
}

// Exclusive scans of three arrays of nb entries in place, grand totals to
// totals[3].  Chunks of kSums3Chunk entries of each go through LDS: loaded
// and stored coalesced, scanned there with four consecutive entries per
// thread (per-thread contiguous global reads were uncoalesced).
constexpr int kSums3Chunk = kSums3Block * 4;

__global__ __launch_bounds__(kSums3Block) void k_scan_sums3(uint32_t *__restrict__ a0,
                                                            uint32_t *__restrict__ a1,
                                                            uint32_t *__restrict__ a2, int nb,
                                                            uint32_t *__restrict__ totals)
{
    __shared__ uint32_t l[3][kSums3Chunk];
    __shared__ uint32_t ws[kSums3Block / 64];
    uint32_t *const a[3] = {a0, a1, a2};
    uint32_t carry[3] = {0, 0, 0};
    for (int c0 = 0; c0 < nb; c0 += kSums3Chunk) {
        const int m = nb - c0 < kSums3Chunk ? nb - c0 : kSums3Chunk;
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = k * kSums3Block + (int)threadIdx.x;
                l[q][i] = i < m ? a[q][c0 + i] : 0u;
            }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            uint32_t v[4], sum = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = l[q][4 * threadIdx.x + k];
                sum += v[k];
            }
            uint32_t tot;
            uint32_t r = carry[q] + block_scan_excl_1024(sum, &tot, ws);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                l[q][4 * threadIdx.x + k] = r;
                r += v[k];
            }
            carry[q] += tot;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = k * kSums3Block + (int)threadIdx.x;
                if (i < m) a[q][c0 + i] = l[q][i];
            }
        __syncthreads();   // refilled by the next chunk
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 3; ++q) totals[q] = carry[q];
}

// one block: exclusive scan of the tile sums in place, grand total after
// them.  Each thread owns a contiguous chunk (sum it, one block scan of the
// chunk totals, then write the chunk's prefixes): walking 256 sums per
// block-wide step took 35 us for 32k tiles.
__global__ __launch_bounds__(kBlock) void k_scan_sums(uint32_t *__restrict__ sums, int nb)
{
    const int per = (nb + kBlock - 1) / kBlock;
    const int lo = (int)threadIdx.x * per;
    const int hi = lo + per < nb ? lo + per : nb;
    // chunks are read and written 16 entries at a time so that the loads
    // of a group are in flight together
    uint32_t s = 0;
    for (int i0 = lo; i0 < hi; i0 += 16) {
        uint32_t v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = i0 + k < hi ? sums[i0 + k] : 0u;
#pragma unroll
        for (int k = 0; k < 16; ++k) s += v[k];
    }
    uint32_t tot;
    uint32_t run = block_scan_excl(s, &tot);
    for (int i0 = lo; i0 < hi; i0 += 16) {
        uint32_t v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = i0 + k < hi ? sums[i0 + k] : 0u;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if (i0 + k < hi) sums[i0 + k] = run;
            run += v[k];
        }
    }
    if (threadIdx.x == 0) sums[nb] = tot;
}

__global__ __launch_bounds__(kBlock) void k_scan_add(uint32_t *__restrict__ out, int64_t n,
                                                     const uint32_t *__restrict__ sums)
{
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    const uint32_t add = sums[blockIdx.x];
    for (int k = threadIdx.x; k < kScanTile; k += kBlock)
        if (base + k < n) out[base + k] += add;
}

// ---- the case table (host) -------------------------------------------------
// Corner k of a cell is (k & 1, k >> 1 & 1, k >> 2 & 1); edge e = 4 axis + j
// joins the j-th corner (ascending) with bit `axis` clear to that corner plus
// the unit step along `axis`.
struct Table {
    uint8_t count[256];
    int8_t tri[256][15];
};

void make_table(Table &t)
{
    int ea[12], eb[12];
    int edge_of[8][8];
    for (int a = 0; a < 8; ++a)
        for (int b = 0; b < 8; ++b) edge_of[a][b] = -1;
    int ne = 0;
    for (int axis = 0; axis < 3; ++axis)
        for (int a = 0; a < 8; ++a)
            if (!((a >> axis) & 1)) {
                ea[ne] = a;
                eb[ne] = a | (1 << axis);
                edge_of[a][eb[ne]] = edge_of[eb[ne]][a] = ne;
                ++ne;
            }
    // faces: corners counter-clockwise about the outward normal
    int face[6][4];
    int nf = 0;
    for (int axis = 0; axis < 3; ++axis) {
        const int u = (axis + 1) % 3, v = (axis + 2) % 3;
        for (int side = 0; side < 2; ++side) {
            const int uv[4][2] = {{0, 0}, {1, 0}, {1, 1}, {0, 1}};   // about +axis
            for (int k = 0; k < 4; ++k) {
                const int kk = side ? k : 3 - k;                     // -axis: reversed
                const int cu = uv[kk][0], cv = uv[kk][1];
                face[nf][k] = (side << axis) | (cu << u) | (cv << v);
            }
            ++nf;
        }
    }
    unsigned efaces[12] = {0};
    for (int f = 0; f < 6; ++f)
        for (int k = 0; k < 4; ++k) efaces[edge_of[face[f][k]][face[f][(k + 1) % 4]]] |= 1u << f;
    (void)ea;
    (void)eb;
    for (int cs = 0; cs < 256; ++cs) {
        int succ[12];
        for (int e = 0; e < 12; ++e) succ[e] = -1;
        for (int f = 0; f < 6; ++f) {
            int ce[4], cin[4], nc = 0;   // crossings in walk order; cin = outside->inside
            for (int k = 0; k < 4; ++k) {
                const int a = face[f][k], b = face[f][(k + 1) % 4];
                const int ia = (cs >> a) & 1, ib = (cs >> b) & 1;
                if (ia != ib) {
                    ce[nc] = edge_of[a][b];
                    cin[nc] = ib;
                    ++nc;
                }
            }
            for (int j = 0; j < nc; ++j) {
                if (!cin[j]) continue;
                for (int s = 1; s < nc; ++s) {
                    const int q = (j + s) % nc;
                    if (!cin[q]) {
                        succ[ce[j]] = ce[q];
                        break;
                    }
                }
            }
        }
        int n = 0;
        bool seen[12] = {false};
        for (int e0 = 0; e0 < 12; ++e0) {
            if (succ[e0] < 0 || seen[e0]) continue;
            int loop[12], k = 0;
            int e = e0;
            do {
                loop[k++] = e;
                seen[e] = true;
                e = succ[e];
            } while (e != e0);
            // fan apex: first vertex whose diagonals join edges sharing no face
            int apex = 0;
            for (int j = 0; j < k; ++j) {
                bool ok = true;
                for (int q = 0; q < k && ok; ++q) {
                    if (q == j || q == (j + 1) % k || q == (j + k - 1) % k) continue;
                    if (efaces[loop[j]] & efaces[loop[q]]) ok = false;
                }
                if (ok) {
                    apex = j;
                    break;
                }
            }
            for (int q = 1; q + 1 < k; ++q) {
                t.tri[cs][3 * n + 0] = (int8_t)loop[apex];
                t.tri[cs][3 * n + 1] = (int8_t)loop[(apex + q) % k];
                t.tri[cs][3 * n + 2] = (int8_t)loop[(apex + q + 1) % k];
                ++n;
            }
        }
        t.count[cs] = (uint8_t)n;
        for (int q = 3 * n; q < 15; ++q) t.tri[cs][q] = -1;
    }
}

const Table &table()
{
    static Table t;
    static std::once_flag once;
    std::call_once(once, [] { make_table(t); });
    return t;
}

hipError_t scan_launch(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *sums,
                       hipStream_t s)
{
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)nb), dim3(kBlock), 0, s, in, out, n, sums);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kBlock), 0, s, sums, (int)nb);
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(kBlock), 0, s, out, n, sums);
    return hipGetLastError();
}

}  // namespace

void mc_table_copy(uint8_t *count, int8_t *tri)
{
    const Table &t = table();
    for (int c = 0; c < 256; ++c) {
        count[c] = t.count[c];
        for (int q = 0; q < 15; ++q) tri[15 * c + q] = t.tri[c][q];
    }
}

int64_t mc_scan_sums_len(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

size_t tsdf_smooth_a_bytes(const TsdfGrid &g) { return (size_t)(4 * g.n); }
size_t tsdf_smooth_b_bytes(const TsdfGrid &g) { return (size_t)(8 * g.n); }

hipError_t tsdf_smooth_launch(const uint8_t *surf, uint32_t *a, uint64_t *b, uint8_t *vt,
                              const TsdfGrid &g, const Binomial &w, uint64_t thr, hipStream_t s)
{
    const unsigned grid = grid_for(g.n, kBlock);
    hipLaunchKernelGGL(k_smooth_x, dim3(grid), dim3(kBlock), 0, s, surf, a, g, w);
    hipLaunchKernelGGL(k_smooth_y, dim3(grid), dim3(kBlock), 0, s, a, b, g, w);
    hipLaunchKernelGGL(k_smooth_z, dim3(grid), dim3(kBlock), 0, s, b, vt, g, w, thr);
    return hipGetLastError();
}

hipError_t tsdf_smooth_sums_launch(const uint8_t *surf, uint32_t *a, uint64_t *b, uint64_t *sums,
                                   const TsdfGrid &g, const Binomial &w, hipStream_t s)
{
    const unsigned grid = grid_for(g.n, kBlock);
    hipLaunchKernelGGL(k_smooth_x, dim3(grid), dim3(kBlock), 0, s, surf, a, g, w);
    hipLaunchKernelGGL(k_smooth_y, dim3(grid), dim3(kBlock), 0, s, a, b, g, w);
    hipLaunchKernelGGL(k_smooth_z_sum, dim3(grid), dim3(kBlock), 0, s, b, sums, g, w);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_stride_gather(const float *__restrict__ phi, TsdfGrid g,
                                                          int step, int mx, int my, int64_t m,
                                                          float *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= m) return;
    const int64_t x = i % mx, yz = i / mx;
    const int64_t y = yz % my, z = yz / my;
    out[i] = phi[((z * step) * g.ny + y * step) * (int64_t)g.nx + x * step];
}

hipError_t mc_stride_gather_launch(const float *phi, const TsdfGrid &g, int step, int mx, int my,
                                   int mz, float *out, hipStream_t s)
{
    const int64_t m = (int64_t)mx * my * mz;
    hipLaunchKernelGGL(k_stride_gather, dim3(grid_for(m, kBlock)), dim3(kBlock), 0, s, phi, g,
                       step, mx, my, m, out);
    return hipGetLastError();
}

hipError_t tsdf_threshold_pack_launch(const uint64_t *sums, const uint64_t *thr, uint8_t *vt,
                                      uint64_t *F, uint64_t *O, const TsdfGrid &g, hipStream_t s)
{
    const int W = (g.nx + 63) / 64;
    hipLaunchKernelGGL(k_threshold_pack, dim3(grid_for((int64_t)W * g.ny * g.nz, kPackSums * (kBlock / 64))),
                       dim3(kBlock), 0, s, sums, thr, vt, g, W, F, O);
    return hipGetLastError();
}

int tsdf_words_per_row(const TsdfGrid &g) { return (g.nx + 63) / 64; }

static Cols cols_of(const TsdfGrid &g, int axis)
{
    const int W = tsdf_words_per_row(g);
    Cols c;
    c.rows = axis == 1 ? g.ny : g.nz;
    c.ncols = (int64_t)W * (axis == 1 ? g.nz : g.ny);
    c.stride = axis == 1 ? W : (int64_t)W * g.ny;
    c.nseg = (c.rows + kSegRows - 1) / kSegRows;
    return c;
}

int64_t tsdf_seg_words(const TsdfGrid &g)
{
    const Cols a = cols_of(g, 1), b = cols_of(g, 2);
    const int64_t na = a.ncols * a.nseg, nb = b.ncols * b.nseg;
    return na > nb ? na : nb;
}

bool tsdf_smooth_on_bits(const Binomial &w) { return w.n >= 1 && w.n <= 3; }

hipError_t tsdf_smooth_bits_launch(const uint8_t *surf, uint64_t *bits, uint8_t *vt, uint64_t *F,
                                   uint64_t *O, const TsdfGrid &g, const Binomial &w, uint64_t thr,
                                   hipStream_t s)
{
    const int W = tsdf_words_per_row(g);
    const dim3 tiles = xcd_tiles((int64_t)W * ((g.ny + kSmY - 1) / kSmY) * ((g.nz + kSmZ - 1) / kSmZ));
    hipLaunchKernelGGL(k_pack_bits<false>, dim3(grid_for((int64_t)W * g.ny * g.nz, kPackRun * (kBlock / 4))),
                       dim3(kBlock), 0, s, surf, g, W, fastdiv_constant((uint32_t)W), bits,
                       (uint64_t *)nullptr);
    switch (w.n) {
    case 1: hipLaunchKernelGGL(k_smooth_bits<1>, tiles, dim3(kBlock), 0, s, bits, vt, g, thr, W, F, O); break;
    case 2: hipLaunchKernelGGL(k_smooth_bits<2>, tiles, dim3(kBlock), 0, s, bits, vt, g, thr, W, F, O); break;
    case 3: hipLaunchKernelGGL(k_smooth_bits<3>, tiles, dim3(kBlock), 0, s, bits, vt, g, thr, W, F, O); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t tsdf_pack_launch(const uint8_t *vt, uint64_t *F, uint64_t *O, const TsdfGrid &g,
                            hipStream_t s)
{
    const int W = tsdf_words_per_row(g);
    hipLaunchKernelGGL(k_pack_bits<true>, dim3(grid_for((int64_t)W * g.ny * g.nz, kPackRun * (kBlock / 4))),
                       dim3(kBlock), 0, s, vt, g, W, fastdiv_constant((uint32_t)W), F, O);
    return hipGetLastError();
}

// x and y together, where a slice's words fit LDS, unless there are many thin
// slices: a block's chain takes as long for few words, so that beyond one block
// of each of the chip's 1,024 places (kSliceFew) the row sweep, which packs the
// rows of many slices into a block, is the faster one on slices of fewer than
// kSliceMany words.  us a TSDF call on noise, together / apart, by words a slice:
//   64 x 64 x 1,024 (64): 549 / 584       64 x 16 x 20,000 (16): 3,209 / 2,224
//   64 x 64 x 2,000 (64): 602 / 550       256 x 64 x 4,096 (256): 1,455 / 1,175
//   64 x 256 x 1,400 (256): 653 / 665     256 x 128 x 2,048 (512): 1,224 / 1,137
//   128 x 256 x 1,500 (512): 956 / 964    256 x 256 x 4,096 (1,024): 3,220 / 3,217
//   320 x 200 x 3,000 (1,000): 2,436 / 2,488   512 x 256 x 2,048 (2,048): 2,715 / 3,660
constexpr int kSliceFew = 1024, kSliceMany = 768;

static bool sweep_slices(const TsdfGrid &g)
{
    const int64_t words = (int64_t)slice_pitch(tsdf_words_per_row(g)) * g.ny;
    return words <= kSliceWords && (g.nz <= kSliceFew || words >= kSliceMany) &&
           (int64_t)g.nz * kSliceBlock <= 0x7fffffffLL;       // a launch's blocks
}

bool tsdf_label_small(const TsdfGrid &g)
{
    const int W = tsdf_words_per_row(g);
    return W <= kLabelColumn && g.ny <= kLabelColumn && g.nz <= kLabelColumn &&
           (int64_t)label_pitch(g, W) * g.nz <= kSliceWords;
}

hipError_t tsdf_label_small_launch(const uint64_t *F, uint64_t *O, const TsdfGrid &g, hipStream_t s)
{
    hipLaunchKernelGGL(k_label_small, dim3(1), dim3(kLabelBlock), 0, s, F, O, g,
                       tsdf_words_per_row(g));
    return hipGetLastError();
}

hipError_t tsdf_flood_round_launch(const uint64_t *F, uint64_t *O, uint64_t *seg,
                                   const TsdfGrid &g, const int32_t *prev, int32_t *changed,
                                   hipStream_t s)
{
    const int W = tsdf_words_per_row(g);
    const bool slices = sweep_slices(g);
    if (slices && (int64_t)slice_pitch(W) * g.ny <= kSliceSmall)
        hipLaunchKernelGGL(k_sweep_slice<kSliceSmall>, dim3((unsigned)g.nz), dim3(kSliceBlock), 0, s,
                           F, O, g, W, changed, prev);
    else if (slices)
        hipLaunchKernelGGL(k_sweep_slice<kSliceWords>, dim3((unsigned)g.nz), dim3(kSliceBlock), 0, s,
                           F, O, g, W, changed, prev);
    else
        hipLaunchKernelGGL(k_sweep_x, dim3(grid_for((int64_t)g.ny * g.nz, kBlock)), dim3(kBlock), 0,
                           s, F, O, g, W, changed, prev);
    const int64_t ns = tsdf_seg_words(g);
    uint64_t *A = seg, *B = seg + ns, *T = seg + 2 * ns, *C = seg + 3 * ns, *D = seg + 4 * ns;
    for (int axis = slices ? 2 : 1; axis <= 2; ++axis) {
        const Cols cl = cols_of(g, axis);
        if (cl.nseg <= kFusedSegs) {
            const int cj = (kBlock / cl.nseg) & ~7;       // >= 8: whole 64-byte rows of words
            const unsigned gb = (unsigned)((cl.ncols + cj - 1) / cj);
            if (axis == 1)
                hipLaunchKernelGGL(k_seg_fused<1>, dim3(gb), dim3(kBlock), 0, s, F, O, g, W, cl,
                                   cj, changed, prev);
            else
                hipLaunchKernelGGL(k_seg_fused<2>, dim3(gb), dim3(kBlock), 0, s, F, O, g, W, cl,
                                   cj, changed, prev);
            continue;
        }
        const unsigned gs = grid_for(cl.ncols * cl.nseg, kBlock);
        if (axis == 1)
            hipLaunchKernelGGL(k_seg_summary<1>, dim3(gs), dim3(kBlock), 0, s, F, O, g, W, cl, A, B,
                               T, prev);
        else
            hipLaunchKernelGGL(k_seg_summary<2>, dim3(gs), dim3(kBlock), 0, s, F, O, g, W, cl, A, B,
                               T, prev);
        hipLaunchKernelGGL(k_seg_carry, dim3(grid_for(cl.ncols, kBlock)), dim3(kBlock), 0, s, A, B,
                           T, cl, C, D, prev);
        if (axis == 1)
            hipLaunchKernelGGL(k_seg_apply<1>, dim3(gs), dim3(kBlock), 0, s, F, O, g, W, cl, C, D,
                               changed, prev);
        else
            hipLaunchKernelGGL(k_seg_apply<2>, dim3(gs), dim3(kBlock), 0, s, F, O, g, W, cl, C, D,
                               changed, prev);
    }
    return hipGetLastError();
}

// one z-layer plus two words, rounded up to a word: the farthest neighbour
// word of the four-voxel shell kernel
int64_t tsdf_shell_pad(const TsdfGrid &g) { return (((int64_t)g.nx * g.ny + 8) + 3) & ~(int64_t)3; }

bool tsdf_shells_on_bits(int shells) { return shells >= 1 && shells <= 4; }

hipError_t tsdf_shells_phi_bits_launch(const uint64_t *F, const uint64_t *O, float *phi,
                                       const TsdfGrid &g, int shells, float h, float r,
                                       const int32_t *unsettled, hipStream_t s)
{
    const int W = tsdf_words_per_row(g);
    const dim3 tiles = xcd_tiles((int64_t)W * ((g.ny + kShY - 1) / kShY) * ((g.nz + kShZ - 1) / kShZ));
    switch (shells) {
    case 1: hipLaunchKernelGGL(k_shells_phi_bits<1>, tiles, dim3(kBlock), 0, s, F, O, phi, g, W, h, r, unsettled); break;
    case 2: hipLaunchKernelGGL(k_shells_phi_bits<2>, tiles, dim3(kBlock), 0, s, F, O, phi, g, W, h, r, unsettled); break;
    case 3: hipLaunchKernelGGL(k_shells_phi_bits<3>, tiles, dim3(kBlock), 0, s, F, O, phi, g, W, h, r, unsettled); break;
    case 4: hipLaunchKernelGGL(k_shells_phi_bits<4>, tiles, dim3(kBlock), 0, s, F, O, phi, g, W, h, r, unsettled); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t tsdf_shells_phi_launch(const uint8_t *vt, const uint64_t *O, uint8_t *p, float *phi,
                                  const TsdfGrid &g, int shells, float h, float r, hipStream_t s)
{
    const unsigned grid = grid_for(g.n, kBlock);
    const unsigned grid4 = grid_for((g.n + 3) / 4, kBlock);
    if (((uintptr_t)vt & 3) == 0)
        hipLaunchKernelGGL(k_shell0, dim3(grid4), dim3(kBlock), 0, s, vt, p, g);
    else
        hipLaunchKernelGGL(k_shell0_1, dim3(grid), dim3(kBlock), 0, s, vt, p, g);
    for (int m = 1; m <= shells; ++m)
        hipLaunchKernelGGL(k_shell, dim3(grid4), dim3(kBlock), 0, s, p, g, m);
    hipLaunchKernelGGL(k_phi, dim3(grid4), dim3(kBlock), 0, s, p, O, phi, g, tsdf_words_per_row(g),
                       h, r, ((uintptr_t)phi & 15) == 0 ? 1 : 0);
    return hipGetLastError();
}

int64_t mc_words(int64_t n) { return (n + 63) / 64; }
int64_t mc_blocks(int64_t n) { return (mc_words(n) + kMcWords - 1) / kMcWords; }
size_t mc_word_bytes() { return sizeof(McWord); }

hipError_t mc_count_launch(const float *phi, const TsdfGrid &g, float iso, const uint8_t *ntri,
                           const McBuffers &b, hipStream_t s)
{
    const int64_t nw = mc_words(g.n), nb = mc_blocks(g.n);
    hipLaunchKernelGGL(k_mc_inside, dim3(grid_for(nw, kMcInsideRun * (kBlock / 64))), dim3(kBlock),
                       0, s, phi, g.n, iso, b.inside);
    hipLaunchKernelGGL(k_mc_count, dim3((unsigned)nb), dim3(kMcWords), 0, s, b.inside, g, nw, ntri,
                       static_cast<McWord *>(b.words), b.cells, b.list, b.group, b.nlist, b.vsums, b.tsums,
                       b.gsums);
    hipLaunchKernelGGL(k_scan_sums3, dim3(1), dim3(kSums3Block), 0, s, b.vsums, b.tsums, b.gsums,
                       (int)nb, b.totals);
    return hipGetLastError();
}

hipError_t mc_emit_launch(const float *phi, const TsdfGrid &g, float iso, const uint8_t *ntri,
                          const int8_t *tris_of, const McBuffers &b, uint32_t cap_verts,
                          uint32_t cap_tris, float *verts, int32_t *tris, float *normals,
                          hipStream_t s)
{
    // at most one group a word; waves go on to further groups
    const int64_t nw = mc_words(g.n);
    const unsigned blocks = grid_for(nw, kMcEmitWaves);
    hipLaunchKernelGGL(k_mc_emit, dim3(blocks < kMcEmitBlocks ? blocks : kMcEmitBlocks),
                       dim3(kBlock), 0, s, phi, g, iso, nw, (uint32_t)mc_blocks(g.n), b.totals,
                       cap_verts, cap_tris, ntri, tris_of, b.inside,
                       static_cast<const McWord *>(b.words), b.cells, b.list, b.group, b.nlist,
                       b.vsums, b.tsums, b.gsums, verts, tris, normals);
    return hipGetLastError();
}

hipError_t scan_u32_launch(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *sums,
                           hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    return scan_launch(in, out, n, sums, s);
}
