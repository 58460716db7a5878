"""Denoising, flood-fill sign, narrow-band TSDF and marching cubes on the GPU
vs the oracle (oracle/tsdf.py), FGGS-LiDAR Sec. IV-B.

Parity bar.  V~ is decided on exact integer sums, the sign and shell
indices are integer and phi is one float32 product and a clip: bit-exact.
The mesh's topology (which edges carry vertices, the triangles, the
canonical numbering) comes from exact comparisons of the same float32 phi:
bit-exact.  Vertex positions and normals are compared with the FP64
definitions (oracle.tsdf.marching_cubes_fp64) within the derived float32
error bounds of each vertex; as a second check they also equal, bit for
bit, the oracle's float32 evaluation in the kernel's operation order
(t = (iso - phi_a) / (phi_b - phi_a), x = c_a + t h; w = 1 - t,
n = w g_a + t g_b, n / |n|).
"""
import numpy as np
import pytest

import synth
from gpu_util import cuda, log
from oracle import gauss as og
from oracle import tsdf as ot
from paper_2509_17390_amd import Context
from paper_2509_17390_amd import rcast

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    c = Context(0)
    yield c
    c.close()


def gpu_tsdf(ctx, surf, origin, h, sigma, tau, band):
    import torch
    nz, ny, nx = surf.shape
    g = ctx.grid(origin, h, (nx, ny, nz), 0.0)
    phi = torch.full((nz, ny, nx), 7.0, dtype=torch.float32, device="cuda")
    vt = torch.full((nz, ny, nx), 9, dtype=torch.uint8, device="cuda")
    ctx.tsdf(g, cuda(surf), phi, sigma, tau, band, out_vtilde=vt)
    torch.cuda.synchronize()
    return phi.cpu().numpy(), vt.cpu().numpy(), g


def check_tsdf(ctx, surf, origin, h, sigma, tau, band, tag=""):
    phi_g, vt_g, g = gpu_tsdf(ctx, surf, origin, h, sigma, tau, band)
    phi, vt, sgn, p = ot.tsdf(surf, h, sigma, tau, band)
    np.testing.assert_array_equal(vt_g, vt)
    np.testing.assert_array_equal(phi_g.view(np.uint32), phi.view(np.uint32))
    log(f"{tag}: {surf.size} voxels, V~ {int(vt.sum())}, outside {int((sgn > 0).sum())}")
    return phi_g, g


def check_mc(ctx, phi, g, origin, h, iso, tag=""):
    """Mesh without normals, then with them: topology exact, positions and
    normals within the FP64 definitions' bounds, and equal to the float32
    evaluation bit for bit."""
    import torch
    vo, to, no = ot.marching_cubes(phi, origin, h, iso, normals=True)
    x64, n64, ptol, ntol = ot.marching_cubes_fp64(phi, origin, h, iso)
    for with_n in (False, True):
        out = ctx.marching_cubes(g, cuda(phi), iso, normals=with_n)
        torch.cuda.synchronize()
        v, t = out[0].cpu().numpy(), out[1].cpu().numpy()
        assert v.shape == vo.shape and t.shape == to.shape, (v.shape, vo.shape, t.shape, to.shape)
        np.testing.assert_array_equal(t, to)
        r_pos = np.abs(v.astype(np.float64) - x64) / ptol
        assert np.all(r_pos <= 1.0), float(r_pos.max())
        np.testing.assert_array_equal(v.view(np.uint32), vo.view(np.uint32))
        if with_n:
            n = out[2].cpu().numpy()
            r_n = np.abs(n.astype(np.float64) - n64).max(axis=1) / ntol
            assert np.all(r_n <= 1.0), float(r_n.max())
            np.testing.assert_array_equal(n.view(np.uint32), no.view(np.uint32))
    log(f"{tag}: {len(v)} vertices, {len(t)} triangles, positions and normals within bounds")
    return v, t


@pytest.mark.parametrize("seed", [0, 1])
def test_random_masks(ctx, seed):
    rng = np.random.default_rng(seed)
    surf = (rng.random((19, 23, 29)) < 0.15).astype(np.uint8)
    # smoothing of n = 2, 6, 1 and 3 steps (the tiled pass takes 1..3)
    for sigma, tau, band in ((0.02, 0.05, 0.06), (0.035, 0.2, 0.1), (0.01, 0.5, 0.02),
                             (0.025, 0.15, 0.08)):
        phi, g = check_tsdf(ctx, surf, (0.1, -0.2, 0.3), 0.02, sigma, tau, band,
                            tag=f"random {seed} sigma {sigma}")
        check_mc(ctx, phi, g, (0.1, -0.2, 0.3), 0.02, 0.0, tag=f"random {seed} mc")


def test_cavity_and_tunnel(ctx):
    surf = np.zeros((20, 21, 22), np.uint8)
    surf[3:17, 3:18, 3:19] = 1
    surf[4:16, 4:17, 4:18] = 0                        # closed shell
    phi, g = check_tsdf(ctx, surf, (0, 0, 0), 0.05, 0.001, 0.4, 0.2, tag="shell")
    assert phi[10, 10, 10] < 0                        # the cavity is not outside
    surf[10, 10, 3] = 0                               # a tunnel
    phi2, _ = check_tsdf(ctx, surf, (0, 0, 0), 0.05, 0.001, 0.4, 0.2, tag="tunnel")
    assert phi2[10, 10, 10] > 0


def test_gaussian_surface_to_mesh(ctx):
    """Surface mask from the Gaussian conversion of a region of the indoor
    scene, then TSDF and marching cubes."""
    import torch
    m, q, s, a, room = synth.splat_scene(1, 200000)
    lo = np.array([-0.1, 2.0, 0.9])
    grid = og.Grid(lo, 0.02, (44, 40, 36), tile=8, theta=0.2)
    hi = lo + 0.02 * np.array(grid.dims)
    boxes = og.gauss_boxes(m, q, s, 3.0)
    sel = np.all((boxes[:, :3] <= hi + 0.3) & (boxes[:, 3:] >= lo - 0.3), axis=1)
    gset = ctx.upload_gaussians(m[sel], q[sel], s[sel], a[sel])
    ctx.build_gaussians(gset)
    nx, ny, nz = grid.dims
    O = torch.empty((nz, ny, nx), dtype=torch.uint8, device="cuda")
    S = torch.empty((nz, ny, nx), dtype=torch.uint8, device="cuda")
    ctx.voxelize(gset, ctx.grid(lo, 0.02, grid.dims, 0.2), None, O, S)
    torch.cuda.synchronize()
    surf = S.cpu().numpy()
    ctx.release_gaussians(gset)
    phi, g = check_tsdf(ctx, surf, lo, 0.02, 0.02, 0.15, 0.06, tag="splat")
    v, t = check_mc(ctx, phi, g, lo, 0.02, 0.0, tag="splat mc")
    assert len(t) > 1000


def test_sphere_field_and_exact_iso(ctx):
    n = 31
    iz, iy, ix = np.meshgrid(np.arange(n), np.arange(n), np.arange(n), indexing="ij")
    h = 0.1
    X, Y, Z = (-1.5 + (ix + 0.5) * h, -1.5 + (iy + 0.5) * h, -1.5 + (iz + 0.5) * h)
    phi = (np.sqrt(X ** 2 + Y ** 2 + Z ** 2) - 1.1).astype(np.float32)
    import torch
    g = ctx.grid((-1.5, -1.5, -1.5), h, (n, n, n), 0.0)
    for iso in (0.0, 0.05, -0.2):
        check_mc(ctx, phi, g, (-1.5, -1.5, -1.5), h, iso, tag=f"sphere iso {iso}")
    q = np.round(phi * 10).astype(np.float32) / 10   # many corners exactly at iso
    check_mc(ctx, q, g, (-1.5, -1.5, -1.5), h, 0.0, tag="sphere quantised")


@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 2, 2), (1, 5, 7), (9, 1, 4)])
def test_tiny_grids(ctx, dims):
    rng = np.random.default_rng(sum(dims))
    nx, ny, nz = dims
    surf = (rng.random((nz, ny, nx)) < 0.5).astype(np.uint8)
    phi, g = check_tsdf(ctx, surf, (0, 0, 0), 0.1, 0.1, 0.3, 0.3, tag=f"tiny {dims}")
    check_mc(ctx, phi, g, (0, 0, 0), 0.1, 0.0, tag=f"tiny {dims} mc")


def test_constant_fields_have_no_mesh(ctx):
    import torch
    g = ctx.grid((0, 0, 0), 0.1, (10, 11, 12), 0.0)
    for val in (-1.0, 1.0, 0.0):
        phi = torch.full((12, 11, 10), val, dtype=torch.float32, device="cuda")
        v, t = ctx.marching_cubes(g, phi, 0.0)
        assert v.shape[0] == 0 and t.shape[0] == 0


def test_errors(ctx):
    import torch
    g = ctx.grid((0, 0, 0), 0.01, (8, 8, 8), 0.0)
    surf = torch.zeros((8, 8, 8), dtype=torch.uint8, device="cuda")
    phi = torch.zeros((8, 8, 8), dtype=torch.float32, device="cuda")
    for sigma, tau, band in ((0.1, 0.5, 0.02), (0.01, 0.5, 3.0), (0.0, 0.5, 0.02),
                             (0.01, float("nan"), 0.02), (0.01, 0.5, -1.0)):
        with pytest.raises(rcast.RcastError) as e:
            ctx.tsdf(g, surf, phi, sigma, tau, band)
        assert e.value.status == rcast.RC_E_INVAL
    # capacity too small: sizes are still reported
    field = torch.ones((8, 8, 8), dtype=torch.float32, device="cuda")
    field[3:5, 3:5, 3:5] = -1.0
    import ctypes
    lib = rcast.load()
    nv, nt = ctypes.c_int64(), ctypes.c_int64()
    V = torch.empty((1, 3), dtype=torch.float32, device="cuda")
    T = torch.empty((1, 3), dtype=torch.int32, device="cuda")
    st = lib.rc_marching_cubes(ctx._h, ctypes.byref(g), field.data_ptr(), 0.0, V.data_ptr(),
                               T.data_ptr(), None, 1, 1, ctypes.byref(nv), ctypes.byref(nt),
                               torch.cuda.current_stream().cuda_stream)
    assert st == rcast.RC_E_NOMEM and nv.value > 1 and nt.value > 1
    st = lib.rc_marching_cubes(ctx._h, ctypes.byref(g), field.data_ptr(), 0.0, V.data_ptr(),
                               None, None, 1, 1, ctypes.byref(nv), ctypes.byref(nt),
                               torch.cuda.current_stream().cuda_stream)
    assert st == rcast.RC_E_INVAL


@pytest.mark.parametrize("dims", [(150, 40, 37), (128, 17, 33), (65, 70, 18), (70, 530, 12),
                                  (66, 12, 600)])
def test_wide_rows_and_long_columns(ctx, dims):
    """Rows of several 64-voxel words (ragged and exact) and columns of
    several 16-row segments, for the packed outside labelling, with both
    smoothing paths (n = 2 and n = 6), then marching cubes.  Columns of up
    to 32 segments take the one-kernel column pass, longer ones (530 rows
    along y, 600 along z) the three-kernel one."""
    nx, ny, nz = dims
    rng = np.random.default_rng(nx + ny + nz)
    surf = (rng.random((nz, ny, nx)) < 0.12).astype(np.uint8)
    # a closed box shell with one hole: its inside is reached only through it
    surf[4:nz - 4, 5:ny - 5, 6:nx - 6] = 1
    surf[5:nz - 5, 6:ny - 6, 7:nx - 7] = 0
    surf[nz // 2, ny // 2, 6] = 0
    for sigma, tau, band in ((0.02, 0.15, 0.06), (0.035, 0.2, 0.1)):
        phi, g = check_tsdf(ctx, surf, (0.05, 0.0, -0.1), 0.02, sigma, tau, band,
                            tag=f"wide {dims} sigma {sigma}")
    check_mc(ctx, phi, g, (0.05, 0.0, -0.1), 0.02, 0.0, tag=f"wide {dims} mc")


def test_unaligned_output_buffers(ctx):
    """The surface mask, phi and V~ as views one element into larger
    buffers (not 4- / 16-byte aligned): the library falls back to its
    element-wise paths and the results stay bit-exact."""
    import torch
    nz, ny, nx = 21, 26, 70
    rng = np.random.default_rng(5)
    surf = (rng.random((nz, ny, nx)) < 0.15).astype(np.uint8)
    g = ctx.grid((0.1, -0.2, 0.3), 0.02, (nx, ny, nz), 0.0)
    n = nx * ny * nz
    phi_buf = torch.full((n + 1,), 7.0, dtype=torch.float32, device="cuda")
    vt_buf = torch.full((n + 1,), 9, dtype=torch.uint8, device="cuda")
    phi = phi_buf[1:].view(nz, ny, nx)
    vt = vt_buf[1:].view(nz, ny, nx)
    assert phi.data_ptr() % 16 != 0 and vt.data_ptr() % 4 != 0
    surf_buf = torch.zeros((n + 1,), dtype=torch.uint8, device="cuda")
    surf_buf[1:] = cuda(surf).reshape(-1)
    surf_d = surf_buf[1:].view(nz, ny, nx)
    ctx.tsdf(g, surf_d, phi, 0.02, 0.15, 0.06, out_vtilde=vt)
    torch.cuda.synchronize()
    phi_o, vt_o, _, _ = ot.tsdf(surf, 0.02, 0.02, 0.15, 0.06)
    np.testing.assert_array_equal(vt.cpu().numpy(), vt_o)
    np.testing.assert_array_equal(phi.cpu().numpy().view(np.uint32), phi_o.view(np.uint32))
    # the elements before the views are untouched
    assert float(phi_buf[0]) == 7.0 and int(vt_buf[0]) == 9


# ---- quantile re-threshold and mc_step -------------------------------------

@pytest.mark.parametrize("q", [0.0, 0.35, 0.5, 0.93, 1.0])
def test_quantile_rethreshold(ctx, q):
    # V~ = [V' >= Quantile_q(V')] decided on the exact integer sums: V~ and
    # phi bit-exact with the oracle, on a ragged grid with a 2-step kernel
    import torch
    rng = np.random.default_rng(21)
    surf = (rng.random((13, 17, 29)) < 0.2).astype(np.uint8)
    h, sigma, band = 0.05, 0.05, 0.15
    nz, ny, nx = surf.shape
    g = ctx.grid((0.1, -0.3, 0.0), h, (nx, ny, nz), 0.0)
    phi = torch.full((nz, ny, nx), 7.0, dtype=torch.float32, device="cuda")
    vt = torch.full((nz, ny, nx), 9, dtype=torch.uint8, device="cuda")
    ctx.tsdf(g, cuda(surf), phi, sigma, 0.0, band, out_vtilde=vt, quantile=q)
    torch.cuda.synchronize()
    phi_o, vt_o, _, _ = ot.tsdf(surf, h, sigma, 0.0, band, quantile=q)
    np.testing.assert_array_equal(vt.cpu().numpy(), vt_o)
    np.testing.assert_array_equal(phi.cpu().numpy().view(np.uint32), phi_o.view(np.uint32))
    log(f"quantile {q}: V~ {int(vt_o.sum())} of {surf.size}")


def test_quantile_rethreshold_large_kernel(ctx):
    # 8-step kernel: sums up to 2^48, many distinct values
    import torch
    rng = np.random.default_rng(22)
    surf = (rng.random((20, 24, 30)) < 0.15).astype(np.uint8)
    h, sigma, band = 0.02, 0.04, 0.06
    nz, ny, nx = surf.shape
    g = ctx.grid((0.0, 0.0, 0.0), h, (nx, ny, nz), 0.0)
    phi = torch.empty((nz, ny, nx), dtype=torch.float32, device="cuda")
    vt = torch.empty((nz, ny, nx), dtype=torch.uint8, device="cuda")
    for q in (0.6, 0.85):
        ctx.tsdf(g, cuda(surf), phi, sigma, 0.0, band, out_vtilde=vt, quantile=q)
        torch.cuda.synchronize()
        phi_o, vt_o, _, _ = ot.tsdf(surf, h, sigma, 0.0, band, quantile=q)
        np.testing.assert_array_equal(vt.cpu().numpy(), vt_o)
        np.testing.assert_array_equal(phi.cpu().numpy().view(np.uint32), phi_o.view(np.uint32))


def test_quantile_rejects_bad_values(ctx):
    import torch
    surf = np.zeros((4, 4, 4), np.uint8)
    g = ctx.grid((0, 0, 0), 0.1, (4, 4, 4), 0.0)
    phi = torch.empty((4, 4, 4), dtype=torch.float32, device="cuda")
    for q in (-0.1, 1.5, float("nan")):
        with pytest.raises(rcast.RcastError) as e:
            ctx.tsdf(g, cuda(surf), phi, 0.1, 0.0, 0.2, quantile=q)
        assert e.value.status == rcast.RC_E_INVAL


@pytest.mark.parametrize("step", [1, 2, 3, 5])
def test_mc_step(ctx, step):
    # marching cubes on every step-th lattice point: topology, numbering and
    # float32 positions and normals bit-exact with the oracle's evaluation
    # on the coarse lattice, positions within the FP64 definition's bounds
    import torch
    rng = np.random.default_rng(30 + step)
    surf = (rng.random((26, 31, 37)) < 0.05).astype(np.uint8)
    origin, h = (0.25, -0.5, 0.125), 0.04
    phi, g = check_tsdf(ctx, surf, origin, h, 0.04, 0.1, 0.16, tag=f"mc_step {step} field")
    vo, to, no = ot.marching_cubes_step(phi, origin, h, step, 0.0, normals=True)
    hs = float(np.float32(np.float32(h) * np.float32(step)))
    o2 = tuple(float(np.float32(float(np.float32(o)) - (step - 1) * float(np.float32(h)) / 2.0))
               for o in origin)
    coarse = np.ascontiguousarray(phi[::step, ::step, ::step])
    x64, n64, ptol, ntol = ot.marching_cubes_fp64(coarse, o2, hs, 0.0)
    v, t, n = ctx.marching_cubes(g, cuda(phi), 0.0, normals=True, step=step)
    torch.cuda.synchronize()
    v, t, n = v.cpu().numpy(), t.cpu().numpy(), n.cpu().numpy()
    np.testing.assert_array_equal(t, to)
    np.testing.assert_array_equal(v.view(np.uint32), vo.view(np.uint32))
    np.testing.assert_array_equal(n.view(np.uint32), no.view(np.uint32))
    assert np.all(np.abs(v.astype(np.float64) - x64) <= ptol)
    log(f"mc_step {step}: {len(v)} vertices, {len(t)} triangles")


def test_mc_step_rejects_zero(ctx):
    surf = np.zeros((4, 4, 4), np.float32)
    g = ctx.grid((0, 0, 0), 0.1, (4, 4, 4), 0.0)
    with pytest.raises(rcast.RcastError) as e:
        ctx.marching_cubes(g, cuda(surf), 0.0, step=0)
    assert e.value.status == rcast.RC_E_INVAL


def test_marching_cubes_many_scan_tiles(ctx):
    # 9.2M lattice points: 9,000 scan tiles of 1,024 points, more than the
    # 8,192 tile totals one LDS chunk of the tile-offset scan holds, so the
    # scan carries its running totals across chunks; two spheres, compared
    # bit for bit with the oracle's float32 evaluation
    import torch
    nz, ny, nx = 96, 300, 320
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    phi = (np.minimum(np.sqrt((x - 100.3) ** 2 + (y - 150.2) ** 2 + (z - 48.1) ** 2) - 40.7,
                      np.sqrt((x - 230.6) ** 2 + (y - 120.4) ** 2 + (z - 50.3) ** 2) - 35.2)
           * 0.01).astype(np.float32)
    g = ctx.grid((0.0, 0.0, 0.0), 0.01, (nx, ny, nz), 0.0)
    log(f"marching cubes on {phi.size} points")
    vg, tg, ng = ctx.marching_cubes(g, torch.from_numpy(phi).cuda(), 0.0, normals=True)
    torch.cuda.synchronize()
    vo, to, no = ot.marching_cubes(phi, (0.0, 0.0, 0.0), 0.01, 0.0, normals=True)
    assert len(to) > 100_000
    np.testing.assert_array_equal(tg.cpu().numpy(), to)
    np.testing.assert_array_equal(vg.cpu().numpy().view(np.uint32), vo.view(np.uint32))
    np.testing.assert_array_equal(ng.cpu().numpy().view(np.uint32), no.view(np.uint32))


@pytest.mark.parametrize("shape,share", [
    ((2, 2, 2), 0.5), ((1, 5, 7), 0.5), ((5, 3, 1), 0.5), ((3, 4, 63), 0.5), ((3, 4, 64), 0.5),
    ((3, 5, 65), 0.5), ((2, 130, 129), 0.5), ((3, 64, 86), 0.02), ((17, 31, 63), 0.001),
    ((40, 90, 130), 0.5), ((40, 90, 130), 0.003)])
def test_marching_cubes_word_edges(ctx, shape, share):
    # rows that begin anywhere in a 64-point word, grids of one and of many
    # 256-word blocks, words of 0 to 192 vertices in groups of one to eight:
    # a lattice of independent signs, `share` of them inside
    rng = np.random.default_rng(sum(shape))
    mag = rng.uniform(0.1, 1.0, shape).astype(np.float32)
    phi = np.where(rng.random(shape) < share, -mag, mag)
    phi.reshape(-1)[0] = -0.5
    nz, ny, nx = shape
    g = ctx.grid((0.5, -0.25, 0.125), 0.25, (nx, ny, nz), 0.0)
    log(f"marching cubes, {shape}, {share}")
    check_mc(ctx, phi, g, (0.5, -0.25, 0.125), 0.25, 0.0, tag=f"{shape}")


def test_marching_cubes_scan_of_many_blocks(ctx):
    # 80M lattice points: 4,900 blocks of 16,384, more than the 4,096 one LDS
    # chunk of the offset scan holds.  Two balls, in the first and the last
    # layers; the spacing is a power of two, so the last one's mesh is that of
    # its own layers moved by whole voxels, with its ids behind the first one's
    import torch
    nz, ny, nx = 80, 1000, 1001
    phi = torch.ones((nz, ny, nx), dtype=torch.float32, device="cuda")
    z, y, x = np.meshgrid(np.arange(12), np.arange(60), np.arange(70), indexing="ij")
    ball = (np.sqrt((x - 31.3) ** 2 + (y - 28.2) ** 2 + (z - 5.1) ** 2) - 4.4).astype(np.float32)
    part = np.full((12, ny, nx), 1.0, np.float32)
    part[:, 300:360, 500:570] = np.minimum(ball, 1.0)
    phi[:12] = torch.from_numpy(part).cuda()
    phi[-12:] = torch.from_numpy(part).cuda()
    g = ctx.grid((0.0, 0.0, 0.0), 0.5, (nx, ny, nz), 0.0)
    log(f"marching cubes on {phi.numel()} points")
    vg, tg = ctx.marching_cubes(g, phi, 0.0)
    sub = part[:, 295:365, 495:575]
    v0, t0 = ot.marching_cubes(sub, (495 * 0.5, 295 * 0.5, 0.0), 0.5, 0.0)
    v1, t1 = ot.marching_cubes(sub, (495 * 0.5, 295 * 0.5, (nz - 12) * 0.5), 0.5, 0.0)
    np.testing.assert_array_equal(vg.cpu().numpy(), np.concatenate([v0, v1]))
    np.testing.assert_array_equal(tg.cpu().numpy(), np.concatenate([t0, t1 + len(v0)]))


@pytest.mark.parametrize("shape", [
    (1, 1, 1), (2, 3, 5), (1, 17, 64), (16, 16, 65), (17, 33, 63), (18, 15, 130), (3, 9, 577),
    (33, 2, 1), (2, 577, 40), (2, 3073, 65)])
def test_bit_words_and_tiles(ctx, shape):
    # words of one to 64 voxels, rows of one to ten words (more than a sweep
    # reads together), rows of a slice on either side of its threads and of a
    # lane's nine, a slice that does not fit LDS; smoothing of 1 to 3 steps on
    # bits and of 4 by voxels, 1 to 4 shells on bits and 5 by voxels, with and
    # without V~; masks between open and closed, the second time of any
    # non-zero bytes, which count as 1 (the oracle adds up the mask's values
    # and takes 0 and 1)
    import torch
    h = 0.5
    rng = np.random.default_rng(sum(shape))
    nz, ny, nx = shape
    for n, shells in ((1, 1), (1, 3), (2, 2), (3, 4), (1, 5), (4, 3)):
        sigma, band = h * float(np.sqrt(n / 2)), (shells - 0.5) * h
        surf = np.where(rng.random(shape) < 0.45, rng.integers(1, 256, shape), 0).astype(np.uint8)
        log(f"{shape}: n = {n}, {shells} shells")
        phi, g = check_tsdf(ctx, (surf != 0).astype(np.uint8), (0.25, 0.5, -0.125), h, sigma, 0.46, band, tag=f"{shape}")
        alone = torch.empty(shape, dtype=torch.float32, device="cuda")
        ctx.tsdf(g, cuda(surf), alone, sigma, 0.46, band)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(alone.cpu().numpy().view(np.uint32), phi.view(np.uint32))


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 63), (2, 1, 64), (5, 4, 65), (7, 3, 130),
                                   (2, 3, 577)])
def test_quantile_words(ctx, shape):
    # quantile threshold straight to words: rows about a word's 64 voxels, word
    # counts that a wave's four do and do not divide, with and without V~, and
    # with the shells that read V~ bytes (5)
    import torch
    h = 0.5
    surf = (np.random.default_rng(sum(shape)).random(shape) < 0.3).astype(np.uint8)
    nz, ny, nx = shape
    g = ctx.grid((0.0, 0.0, 0.0), h, (nx, ny, nz), 0.0)
    for q, shells in ((0.4, 2), (0.9, 4), (0.7, 5)):
        sigma, band = h, (shells - 0.5) * h
        log(f"{shape}: quantile {q}, {shells} shells")
        phi_o, vt_o, _, _ = ot.tsdf(surf, h, sigma, 0.0, band, quantile=q)
        for vt in (None, torch.full(shape, 9, dtype=torch.uint8, device="cuda")):
            phi = torch.full(shape, 7.0, dtype=torch.float32, device="cuda")
            ctx.tsdf(g, cuda(surf), phi, sigma, 0.0, band, out_vtilde=vt, quantile=q)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(phi.cpu().numpy().view(np.uint32), phi_o.view(np.uint32))
        np.testing.assert_array_equal(vt.cpu().numpy(), vt_o)


@pytest.mark.parametrize("short", ["verts", "tris"])
def test_marching_cubes_writes_nothing_beyond_capacity(ctx, short):
    # one entry short in either array: the sizes come back, nothing is written;
    # with just enough the mesh is the one extracted with room to spare
    import ctypes

    import torch
    rng = np.random.default_rng(31)
    field = cuda(rng.standard_normal((9, 20, 70)).astype(np.float32))
    g = ctx.grid((0.0, 0.0, 0.0), 0.5, (70, 20, 9), 0.0)
    v, t = ctx.marching_cubes(g, field, 0.0)
    lib = rcast.load()
    for less in (1, 0):
        nv, nt = ctypes.c_int64(), ctypes.c_int64()
        V = torch.full((len(v) + 1, 3), -7.0, dtype=torch.float32, device="cuda")
        T = torch.full((len(t) + 1, 3), -7, dtype=torch.int32, device="cuda")
        cv = len(v) - (less if short == "verts" else 0)
        ct = len(t) - (less if short == "tris" else 0)
        st = lib.rc_marching_cubes(ctx._h, ctypes.byref(g), field.data_ptr(), 0.0, V.data_ptr(),
                                   T.data_ptr(), None, cv, ct, ctypes.byref(nv),
                                   ctypes.byref(nt), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert (nv.value, nt.value) == (len(v), len(t))
        if less:
            assert st == rcast.RC_E_NOMEM
            assert bool((V == -7.0).all()) and bool((T == -7).all())
        else:
            assert st == rcast.RC_OK
            assert torch.equal(V[:-1], v) and torch.equal(T[:-1], t)
            assert bool((V[-1] == -7.0).all()) and bool((T[-1] == -7).all())


@pytest.mark.parametrize("shape", [(9, 10, 64), (10, 9, 65), (19, 73, 130), (73, 18, 20),
                                   (576, 5, 40), (577, 5, 40), (5, 576, 70), (96, 95, 64),
                                   (96, 96, 64), (4, 3, 3700)])
def test_labelling_by_one_block(ctx, shape):
    # columns about a lane's run of 9 and a wave's 576, rows of 1 to 58 words,
    # grids on either side of what one block holds; noise, and a passage that
    # goes to and fro through walls with one hole each (a round or two a wall)
    nz, ny, nx = shape
    rng = np.random.default_rng(nz + ny + nx)
    passage = np.zeros(shape, np.uint8)
    passage[:, [0, -1]] = 1
    passage[:, :, [0, -1]] = 1
    passage[0] = passage[-1] = 1
    for i, z in enumerate(range(0, nz, 3)):
        passage[z] = 1
        passage[z, 1 if i % 2 else -2, 1 if i % 2 else -2] = 0
    h = 0.5
    for surf, sigma, tau in (((rng.random(shape) < 0.3).astype(np.uint8), h, 0.3),
                             (passage, 0.25 * h, 0.5)):
        log(f"{shape}: {int(surf.sum())} set")
        check_tsdf(ctx, surf, (0.25, 0.5, -0.125), h, sigma, tau, 2 * h, tag=f"{shape}")


@pytest.mark.parametrize("shape", [((1 << 23) + 3, 1, 1), (1_100_000, 3, 2)])
def test_thin_grids_of_many_tiles(ctx, shape):
    # tiles of 16 and 96 voxels, more than one row of a launch's blocks; more
    # slices than a launch has blocks of a sweep
    rng = np.random.default_rng(sum(shape))
    surf = (rng.random(shape, dtype=np.float32) < 0.6).astype(np.uint8)
    log(f"{shape}")
    check_tsdf(ctx, surf, (0.0, 0.0, 0.0), 0.5, 0.35, 0.2, 1.0, tag=f"{shape}")


@pytest.mark.parametrize("shape", [(1024, 20, 33), (1025, 20, 33), (1030, 255, 190), (1030, 256, 190),
                                   (40, 768, 190), (40, 769, 190)])
def test_sweeps_by_slices_and_by_rows(ctx, shape):
    # the last grid of few slices and the next one, slices of 765 and 768 words
    # among many, and slices of 2,304 and 2,307 (four blocks a CU or one)
    rng = np.random.default_rng(sum(shape))
    surf = (rng.random(shape, dtype=np.float32) < 0.3).astype(np.uint8)
    log(f"{shape}")
    check_tsdf(ctx, surf, (0.0, 0.0, 0.0), 0.5, 0.5, 0.3, 1.0, tag=f"{shape}")


def test_scratch_holds_the_mesh_extraction(ctx):
    # a new context's scratch is allocated once for a field and its mesh; a
    # budget that has room for the field alone still gives the field
    import torch
    shape = (60, 70, 80)
    surf = cuda((np.random.default_rng(3).random(shape) < 0.3).astype(np.uint8))
    phi = torch.empty(shape, dtype=torch.float32, device="cuda")
    tiny = torch.ones((2, 2, 2), dtype=torch.float32, device="cuda")
    used = []
    for budget in (0, 1):
        c = rcast.Context(0, budget_bytes=used[0] - 1 if budget else 0)
        c.marching_cubes(c.grid((0, 0, 0), 0.5, (2, 2, 2), 0.0), tiny, 0.0)    # the case table
        g = c.grid((0, 0, 0), 0.5, shape[::-1], 0.0)
        phi.fill_(9.0)
        c.tsdf(g, surf, phi, 0.4, 0.3, 1.5)
        torch.cuda.synchronize()
        used.append(c.device_bytes())
        assert bool((phi != 9.0).all())
        if not budget:
            first = phi.clone()
            c.marching_cubes(g, phi, 0.0)
            assert c.device_bytes() == used[0]
        else:
            assert torch.equal(phi, first) and used[1] < used[0]
        c.close()
