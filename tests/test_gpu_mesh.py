"""Surface extraction on the device against the FP64 oracle (oracle/mesh.py).

Marching tetrahedra decides inside/outside by phi < 0; on identical float32
lattices both sides take the same decisions, so the triangle count is exact
and the triangles agree to float32 rounding of the crossing points.  The SDF
lattice is compared at the same float32 lattice positions to the forward
tolerance.
"""
import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

import synth
from oracle import mesh as MS
from tests.helpers import FWD_TOL, check_close, sphere_case

pytestmark = pytest.mark.gpu

OB3 = 2112            # packed offset of the geometry decoder's output bias (b3[0] is phi's)


def _G():
    from paper_2206_14735_amd import gosurf as G
    G.lib()
    return G


def _area(t):
    t = np.asarray(t, dtype=np.float64)
    return 0.5 * np.linalg.norm(np.cross(t[:, 1] - t[:, 0], t[:, 2] - t[:, 0]), axis=1).sum()


def _f32_lattice(p0, h, dims):
    """Lattice positions rounded as the device forms them (float32 i*h, then + p0)."""
    nx, ny, nz = dims
    h32 = np.float32(h)
    ax = [np.float32(np.float32(np.arange(n, dtype=np.float32) * h32) + np.float32(p0[a]))
          for a, n in enumerate((nx, ny, nz))]
    z, y, x = np.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    return np.stack([x, y, z], -1).reshape(-1, 3).astype(np.float64)


def _compare_meshes(got, count, ref, tol):
    assert count == len(ref), (count, len(ref))
    cg = np.asarray(got, np.float64).mean(1)
    cr = ref.mean(1)
    d1, _ = cKDTree(cr).query(cg)
    d2, _ = cKDTree(cg).query(cr)
    print(f"{count} triangles; centroid distance max {max(d1.max(), d2.max()):.2e}", flush=True)
    assert d1.max() <= tol and d2.max() <= tol
    assert _area(got) == pytest.approx(_area(ref), rel=1e-5)


def test_marching_tetrahedra_matches_oracle_on_an_identical_lattice():
    G = _G()
    rng = np.random.default_rng(8)
    dims = (37, 29, 23)                     # ragged against 256-thread blocks
    h, p0 = 0.05, (-0.9, -0.7, -0.55)
    x = MS.lattice_points(p0, h, dims)
    phi = (np.linalg.norm(x - [0.05, -0.02, 0.0], axis=1) - 0.45) + 0.03 * np.sin(7 * x[:, 0]) * np.cos(5 * x[:, 1])
    phi = np.float32(phi + 0.002 * rng.standard_normal(phi.shape)).reshape(dims[2], dims[1], dims[0])
    ref = MS.marching_tetrahedra(np.float64(phi), p0, h)
    tris, cnt = G.gosurf_marching_tetrahedra(torch.as_tensor(phi).cuda(), p0, h, max_triangles=len(ref) + 100)
    torch.cuda.synchronize()
    n = G.triangle_count(cnt)
    _compare_meshes(tris[:n].cpu().numpy(), n, ref, 1e-5)


def test_marching_tetrahedra_reports_overflow_and_writes_within_capacity():
    G = _G()
    dims = (20, 20, 20)
    h, p0 = 0.1, (-1.0, -1.0, -1.0)
    x = MS.lattice_points(p0, h, dims)
    phi = np.float32(np.linalg.norm(x, axis=1) - 0.6).reshape(20, 20, 20)
    ref = MS.marching_tetrahedra(np.float64(phi), p0, h)
    cap = len(ref) // 3
    guard = torch.full((cap + 50, 3, 3), 7.0, device="cuda")
    tris, cnt = G.gosurf_marching_tetrahedra(torch.as_tensor(phi).cuda(), p0, h, max_triangles=cap,
                                             triangles=guard)
    torch.cuda.synchronize()
    assert G.triangle_count(cnt) == len(ref)
    assert torch.all(guard[cap:] == 7.0)     # nothing written past the capacity
    assert torch.all(guard[:cap].abs() <= 1.0)


def test_sdf_lattice_matches_oracle_over_several_slabs():
    G = _G()
    # the unshifted field: phi stays away from 0 (0.04-0.15), where the forward
    # tolerance applies entry by entry; near 0, phi is a difference of terms of
    # ~0.1 and carries their float32 rounding (~1e-7) as absolute error
    L, fr, b, grid, mlp = sphere_case(M=8, S=0, grid_std=0.3)
    dims = (23, 19, 17)
    h = 0.09
    p0 = (L.p0[0] + 0.013, L.p0[1] + 0.021, L.p0[2] + 0.007)
    model = G.make_model(L)
    ws = torch.empty(G.gosurf_lattice_workspace_bytes(dims[0], dims[1], 5), dtype=torch.uint8, device="cuda")
    phi = G.gosurf_sdf_lattice(model, grid.cuda().contiguous(), mlp.cuda().contiguous(), p0, h, dims, workspace=ws)
    torch.cuda.synchronize()
    x = _f32_lattice(p0, h, dims)
    assert np.all(x <= np.asarray(L.p1)) and np.all(x >= np.asarray(L.p0))
    ref = MS.field_sdf(grid.numpy(), mlp.numpy(), L)(x)
    check_close("lattice phi", phi.cpu().numpy().reshape(-1), ref, FWD_TOL)


@pytest.mark.parametrize("dims", [(2, 2, 2), (2, 3, 7), (3, 2, 41), (15, 4, 2), (16, 3, 3), (17, 2, 5), (33, 31, 4)])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_lattice_rows_of_any_length(dims, precision):
    """Tiles of 16 points run over row and layer ends.  In FP32 the points match
    the oracle; in BF16, where the lattice's layers are those of the forward,
    they equal its SDF at the same points bit for bit, outside the box too."""
    from oracle import step as ostep
    G = _G()
    L, fr, b, grid, mlp = sphere_case(M=8, S=0, grid_std=0.3)
    nx, ny, nz = dims
    prec = G.BF16 if precision == "bf16" else G.FP32
    h = 0.05 if prec == G.FP32 else 0.2
    p0 = (L.p0[0] + 0.013, L.p0[1] + 0.021, L.p0[2] + 0.007)
    g, m = grid.cuda().contiguous(), mlp.cuda().contiguous()
    model = G.make_model(L, prec)
    kw = {}
    if prec == G.BF16:
        kw["grid_bf16"] = torch.empty(g.shape, dtype=torch.bfloat16, device="cuda")
        G.gosurf_refresh_bf16(g, kw["grid_bf16"])
    phi = G.gosurf_sdf_lattice(model, g, m, p0, h, dims, **kw).cpu().numpy().reshape(-1)
    x = _f32_lattice(p0, h, dims)
    if prec == G.FP32:
        assert np.all(x <= np.asarray(L.p1)) and np.all(x >= np.asarray(L.p0))
        check_close("lattice phi", phi, MS.field_sdf(grid.numpy(), mlp.numpy(), L)(x), FWD_TOL)
        return
    o = x.reshape(nz * ny, nx, 3)[:, 0].astype(np.float32)
    r = np.tile(np.float32([1, 0, 0]), (nz * ny, 1))
    t = np.tile(np.arange(nx, dtype=np.float32) * np.float32(h), nz * ny)
    zero = np.zeros((0, 3), np.float32)
    rays = ostep.Batch(o, r, np.zeros_like(o), np.zeros(nz * ny, np.float32), t,
                       np.arange(0, nx * ny * nz + 1, nx, dtype=np.int32), zero, zero)
    db = G.RayBatch.from_host(rays)
    out = G.gosurf_forward(model, g, m, db, G.make_loss_cfg((10.0, 1.0, 10.0, 1.0, 0.0, 0.0)),
                           G.workspace_for(model, db.M, db.total, db.S), **kw)
    ref = out.sample_values(db.total)[0].cpu().numpy()
    assert np.array_equal(phi, ref)


def test_mesh_of_the_field_matches_oracle():
    G = _G()
    L, fr, b, grid, mlp = sphere_case(M=8, S=0, grid_std=0.3)
    mlp[OB3] -= 0.095     # shift phi so that its zero level set runs through the lattice
    dims = (41, 41, 41)
    h = 0.045
    p0 = (L.p0[0] + 0.01, L.p0[1] + 0.01, L.p0[2] + 0.01)
    model = G.make_model(L)
    phi = G.gosurf_sdf_lattice(model, grid.cuda().contiguous(), mlp.cuda().contiguous(), p0, h, dims)
    ref_phi = MS.field_sdf(grid.numpy(), mlp.numpy(), L)(_f32_lattice(p0, h, dims)).reshape(dims[2], dims[1], dims[0])
    ref = MS.marching_tetrahedra(ref_phi, p0, h)
    assert len(ref) > 100
    tris, cnt = G.gosurf_marching_tetrahedra(phi, p0, h, max_triangles=2 * len(ref) + 1000)
    torch.cuda.synchronize()
    n = G.triangle_count(cnt)
    got = tris[:n].cpu().numpy()
    # the SDF differs by float32 rounding, so a few lattice values near 0 may change sign
    near_zero = float(np.mean(np.abs(ref_phi) < 1e-5))
    print(f"device {n} triangles, oracle {len(ref)}; lattice values within 1e-5 of 0: {near_zero:.2e}", flush=True)
    assert abs(n - len(ref)) <= max(2, 0.001 * len(ref))
    d, _ = cKDTree(ref.mean(1)).query(np.float64(got).mean(1))
    assert np.mean(d <= 1e-4) >= 0.999


@pytest.mark.parametrize("corner,count", [(0, 6), (7, 6), (1, 2), (6, 2)])
def test_single_cube(corner, count):
    G = _G()
    phi = np.ones((2, 2, 2), dtype=np.float32)
    bx, by, bz = corner & 1, (corner >> 1) & 1, (corner >> 2) & 1
    phi[bz, by, bx] = -1.0
    ref = MS.marching_tetrahedra(np.float64(phi), (0.0, 0.0, 0.0), 1.0)
    assert len(ref) == count
    tris, cnt = G.gosurf_marching_tetrahedra(torch.as_tensor(phi).cuda(), (0.0, 0.0, 0.0), 1.0, max_triangles=16)
    torch.cuda.synchronize()
    _compare_meshes(tris[:G.triangle_count(cnt)].cpu().numpy(), G.triangle_count(cnt), ref, 1e-6)


def test_count_only_call():
    G = _G()
    dims = (16, 16, 16)
    h, p0 = 0.1, (-0.8, -0.8, -0.8)
    x = MS.lattice_points(p0, h, dims)
    phi = np.float32(np.linalg.norm(x, axis=1) - 0.5).reshape(16, 16, 16)
    ref = MS.marching_tetrahedra(np.float64(phi), p0, h)
    empty = torch.empty(0, 3, 3, device="cuda")
    _, cnt = G.gosurf_marching_tetrahedra(torch.as_tensor(phi).cuda(), p0, h, max_triangles=0, triangles=empty)
    torch.cuda.synchronize()
    assert G.triangle_count(cnt) == len(ref)


def test_bf16_lattice_and_importance_follow_fp32():
    """The BF16 paths (gathers from the bfloat16 mirror, bf16 decoders) of the SDF lattice and of the
    importance sampler stay within bfloat16 error of the FP32 paths."""
    G = _G()
    L, fr, b, grid, mlp = sphere_case(M=128, S=0, grid_std=0.3)
    g, m = grid.cuda().contiguous(), mlp.cuda().contiguous()
    gb = torch.empty(g.shape, dtype=torch.bfloat16, device="cuda")
    G.gosurf_refresh_bf16(g, gb)
    m32, m16 = G.make_model(L, G.FP32), G.make_model(L, G.BF16)
    dims, h = (21, 19, 17), 0.1
    p0 = (L.p0[0] + 0.02, L.p0[1] + 0.02, L.p0[2] + 0.02)
    phi32 = G.gosurf_sdf_lattice(m32, g, m, p0, h, dims)
    phi16 = G.gosurf_sdf_lattice(m16, g, m, p0, h, dims, grid_bf16=gb)
    db = G.RayBatch.from_host(b)
    cfg = G.make_importance_cfg(seed=3, step=2)
    out32 = G.gosurf_importance_sample(m32, g, m, db, cfg)
    t32 = out32.t.clone()
    out16 = G.gosurf_importance_sample(m16, g, m, db, cfg, grid_bf16=gb)
    torch.cuda.synchronize()
    scale = float(phi32.abs().max())
    err = float((phi16 - phi32).abs().max()) / scale
    print(f"BF16 lattice phi: max error {err:.2e} of the largest |phi|", flush=True)
    assert 0 < err < 0.05
    n0 = b.t.size // 128
    t16 = out16.t.view(128, -1)
    assert torch.all(t16[:, 1:] >= t16[:, :-1])
    assert torch.equal(out16.seg, out32.seg)
    d = (t16 - t32.view(128, -1)).abs()
    print(f"BF16 importance depths: median difference {float(d.median()):.2e} m", flush=True)
    assert float(d.median()) < 1e-2
    assert t16.shape[1] == n0 + 36


def test_lattice_of_several_launches():
    """A layer of 2^28 points fills a launch, so that the second layer has one of
    its own: points drawn from both match the oracle (a layer's step moves phi by
    more than the tolerance)."""
    G = _G()
    L, fr, b, grid, mlp = sphere_case(M=8, S=0, grid_std=0.3)
    dims, h = (1 << 14, 1 << 14, 2), 2.5 / (1 << 14)
    p0 = (L.p0[0] + 0.013, L.p0[1] + 0.021, L.p0[2] + 0.077)
    ws = torch.empty(G.gosurf_lattice_workspace_bytes(dims[0], dims[1], 1), dtype=torch.uint8, device="cuda")
    phi = G.gosurf_sdf_lattice(G.make_model(L), grid.cuda().contiguous(), mlp.cuda().contiguous(), p0, h, dims,
                               workspace=ws)
    rng = np.random.default_rng(3)
    i, j, k = rng.integers(0, dims[0], 4096), rng.integers(0, dims[1], 4096), rng.integers(0, 2, 4096)
    i[:4], j[:4], k[:4] = (0, dims[0] - 1, 0, dims[0] - 1), (0, dims[1] - 1, 0, dims[1] - 1), (0, 0, 1, 1)
    got = phi[torch.from_numpy(k).cuda(), torch.from_numpy(j).cuda(), torch.from_numpy(i).cuda()].cpu().numpy()
    f = np.float32
    x = np.stack([f(n) * f(h) + f(p) for n, p in zip((i, j, k), p0)], 1)
    assert np.all(x <= np.asarray(L.p1)) and np.all(x >= np.asarray(L.p0))
    ref = MS.field_sdf(grid.numpy(), mlp.numpy(), L)(x)
    moved = MS.field_sdf(grid.numpy(), mlp.numpy(), L)(x - np.array([0, 0, h]) * k[:, None])
    assert np.median(np.abs(moved - ref)[k == 1] / np.abs(ref)[k == 1]) > 10 * FWD_TOL
    check_close("lattice phi", got, ref, FWD_TOL)
