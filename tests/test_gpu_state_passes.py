"""Passes over the whole state beside the step: the diagnostics where the
tiles outnumber the rows of the reduction buffer, the first collision that
lbm_init makes in its own launch, and the grid transfers at the edges of
their tiles."""
import numpy as np
import pytest

from oracle import coupling_oracle as co

from gpu_common import gpu_fields, say
from paper_2407_12263_amd import inputs, lbm

pytestmark = pytest.mark.gpu

SCALE = np.array([1.0, 0.02, 0.02, 0.02, 4e-4] + [1.0] * 11, dtype=np.float32)


@pytest.fixture(scope="module")
def sur():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_12263_amd import surrogate
    surrogate.load_library()
    return surrogate


def _fields(nx, ny, nz, seed):
    rng = np.random.default_rng(seed)
    shape = (nz, ny, nx)
    return 0.5 + 0.4 * rng.random(shape), 0.01 * (1 + rng.random((3,) + shape)), 1e-4 * rng.random(shape)


# more tiles than nx ceil(ny/256) nz (two widths, one plane), the count equal
# to it, and one block
@pytest.mark.parametrize("nx,ny,nz,walls", [(133, 154, 3, 0), (33, 256, 2, 1), (12, 250, 1, 0),
                                            (129, 255, 9, 0), (128, 256, 2, 0), (5, 3, 1, 0)])
def test_diagnostics_stay_in_the_workspace(nx, ny, nz, walls):
    import torch
    say(f"[state] diagnostics {nx}x{ny}x{nz}")
    phi, u, p = _fields(nx, ny, nz, 1)
    prm = lbm.make_params(nx, ny, nz, precision="fp64", wall=(0, walls, 0), rho2=0.5)
    n = lbm.lbm_workspace_bytes(prm)
    buf = torch.full((n + (1 << 21),), 0xA5, dtype=torch.uint8, device="cuda")
    dev = lambda a: torch.as_tensor(a).cuda()
    ctx = lbm.lbm_init(prm, buf[:n], torch.cuda.current_stream().cuda_stream, dev(phi), dev(u), dev(p))
    ref = torch.as_tensor(0.9 * phi).cuda()
    d = lbm.lbm_diagnostics(ctx, ref)
    out = [torch.empty(phi.shape, dtype=torch.float64, device="cuda"),
           torch.empty(u.shape, dtype=torch.float64, device="cuda")]
    lbm.lbm_fields(ctx, out[0], out[1], None, 0)
    torch.cuda.synchronize()
    lbm.lbm_destroy(ctx)
    assert bool((buf[n:] == 0xA5).all())
    f, v = (a.cpu().numpy() for a in out)
    rho = 0.5 + 0.5 * f
    z, y, x = np.meshgrid(*(np.arange(k) for k in f.shape), indexing="ij")
    want = dict(sum_phi=f, mass=rho * f, ekin=0.5 * rho * (v * v).sum(0), l2_num=(f - 0.9 * phi) ** 2,
                l2_den=(0.9 * phi) ** 2)
    want = {k: (d[k], a) for k, a in want.items()}
    for a, c in enumerate((x, y, z)):
        want[f"mom{a}"] = d["mom"][a], rho * v[a]
        want[f"com{a}"] = d["com"][a], f * c
        want[f"phiu{a}"] = d["phiu"][a], f * v[a]
    for k, (got, terms) in want.items():  # FP64 sums: N roundings of the terms' size
        assert abs(got - terms.sum()) <= (terms.size + 8) * 2.0 ** -52 * np.abs(terms).sum(), k
    assert d["phi_min"] == f.min() and d["phi_max"] == f.max()
    assert abs(d["umax"] - np.sqrt((v * v).sum(0)).max()) <= 1e-15


# FP64 and FP32 storage, whose populations come back from lbm_get_pdfs and
# lbm_set_pdfs unchanged (16-bit storage refits its phi_s to what is loaded)
@pytest.mark.parametrize("precision,lattice,over", [
    ("fp64", 19, {}), ("fp32", 19, dict(wall=(0, 1, 0), wetting=1, cos_theta=0.5)), ("fp32", 19, {}),
    ("fp64", 19, dict(wall=(1, 1, 1))), ("fp32", 27, dict(wall=(0, 0, 1), wetting=1, cos_theta=-0.3)),
    ("fp64", 27, {}), ("fp32", 19, dict(normal_fd=1)), ("fp32", 27, dict(courant=1.0))])
def test_first_collision_equals_a_step_of_the_stored_state(precision, lattice, over):
    """lbm_init collides the populations it has just rounded; a state loaded
    from those populations (lbm_set_pdfs: a pass that stores, then one that
    reads back and collides) goes on with the same bits."""
    say(f"[state] first collision {precision} Q{lattice} {over}")
    w = inputs.static_droplet(n=20, ny=13, nz=9, R=4.0)
    rng = np.random.default_rng(3)
    u0 = 0.02 * rng.standard_normal(w.u0.shape)
    prm = dict(w.params(), precision=precision, lattice=lattice, rho2=0.4, G=(0.0, -1e-5, 0.0),
               mass_fix_every=0, **over)
    a, b = (lbm.Solver(prm, w.phi0, u0, 1e-3 * w.phi0) for _ in range(2))
    b.set_pdfs(*a.get_pdfs())
    for s in (a, b):
        s.step(3)
    # walls in y or z: the step runs its wall-free instance inside, the first
    # collision the wall-aware one everywhere, and the compiler contracts the
    # two differently (a few roundings of each population per step)
    split = any(over.get("wall", (0, 0, 0))[1:]) and not over["wall"][0]
    eps = 2.0 ** (-52 if precision == "fp64" else -23)
    for x, y in zip(gpu_fields(a), gpu_fields(b)):
        assert np.isfinite(x).all()
        assert np.abs(x - y).max() <= 32 * eps if split else np.array_equal(x, y)


# one cell; partial tiles of every width (16, 32 and 64 fine nodes) and in
# each axis; more tiles than the scratch has rows for
@pytest.mark.parametrize("cg", [(1, 1, 1), (3, 2, 5), (8, 1, 17), (12, 3, 2), (33, 5, 9), (40, 2, 1),
                                (17, 1, 1)])
def test_level_set_update_tile_edges(sur, cg):
    import torch
    say(f"[state] prolong_update {cg}")
    rng = np.random.default_rng(5)
    nx, ny, nz = (2 * n for n in cg)
    phi = rng.random((nz, ny, nx)) * 1.02 - 0.01
    u = 0.02 * rng.standard_normal((3, nz, ny, nx))
    p = 4e-4 * rng.standard_normal((nz, ny, nx))
    s0 = np.zeros(cg[::-1] + (16,), dtype=np.float32)
    s0[..., :5] = rng.random(s0[..., :5].shape)
    s1 = (s0 + 0.1 * rng.standard_normal(s0.shape)).astype(np.float32)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    f = [dev(a) for a in (phi, u, p)]
    m = sur.sur_prolong_update_scratch_doubles(cg)
    scr = torch.full((m + 64,), 7.0, dtype=torch.float64, device="cuda")
    sums = torch.full((4 + 64,), 7.0, dtype=torch.float64, device="cuda")
    sur.sur_prolong_update(dev(s0.reshape(-1, 16)), dev(s1.reshape(-1, 16)), cg, dev(SCALE), 4.0, *f, scr, sums)
    rphi, ru, rp, rsums = co.prolong_update(s0.astype(np.float64), s1.astype(np.float64),
                                            SCALE.astype(np.float64), 4.0, phi, u, p)
    # the coarse psi is FP32: a cell clamped at 1 - 1e-4, which FP32 holds as
    # 1 - 1.000166e-4, has a psi W/4 1.66e-4 off, and the FP32 difference of
    # two |psi| <= 10 rounds to 2^-20; phi moves by at most 1/W per unit of psi
    assert np.abs(f[0].cpu().numpy() - rphi).max() <= 1.66e-4 / 4 + 4 * 2.0 ** -20
    assert np.abs(f[1].cpu().numpy() - ru).max() <= 1e-6 * 0.02
    assert np.abs(f[2].cpu().numpy() - rp).max() <= 1e-6 * 4e-4
    g = sums.cpu().numpy()
    assert np.abs(g[:2] - rsums[:2]).max() <= 1e-12 * phi.size
    assert np.abs(g[2:4] - rsums[2:]).max() <= 1e-5 * phi.size
    assert (g[4:] == 7.0).all() and bool((scr[m:] == 7.0).all())


def test_coarsen_row_stores_equal_the_general_kernel(sur):
    import torch
    say("[state] coarsen, aligned and 4-byte aligned fields")
    g = torch.Generator(device="cuda").manual_seed(2)
    grid = (18, 10, 6)
    N = grid[0] * grid[1] * grid[2]
    a = [torch.randn(n, generator=g, device="cuda") for n in (N, 3 * N, N)]
    off = [torch.cat([x[:1], x])[1:] for x in a]
    scale = torch.as_tensor(SCALE).cuda()
    got = []
    for phi, u, p in (a, off):
        f = torch.full((N // 8, 16), 7.0, device="cuda")
        b = torch.full((N // 8, 16), 7, dtype=torch.int16, device="cuda")
        sur.sur_coarsen(phi, u, p, grid, scale, f, b)
        got.append((f, b))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("prec,dtype,walls", [("fp64", 0, 0), ("fp16", 0, 1), ("bf16", 1, 0), ("fp32", 1, 1)])
def test_fields_stored_twice(prec, dtype, walls):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    say(f"[state] fields stored twice {prec} dtype {dtype}")
    phi, u, p = _fields(37, 21, 6, 2)
    s = lbm.Solver(dict(nx=37, ny=21, nz=6, precision=prec, wall=(0, walls, 0), rho2=0.5), phi, u, p)
    s.step(3)
    new = lambda: [torch.full(a.shape, -7.0, dtype=(torch.float64, torch.float32)[dtype], device="cuda")
                   for a in (phi, u, p)]
    want, a, b, c = new(), new(), new(), new()
    lbm.lbm_fields(s.ctx, *want, dtype)
    lbm.lbm_fields_twice(s.ctx, a, b, dtype)
    lbm.lbm_fields_twice(s.ctx, c, (None, c[1].clone(), None), dtype)
    with pytest.raises(lbm.LbmError):
        lbm.lbm_fields_twice(s.ctx, (a[0], None, a[2]), b, dtype)
    torch.cuda.synchronize()
    for w, x, y, z in zip(want, a, b, c):
        assert torch.equal(w, x) and torch.equal(w, y) and torch.equal(w, z)


# the same with every bit, also where a wall-free interior and wall slabs run
# instances of their own (walls in y with 40 rows, in z, in both)
@pytest.mark.parametrize("precision,lattice", [("fp64", 19), ("fp32", 19), ("fp32", 27), ("fp64", 27)])
@pytest.mark.parametrize("shape,wall,over", [((20, 40, 9), (0, 1, 0), {}), ((20, 13, 9), (0, 0, 1), {}),
                                             ((70, 30, 12), (0, 1, 1), dict(wetting=1, cos_theta=0.5)),
                                             ((20, 13, 9), (0, 1, 0), dict(wetting=1, cos_theta=-0.3)),
                                             ((33, 9, 5), (1, 1, 1), {})])
def test_first_collision_equals_a_step_bit_for_bit(precision, lattice, shape, wall, over):
    say(f"[state] first collision {precision} Q{lattice} {shape} walls {wall} {over}")
    nx, ny, nz = shape
    w = inputs.static_droplet(n=nx, ny=ny, nz=nz, R=3.0)
    u0 = 0.02 * np.random.default_rng(3).standard_normal(w.u0.shape)
    prm = dict(w.params(), precision=precision, lattice=lattice, rho2=0.4, G=(0.0, -1e-5, 0.0), wall=wall,
               mass_fix_every=0, **over)
    a, b = (lbm.Solver(prm, w.phi0, u0, 1e-3 * w.phi0) for _ in range(2))
    b.set_pdfs(*a.get_pdfs())
    for s in (a, b):
        s.step(3)
    for x, y in zip(gpu_fields(a), gpu_fields(b)):
        assert np.isfinite(x).all() and np.array_equal(x, y)


# tiles eight nodes wide: remainders in each axis, more tiles than scratch rows
@pytest.mark.parametrize("cg", [(2, 3, 40), (4, 5, 33), (1, 64, 64), (3, 1, 1), (1, 70, 1), (5, 2, 3)])
def test_level_set_update_narrow_tiles(sur, cg):
    test_level_set_update_tile_edges(sur, cg)
