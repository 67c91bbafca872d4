"""Launch shapes of the step: whole-row tiles, blocks of one wavefront, and the
interior and its wall slabs in one launch, against the FP64 oracle on sizes
at the edges of their rules."""
import numpy as np
import pytest

from gpu_common import gpu_fields, gpu_solver, oracle_run, say
from paper_2407_12263_amd import inputs

pytestmark = pytest.mark.gpu


def _workload(nx, ny, nz, wall):
    w = inputs.static_droplet(n=nx, ny=ny, nz=nz, R=max(2.0, min(nx, ny) / 4.0))
    rng = np.random.default_rng(7)
    u0 = 0.01 * rng.standard_normal(w.u0.shape)
    return w.with_(wall=wall, u0=u0, rho2=0.5, G=(0.0, -1e-5, 0.0))


# 32,768 nodes and one plane more (one-wavefront blocks or not); rows of 65 to
# 255 nodes, one and several per tile; rows beyond a block; slabs that meet
# (no interior), leave one row, and end in a partial tile; walls in z, in both,
# and on every face; more than one launch's nodes
@pytest.mark.parametrize("nx,ny,nz,wall", [
    (32, 32, 32, (0, 0, 0)), (32, 32, 33, (0, 0, 0)), (65, 7, 5, (0, 1, 0)), (75, 31, 6, (0, 1, 0)),
    (85, 13, 40, (0, 1, 1)), (129, 9, 4, (0, 1, 0)), (255, 5, 30, (0, 1, 1)), (257, 6, 3, (0, 1, 0)),
    (300, 11, 4, (0, 0, 1)), (12, 33, 5, (0, 1, 0)), (3, 200, 4, (0, 1, 0)), (20, 40, 3, (0, 0, 1)),
    (20, 40, 2, (0, 1, 1)), (33, 20, 9, (1, 1, 1))])
def test_step_matches_the_oracle(nx, ny, nz, wall):
    say(f"[shapes] {nx}x{ny}x{nz} walls {wall}")
    w = _workload(nx, ny, nz, wall)
    o = oracle_run(w, 3)
    sol = gpu_solver(w, "fp64")
    sol.step(3)
    # three steps of an FP64 update: the one-step bound of 1e-14 on each field,
    # three times, and once more for the fields' own sums
    for g, r in zip(gpu_fields(sol), o.fields()):
        assert np.abs(g - np.asarray(r)).max() <= 4e-14


@pytest.mark.parametrize("precision,lattice", [("fp16", 19), ("bf16", 27), ("fp32", 19), ("fp64", 27)])
def test_one_launch_and_split_launches_agree(precision, lattice):
    """A lattice above the one-launch limit (its slabs in launches of their own)
    repeats a smaller one's solution when both are uniform along x."""
    say(f"[shapes] one launch / split launches {precision} Q{lattice}")
    ny, nz = 24, 16
    big = {19: 3328, 27: 1536}[lattice]  # nodes: 1,277,952 and 589,824
    assert big * ny * nz > (1250000 if lattice == 19 else 500000)
    out = []
    for nx in (64, big):
        y = np.arange(ny)[None, :, None] + np.zeros((nz, ny, nx))
        phi0 = 0.5 + 0.5 * np.tanh(0.5 * (y - ny / 2))
        u0 = np.zeros((3, nz, ny, nx))
        u0[2] = 0.01 * np.sin(2 * np.pi * y / ny)
        w = inputs.static_droplet(n=nx, ny=ny, nz=nz, R=4.0).with_(phi0=phi0, u0=u0, wall=(0, 1, 1), rho2=0.5,
                                                                  G=(0.0, -1e-5, 0.0))
        sol = gpu_solver(w, precision, lattice=lattice, mass_fix_every=0)
        sol.step(4)
        out.append([a[..., :64].copy() for a in gpu_fields(sol)])
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)


# widths whose tiles outnumber the rows of the phase-mass partials (256 wide on
# three nodes: 256 tiles a plane against 3 rows; walls add slabs), and widths
# that are taken: the sums stay inside the workspace, the states are the same
@pytest.mark.parametrize("nx,ny,nz,wall,width", [(3, 256, 2, 0, 8), (3, 256, 2, 1, 7), (1, 250, 3, 0, 8),
                                                 (2, 300, 1, 0, 6), (40, 64, 3, 1, 8), (40, 64, 3, 0, 3)])
@pytest.mark.parametrize("precision", ["fp16", "fp64"])
def test_tile_override_stays_in_the_workspace(nx, ny, nz, wall, width, precision, monkeypatch):
    import torch
    from paper_2407_12263_amd import lbm
    say(f"[shapes] {nx}x{ny}x{nz} {precision} tile width 2^{width}")
    w = _workload(nx, ny, nz, (0, wall, 0))
    prm = lbm.make_params(**dict(w.params(), precision=precision, mass_fix_every=1))
    n = lbm.lbm_workspace_bytes(prm)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64).cuda()
    out = []
    for over in (None, str(width)):
        if over:
            monkeypatch.setenv("LBM_TILE_X_LOG2", over)
        buf = torch.full((n + (1 << 21),), 0xA5, dtype=torch.uint8, device="cuda")
        ctx = lbm.lbm_init(prm, buf[:n], torch.cuda.current_stream().cuda_stream, dev(w.phi0), dev(w.u0), dev(w.p0))
        lbm.lbm_step(ctx, 3)
        d = lbm.lbm_diagnostics(ctx)
        phi = torch.empty((nz, ny, nx), dtype=torch.float64, device="cuda")
        lbm.lbm_fields(ctx, phi, None, None, 0)
        torch.cuda.synchronize()
        lbm.lbm_destroy(ctx)
        assert bool((buf[n:] == 0xA5).all())
        out.append((d["sum_phi"], phi))
    # the phase mass is summed in the tiles' groups: the correction may differ
    # in the last bits of an FP64 sum, and a state by its storage's rounding
    eps = 2.0 ** (-11 if precision == "fp16" else -52)
    assert abs(out[0][0] - out[1][0]) <= phi.numel() * eps
    assert float((out[0][1] - out[1][1]).abs().max()) <= 64 * eps


# whole-row tiles where they are fewer rounds of the CUs and not where they are
# as many; bands of 64 rows of nodes with and without a remainder; rows of 224
# and 225 nodes
@pytest.mark.parametrize("nx,ny,nz,wall", [(50, 50, 50, (0, 0, 0)), (20, 70, 50, (0, 0, 0)), (80, 200, 24, (0, 0, 0)),
                                           (20, 170, 90, (0, 1, 0)), (40, 100, 60, (0, 0, 1)), (224, 9, 30, (0, 1, 0)),
                                           (225, 9, 30, (0, 0, 0)), (80, 80, 12, (1, 1, 1))])
def test_row_tiles_and_bands_match_the_oracle(nx, ny, nz, wall):
    test_step_matches_the_oracle(nx, ny, nz, wall)
