"""Convolutions and weight gradients on grids that the 16 x 4 x 4 point tile
does not divide. The LDS-staged kernel must give the general kernel's bits:
the same operands padded to 144 input channels with zeros (which add exactly
nothing to any sum) take the general kernel. The weight gradient's partial
tiles are compared with the oracle."""
import numpy as np
import pytest

from oracle import surrogate_oracle as so

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sur():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_12263_amd import surrogate
    surrogate.load_library()
    return surrogate


def _bf16(shape, seed, scale=1.0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (scale * torch.randn(shape, generator=g, device="cuda")).to(torch.bfloat16).view(torch.int16)


# one point; single tiles of every width (4, 8, 16); remainders in each axis;
# two and three output tiles per block (enough blocks) and one; every input
# slice count; grids of many blocks (three taps a weight stage: 48 channels)
SHAPES = [((1, 1, 1), 16, 16), ((3, 1, 5), 32, 32), ((8, 8, 8), 64, 64), ((17, 5, 9), 112, 48),
          ((15, 4, 4), 96, 16), ((16, 4, 7), 128, 32), ((33, 3, 2), 80, 112), ((40, 24, 56), 80, 32),
          ((50, 46, 62), 48, 16), ((66, 62, 58), 16, 48), ((60, 50, 44), 32, 16)]


@pytest.mark.parametrize("flip", [0, 1])
@pytest.mark.parametrize("grid,cin,cout", SHAPES)
def test_ragged_conv_bits_of_the_general_kernel(sur, grid, cin, cout, flip):
    import torch
    say(f"[ragged] conv {grid} {cin}->{cout} flip={flip}")
    P = grid[0] * grid[1] * grid[2]
    x, w = _bf16((P, cin), 1), _bf16((27, cout, cin), 2, 0.1)
    mask = _bf16((P, cout), 3) if flip else None
    bias = None if flip else _bf16(cout, 4).view(torch.bfloat16).float()
    pad = lambda a: torch.nn.functional.pad(a, (0, 144 - cin)).contiguous()
    out = []
    for xi, wi, ci in ((x, w, cin), (pad(x), pad(w), 144)):
        yb = torch.zeros((P, cout), dtype=torch.int16, device="cuda")
        yf = torch.zeros((P, cout), dtype=torch.float32, device="cuda")
        sur.sur_conv3d(xi, ci, wi, bias, cout, grid, flip=flip, relu=1 - flip, mask=mask, y_bf16=yb,
                       y_f32=yf)
        out.append((yb, yf.view(torch.int32)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert int((out[0][1] != 0).sum()) > 0


def test_ragged_conv_unaligned_operands(sur):
    """Operands off the 8- and 16-byte boundaries: accepted, the same bits."""
    import torch
    say("[ragged] conv, mask and outputs off their alignment")
    grid, cin, cout = (6, 5, 7), 32, 16
    P = grid[0] * grid[1] * grid[2]
    x, w, m = _bf16((P, cin), 1), _bf16((27, cout, cin), 2, 0.1), _bf16((P, cout), 3)
    ref = torch.zeros((P, cout), dtype=torch.int16, device="cuda")
    sur.sur_conv3d(x, cin, w, None, cout, grid, mask=m, y_bf16=ref)
    off = lambda a: torch.cat([a.new_zeros(1), a.reshape(-1)])[1:].view(a.shape)
    for xi, wi, mi, yi in ((off(x), w, m, ref), (x, off(w), m, ref), (x, w, off(m), ref), (x, w, m, off(ref))):
        y = torch.zeros_like(ref) if yi is ref else off(torch.zeros_like(ref))
        sur.sur_conv3d(xi, cin, wi, None, cout, grid, mask=mi, y_bf16=y)
        assert torch.equal(y, ref)


# 255 and 256 points (the per-tap product and the tiled kernel), the smallest
# and largest flushed grids below 4096 points, plain partial tiles, and a
# grid of more than eight tiles per block (flushed)
@pytest.mark.parametrize("grid,cin,cout", [((17, 5, 3), 16, 16), ((4, 8, 8), 64, 64), ((8, 8, 8), 48, 64),
                                           ((13, 17, 18), 112, 48), ((30, 11, 14), 80, 32),
                                           ((20, 12, 28), 32, 48), ((72, 60, 74), 48, 16)])
def test_ragged_weight_gradient(sur, grid, cin, cout):
    import torch
    say(f"[ragged] wgrad {grid} {cin}->{cout}")
    nx, ny, nz = grid
    P = nx * ny * nz
    x, dy = _bf16((P, cin), 5), _bf16((P, cout), 6)
    scratch = torch.empty(sur.sur_wgrad_scratch_floats(cin, cout, grid), dtype=torch.float32, device="cuda")
    dw = torch.empty((27, cout, cin), dtype=torch.float32, device="cuda")
    db = torch.empty(cout, dtype=torch.float32, device="cuda")
    sur.sur_conv3d_wgrad(x, cin, dy, cout, grid, scratch, dw, db)
    f = lambda a, c: a.view(torch.bfloat16).double().cpu().numpy().reshape(nz, ny, nx, c)
    rdw, rdb = so.conv3d_wgrad(f(x, cin), f(dy, cout))
    # FP32 sums of exact products in chains of at most 256 additions (a block's
    # tiles, then the blocks' partials): 256 roundings of 2^-24 of the sum of
    # the terms' sizes, E|x dy| = 2 / pi each
    bound = 256 * 2.0 ** -24 * P * 2.0 / np.pi
    assert np.abs(dw.cpu().numpy() - rdw).max() <= bound
    assert np.abs(db.cpu().numpy() - rdb).max() <= 256 * 2.0 ** -24 * P * np.sqrt(2.0 / np.pi)


# three output tiles of 96 input channels: the weight stage that takes most
# registers (seven pieces a thread), over one and two columns of blocks, beside
# the neighbouring channel counts on the same grid
@pytest.mark.parametrize("flip", [0, 1])
@pytest.mark.parametrize("grid,cin,cout", [((40, 64, 44), 96, 48), ((40, 40, 40), 96, 96), ((56, 56, 56), 96, 48),
                                           ((40, 64, 44), 80, 48), ((40, 64, 44), 112, 48),
                                           ((40, 64, 44), 128, 32)])
def test_ragged_conv_widest_weight_stages(sur, grid, cin, cout, flip):
    test_ragged_conv_bits_of_the_general_kernel(sur, grid, cin, cout, flip)


# an end in x only, in each axis, in all; plain and flushed forms; one and
# three output tiles
@pytest.mark.parametrize("grid,cin,cout", [((20, 12, 28), 16, 16), ((16, 18, 24), 32, 48), ((32, 12, 18), 16, 16),
                                           ((13, 17, 18), 48, 32), ((72, 60, 74), 48, 16)])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_ragged_weight_gradient_of_infinite_inputs(sur, grid, cin, cout, axis):
    """An infinite input at the last and the first point of an axis meets output
    gradients that are never zero: each dW of its channel is infinite, as the
    sum over the grid's points has it, and no other is touched."""
    import torch
    say(f"[ragged] wgrad {grid} {cin}->{cout}, infinite inputs at the ends of axis {axis}")
    P = grid[0] * grid[1] * grid[2]
    scratch = torch.empty(sur.sur_wgrad_scratch_floats(cin, cout, grid), dtype=torch.float32, device="cuda")
    for at in (0, grid[axis] - 1):
        x, dy = _bf16((P, cin), 5), _bf16((P, cout), 6)
        assert int((dy == 0).sum()) == 0
        where = [grid[0] // 2, grid[1] // 2, grid[2] // 2]
        where[axis] = at
        p = where[0] + grid[0] * (where[1] + grid[1] * where[2])
        x.view(torch.bfloat16)[p, 3] = float("inf")
        dw = torch.empty((27, cout, cin), dtype=torch.float32, device="cuda")
        sur.sur_conv3d_wgrad(x, cin, dy, cout, grid, scratch, dw, torch.empty(cout, device="cuda"))
        z, y, xx = np.meshgrid(*[np.arange(3) - 1] * 3, indexing="ij")
        # tap d takes the input at p from the output gradient at p - d
        src = [torch.as_tensor((w - d.ravel()) % n).cuda() for w, d, n in zip(where, (xx, y, z), grid)]
        sign = torch.sign(dy.view(torch.bfloat16)[src[0] + grid[0] * (src[1] + grid[1] * src[2])].float())
        assert bool(torch.isinf(dw[:, :, 3]).all()) and torch.equal(torch.sign(dw[:, :, 3]), sign)
        keep = [c for c in range(cin) if c != 3]
        assert bool(torch.isfinite(dw[:, :, keep]).all())


# the ends of the rule that gives ragged grids their tiles: fewest points with
# rows of one tile and of two, fivefold and fourfold cover, one step below each;
# thin grids; the flushed forms in two parts and in one, and the plain one
@pytest.mark.parametrize("grid,cin,cout", [((8, 8, 8), 16, 16), ((16, 9, 4), 48, 64), ((8, 9, 7), 48, 32),
                                           ((17, 4, 8), 48, 64), ((18, 9, 4), 48, 16), ((40, 4, 4), 16, 32),
                                           ((17, 5, 9), 96, 48), ((33, 5, 5), 48, 64), ((2, 2, 128), 16, 16),
                                           ((1000, 1, 1), 16, 16), ((24, 1, 24), 48, 16), ((50, 50, 1), 48, 16),
                                           ((100, 100, 1), 48, 16), ((15, 17, 16), 64, 64), ((15, 17, 17), 64, 64),
                                           ((19, 5, 8), 48, 64), ((48, 16, 1), 48, 64), ((18, 9, 5), 48, 16)])
def test_ragged_weight_gradient_is_as_exact_as_the_ordered(sur, grid, cin, cout):
    """No further from FP64 sums than the order that the per-tap product has:
    both errors are means over 432 to 82944 weights of independent roundings,
    of which three draws leave less than 2%."""
    import torch
    say(f"[ragged] wgrad {grid} {cin}->{cout}, error against the ordered form")
    P = grid[0] * grid[1] * grid[2]
    scratch = torch.empty(sur.sur_wgrad_scratch_floats(cin, cout, grid), dtype=torch.float32, device="cuda")
    err = [0.0, 0.0]
    for seed in range(3):
        x, dy = _bf16((P, cin), 10 + seed), _bf16((P, cout), 20 + seed)
        X, D = x.view(torch.bfloat16).double().view(grid[2], grid[1], grid[0], cin), dy.view(torch.bfloat16).double()
        ref = torch.stack([D.t() @ torch.roll(X, (1 - t // 9, 1 - t // 3 % 3, 1 - t % 3), (0, 1, 2)).reshape(-1, cin)
                           for t in range(27)])
        for k, f in enumerate((sur.sur_conv3d_wgrad_ordered, sur.sur_conv3d_wgrad)):
            dw = torch.empty((27, cout, cin), dtype=torch.float32, device="cuda")
            f(x, cin, dy, cout, grid, scratch, dw, torch.empty(cout, device="cuda"))
            err[k] += float((dw - ref).norm() / ref.norm())
    assert err[1] <= 1.02 * err[0]


# tile widths taken for a second block on a CU or to fit three output tiles;
# thin grids on either side of the rule that leaves them to the general kernel
@pytest.mark.parametrize("grid,cin,cout", [((60, 60, 60), 48, 64), ((44, 40, 70), 96, 48), ((52, 60, 38), 112, 48),
                                           ((1, 1, 2000), 48, 64), ((1, 1, 9000), 48, 64), ((200, 150, 1), 32, 48),
                                           ((2, 120, 120), 112, 48), ((300, 160, 1), 16, 16)])
def test_ragged_conv_tile_widths_and_thin_grids(sur, grid, cin, cout):
    test_ragged_conv_bits_of_the_general_kernel(sur, grid, cin, cout, 0)
