"""The decoder's first convolution read and differentiated in place: the weight
gradient of the concat [up2(xc), xf] without writing it, and the data gradient
with the upsampling's adjoint in the same pass. Both make the same products and
sums in the same order as the separate passes, so every bit is compared."""
import pytest

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


# (grid, cup, cskip, channels out): one tile; small-grid blocks of one output
# tile; two-tile blocks of four wavefronts, with one input chunk and with
# several, odd tile counts, a block of both kinds of channels; eight wavefronts
SHAPES = [((16, 4, 4), 16, 16, 16), ((32, 32, 32), 64, 48, 48), ((16, 12, 20), 48, 32, 32),
          ((48, 20, 12), 32, 48, 16), ((80, 60, 28), 48, 32, 32), ((112, 76, 92), 32, 16, 16),
          ((112, 76, 92), 16, 64, 48), ((64, 64, 64), 48, 32, 32), ((128, 64, 64), 48, 16, 16),
          ((128, 128, 128), 32, 16, 16)]


@pytest.mark.parametrize("grid,cup,cskip,co", SHAPES)
def test_decoder_backward_in_place_bits(sur, grid, cup, cskip, co):
    import torch
    say(f"[decoder] {grid} {cup}+{cskip}->{co}")
    P, ci = grid[0] * grid[1] * grid[2], cup + cskip
    half = tuple(n // 2 for n in grid)
    dy, wd = _bf16((P, co), 1), _bf16((27, ci, co), 2, 0.1)
    act = torch.relu(_bf16((P // 8, cup), 3).view(torch.bfloat16)).view(torch.int16)
    dx = torch.empty((P, ci), dtype=torch.float32, device="cuda")
    sur.sur_conv3d(dy, co, wd, None, ci, grid, flip=1, y_f32=dx)
    want = torch.zeros((P // 8, cup), dtype=torch.int16, device="cuda")
    sur.sur_upsample2_bwd_mask(dx, ci, 0, cup, half, act, want)
    got = torch.full_like(want, 7)
    skip = torch.full((P, cskip), 7.0, device="cuda")
    sur.sur_conv3d_dgrad_cat(dy, co, wd, cup, cskip, grid, act, got, skip)
    assert torch.equal(got, want)
    assert torch.equal(skip.view(torch.int32), dx[:, cup:].contiguous().view(torch.int32))

    xc, xf = _bf16((P // 8, cup), 4), _bf16((P, cskip), 5)
    cat = torch.empty((P, ci), dtype=torch.int16, device="cuda")
    sur.sur_concat_up2(xc, cup, xf, cskip, grid, cat)
    scr = torch.empty(sur.sur_wgrad_scratch_floats(ci, co, grid), device="cuda")
    out = []
    for cat_form in (0, 1):
        dw, db = torch.zeros((27, co, ci), device="cuda"), torch.zeros(co, device="cuda")
        if cat_form:
            sur.sur_conv3d_wgrad_cat(xc, cup, xf, cskip, dy, co, grid, scr, dw, db)
        else:
            sur.sur_conv3d_wgrad_ordered(cat, ci, dy, co, grid, scr, dw, db)
        out.append((dw, db))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_decoder_backward_refusals(sur):
    import torch
    say("[decoder] sizes and operands that the in-place forms refuse")
    z = lambda n, dt=torch.int16: torch.zeros(n, dtype=dt, device="cuda")
    P = 16 * 4 * 4
    args = dict(dy=z(P * 16), cin=16, w=z(27 * 32 * 16), cup=16, cskip=16, grid=(16, 4, 4),
                act=z(P // 8 * 16), dup_bf16=z(P // 8 * 16), dskip=z(P * 16, torch.float32))
    for bad in (dict(grid=(8, 4, 8)), dict(cup=8), dict(act=z(P // 8 * 16 + 1)[1:]), dict(dskip=None)):
        with pytest.raises(RuntimeError):
            sur.sur_conv3d_dgrad_cat(**(args | bad))


# weight gradients of grouped input chunks: groups of two and three, a last
# group of one and of two chunks, one and two output tiles, sizes that are powers
# of two and not, a tile count that the blocks do not divide
@pytest.mark.parametrize("grid,ci,co", [((96, 96, 96), 32, 16), ((96, 80, 100), 48, 16), ((96, 96, 96), 64, 16),
                                        ((64, 80, 100), 80, 32), ((96, 96, 96), 32, 32), ((96, 96, 96), 80, 16)])
def test_grouped_weight_gradient(sur, grid, ci, co):
    """Against FP64 products: the sums of P products of unit normals in FP32
    blocks of at most 3 P / 256 tiles err by about sqrt(adds) 2^-25 of a sum;
    2e-6 is above twice the largest error that the sizes allow."""
    import torch
    say(f"[wgrad] {grid} {ci}->{co} grouped chunks")
    P = grid[0] * grid[1] * grid[2]
    dy, x = _bf16((P, co), 1), _bf16((P, ci), 4)
    scr = torch.full((sur.sur_wgrad_scratch_floats(ci, co, grid),), float("nan"), device="cuda")
    dw, db = torch.zeros((27, co, ci), device="cuda"), torch.zeros(co, device="cuda")
    sur.sur_conv3d_wgrad(x, ci, dy, co, grid, scr, dw, db)
    X = x.view(torch.bfloat16).double().view(grid[2], grid[1], grid[0], ci)
    D = dy.view(torch.bfloat16).double()
    for t in range(27):
        ref = D.t() @ torch.roll(X, (1 - t // 9, 1 - t // 3 % 3, 1 - t % 3), (0, 1, 2)).reshape(-1, ci)
        assert float((dw[t] - ref).norm() / ref.norm()) < 2e-6, t
    ref = D.sum(0)
    assert float((db - ref).norm() / ref.norm()) < 2e-6


# three output tiles per block: 3, 5 and 7 tiles (the last block has 3, 2 and
# 1), one input chunk and several, weights resident and staged per item, sizes
# that are powers of two and not
@pytest.mark.parametrize("grid,cin,cout", [((64, 64, 64), 16, 48), ((48, 64, 256), 16, 80),
                                           ((48, 64, 256), 48, 48), ((64, 64, 64), 32, 112),
                                           ((64, 64, 64), 80, 80)])
def test_three_output_tiles_bits_of_two(sur, grid, cin, cout, monkeypatch):
    import torch
    say(f"[conv] {grid} {cin}->{cout} three output tiles per block")
    P = grid[0] * grid[1] * grid[2]
    x, w, m = _bf16((P, cin), 1), _bf16((27, cout, cin), 2, 0.1), _bf16((P, cout), 3)
    b = _bf16(cout, 4).view(torch.bfloat16).float()
    out = []
    for form in "01":
        monkeypatch.setenv("SUR_CONV_NT3", form)
        y = [torch.zeros((P, cout), dtype=torch.int16, device="cuda") for _ in range(2)]
        f = torch.zeros((P, cout), device="cuda")
        sur.sur_conv3d(x, cin, w, b, cout, grid, relu=1, y_bf16=y[0], y_f32=f)
        sur.sur_conv3d(x, cin, w, None, cout, grid, flip=1, mask=m, y_bf16=y[1])
        out.append(y + [f.view(torch.int32)])
    for a, c in zip(*out):
        assert int((a != 0).sum()) > 0 and torch.equal(a, c)


# eight wavefronts for one output tile from half a tile per CU on: the smallest
# such grid, one below it, and sizes that are no powers of two
@pytest.mark.parametrize("grid,cc,fc", [((32, 64, 32), 16, 16), ((32, 32, 56), 16, 16), ((48, 48, 48), 32, 16),
                                        ((64, 48, 48), 48, 32)])
def test_eight_wavefronts_bits_of_four(sur, grid, cc, fc, monkeypatch):
    import torch
    say(f"[conv] {grid} {cc}+{fc}->16 eight wavefronts")
    P, ci = grid[0] * grid[1] * grid[2], cc + fc
    x, xc, w, m = _bf16((P, ci), 1), _bf16((P // 8, cc), 5), _bf16((27, 16, ci), 2, 0.1), _bf16((P, 16), 3)
    xf, b = x[:, cc:].contiguous(), _bf16(16, 4).view(torch.bfloat16).float()
    out = []
    for form in ("4", None):
        if form:
            monkeypatch.setenv("SUR_CONV_WV", form)
        else:
            monkeypatch.delenv("SUR_CONV_WV")
        y = [torch.zeros((P, 16), dtype=torch.int16, device="cuda") for _ in range(4)]
        pool = torch.zeros((P // 8, 16), dtype=torch.int16, device="cuda")
        sur.sur_conv3d(x, ci, w, b, 16, grid, relu=1, y_bf16=y[0])
        sur.sur_conv3d(x, ci, w, None, 16, grid, flip=1, mask=m, y_bf16=y[1])
        sur.sur_conv3d_cat(xc, cc, xf, fc, w, b, 16, grid, relu=1, y_bf16=y[2])
        sur.sur_conv3d_pool(x, ci, w, b, 16, grid, relu=1, y_bf16=y[3], y_pool=pool)
        out.append(y + [pool])
    for a, c in zip(*out):
        assert int((a != 0).sum()) > 0 and torch.equal(a, c)


# the ordered sums: those of the plain form where both take the tiled kernel;
# sizes off the tile and grids where the plain form groups chunks, against FP64
@pytest.mark.parametrize("grid,ci,co,same", [((16, 16, 32), 16, 32, True), ((32, 32, 32), 48, 48, True),
                                             ((12, 10, 14), 48, 64, False), ((40, 24, 56), 80, 32, False),
                                             ((96, 96, 96), 32, 16, False)])
def test_ordered_weight_gradient(sur, grid, ci, co, same):
    import torch
    say(f"[wgrad] {grid} {ci}->{co} ordered")
    P = grid[0] * grid[1] * grid[2]
    dy, x = _bf16((P, co), 1), _bf16((P, ci), 4)
    scr = torch.full((sur.sur_wgrad_scratch_floats(ci, co, grid),), float("nan"), device="cuda")
    out = []
    for f in (sur.sur_conv3d_wgrad, sur.sur_conv3d_wgrad_ordered):
        dw, db = torch.zeros((27, co, ci), device="cuda"), torch.zeros(co, device="cuda")
        f(x, ci, dy, co, grid, scr, dw, db)
        out.append((dw, db))
    for a, b in zip(*out):
        assert torch.equal(a, b) if same else float((a - b).norm() / b.norm()) < 4e-6


# no level fits the in-place decoder; one level (no concat at all); the finest
# fits and the next one does not; both fit
@pytest.mark.parametrize("grid,channels,accepted", [((24, 16, 16), (16, 32, 48), True), ((20, 12, 28), (16, 32), True),
                                                    ((16, 8, 8), (16,), True), ((32, 8, 12), (16, 32, 48), False),
                                                    ((32, 8, 16), (16, 32, 48), False)])
def test_backward_after_an_inference_forward(sur, grid, channels, accepted):
    """A forward pass without keep_cat is enough for the backward pass where
    every concat is written, and refused where one is read in place."""
    import torch
    say(f"[decoder] backward after forward without keep_cat {grid}")
    net = sur.UNet(grid, channels=channels, seed=3)
    x, dout = _bf16((net.P[0], 16), 1), _bf16((net.P[0], 16), 2)
    net.forward(x, keep_cat=True)
    net.backward(dout)
    want = net.flat["g"].clone()
    net.flat["g"].zero_()
    net.forward(x)
    if accepted:
        net.backward(dout)
        assert int((want != 0).sum()) > 0 and torch.equal(net.flat["g"], want)
    else:
        with pytest.raises(RuntimeError):
            net.backward(dout)


# every level in place; the finest in place and the coarser ones written; two
# levels in place with tiles that are no powers of two
@pytest.mark.parametrize("grid,channels", [((64, 32, 32), (16, 32, 48)), ((32, 32, 32), (16, 32, 48, 64)),
                                           ((96, 24, 40), (16, 32, 48))])
def test_unet_in_place_decoder_equals_the_written_concat(sur, grid, channels, monkeypatch):
    """A network whose decoders read and differentiate their concat in place
    against one that writes every concat (and pools apart): the forward pass,
    and the output, gradients and weights of two training steps."""
    import torch
    say(f"[decoder] network {grid}, concats in place and written")
    P = grid[0] * grid[1] * grid[2]
    x, tgt, wch = _bf16((P, 16), 1), _bf16((P, 16), 2).view(torch.bfloat16).float(), torch.ones(5, device="cuda")
    out = []
    for written in (False, True):
        if written:
            monkeypatch.setattr(sur, "conv_cat_fits", lambda g: False)
        net = sur.UNet(grid, channels=channels, seed=4)
        assert ("cat0" in net.act) == written
        got = [net.forward(x).clone()]
        for _ in range(2):
            net.train_step(x, tgt, wch)
            got += [net.out.clone(), net.flat["g"].clone(), net.flat["w"].clone()]
        out.append(got)
    for a, b in zip(*out):
        assert bool(torch.isfinite(a).all()) and int((a != 0).sum()) > 0
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


# either side of the range that keeps four wavefronts: more than 1 3/4 tiles per
# CU, several input chunks with uneven planes, and above 1 1/4 tiles
@pytest.mark.parametrize("grid,cc,fc", [((64, 64, 56), 16, 16), ((80, 48, 40), 32, 16), ((64, 64, 48), 48, 32),
                                        ((48, 64, 48), 16, 16)])
def test_wavefront_rule_bits_of_four(sur, grid, cc, fc, monkeypatch):
    test_eight_wavefronts_bits_of_four(sur, grid, cc, fc, monkeypatch)


# three output tiles per block with whole columns (9 tiles) and a last one of a
# single tile (19), and the counts that keep two (7, 8, 10)
@pytest.mark.parametrize("grid,cin,cout", [((64, 64, 64), 48, 144), ((64, 64, 64), 16, 304), ((64, 64, 64), 48, 128),
                                           ((48, 64, 256), 16, 160)])
def test_three_output_tiles_by_columns(sur, grid, cin, cout, monkeypatch):
    test_three_output_tiles_bits_of_two(sur, grid, cin, cout, monkeypatch)
