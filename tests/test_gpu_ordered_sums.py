"""sur_conv3d_wgrad_ordered promises one order of sums over versions of the
library: the bits of its results on fixed inputs. The digests were taken with
the library as it was before sur_conv3d_wgrad had a second, faster order (one
entry point, the per-tap product off the 16 x 4 x 4 tile, one input chunk per
block on it)."""
import hashlib

import numpy as np
import pytest

from gpu_common import say

pytestmark = pytest.mark.gpu

# one chunk of 8192 points and several, a last chunk of a few points, fewer
# points than a 16-point step, one and two groups of 64 input channels; then
# whole tiles: one, fewer and more than the persistent blocks, every number of
# output tiles, sizes that the fast form groups
DIGESTS = {
    ((4, 4, 4), 64, 64): "3f7a4ba3f09b246e",
    ((3, 1, 5), 16, 32): "8a77d30dc26ef434",
    ((17, 5, 9), 48, 64): "d3ead32fbb1d4cd4",
    ((12, 10, 14), 112, 48): "9512b01182b280ba",
    ((24, 18, 20), 144, 16): "6562bf1541e37578",
    ((40, 24, 56), 80, 32): "271128496d9d6f2d",
    ((50, 46, 62), 16, 16): "17cce3118673c497",
    ((16, 4, 4), 16, 16): "bd13a883ade1279e",
    ((48, 20, 12), 80, 48): "09e01e157a65f0d8",
    ((32, 32, 32), 112, 48): "5bc7ca95b7f0b719",
    ((16, 16, 16), 48, 64): "57a6cc29087c02bd",
    ((64, 64, 64), 80, 32): "46927439439cf45d",
    ((96, 80, 100), 48, 16): "a1686a1c77017413",
    ((96, 96, 96), 32, 32): "a808cae15cf7056c",
    ((128, 64, 64), 16, 16): "af292a963f1ba176",
}


def inputs(grid, ci, co):
    """BF16 bits from a generator whose stream is frozen."""
    rng = np.random.RandomState(ci * 1000 + co)
    n = grid[0] * grid[1] * grid[2]
    bits = lambda c: (rng.standard_normal((n, c)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16).view(np.int16)
    return bits(ci), bits(co)


@pytest.mark.parametrize("grid,ci,co", list(DIGESTS))
def test_ordered_weight_gradient_keeps_its_bits(grid, ci, co):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_12263_amd import surrogate as sur
    say(f"[ordered] {grid} {ci}->{co}")
    x, dy = (torch.as_tensor(a).cuda() for a in inputs(grid, ci, co))
    scr = torch.full((sur.sur_wgrad_scratch_floats(ci, co, grid),), float("nan"), device="cuda")
    dw, db = torch.zeros((27, co, ci), device="cuda"), torch.zeros(co, device="cuda")
    sur.sur_conv3d_wgrad_ordered(x, ci, dy, co, grid, scr, dw, db)
    got = hashlib.sha256(dw.cpu().numpy().tobytes() + db.cpu().numpy().tobytes()).hexdigest()[:16]
    assert got == DIGESTS[grid, ci, co]
