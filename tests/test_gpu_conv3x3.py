"""The 3x3 stride-1 convolution kernel where it can go wrong, against the
oracle's fp64 convolution: images smaller than the kernel, image widths at the
bounds of its patch sizes (31, 63) and one past them (64: the implicit GEMM),
tiles that cross rows and images, channels that leave half a 32-channel block
empty, outputs at the edges of each tile width, every tile shape in both patch
sizes with ragged rows and columns; inactive channels poisoned and columns past
n untouched."""
import os
import re

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from test_gpu_ops import _conv_case, _gpu  # noqa: E402,F401
from gpu_util import rel_err  # noqa: E402

# batch, H, W, cs, ca, n, ldy
CASES = [(1, 1, 1, 16, 16, 72, 72), (2, 1, 2, 8, 8, 8, 16), (3, 2, 1, 40, 40, 64, 64),
         (3, 14, 14, 128, 88, 88, 88), (1, 31, 31, 48, 40, 104, 112), (1, 7, 32, 40, 32, 64, 64),
         (1, 5, 63, 72, 64, 136, 136), (2, 6, 64, 24, 24, 48, 48), (5, 7, 7, 264, 248, 200, 200),
         (1, 40, 2, 16, 8, 24, 24), (40, 28, 28, 64, 48, 96, 96), (90, 28, 28, 32, 16, 72, 72),
         (24, 56, 56, 32, 24, 64, 64), (24, 56, 56, 16, 16, 96, 96)]
# Three channel blocks (the last with 8 channels), rows and columns that fill no
# whole number of tiles, for each tile shape the kernel's rule can choose.
TILE_CASES = [(42, 28, 28, 80, 72, 136, 136), (41, 20, 40, 80, 72, 136, 136),   # 256x64
              (47, 15, 31, 80, 72, 136, 144),                                   # 256x96
              (21, 28, 28, 80, 72, 136, 136), (21, 20, 40, 80, 72, 136, 136),   # 128x64
              (52, 14, 15, 80, 72, 136, 136), (10, 33, 33, 80, 72, 136, 144),   # 128x96
              (1, 7, 15, 80, 72, 72, 72), (1, 16, 33, 80, 72, 72, 72)]          # 64x64


def _tile(M, W, ca, n):
    """The tile that launch_conv3x3 takes, by the table and rule in its source."""
    import paper_2609_10018_amd as pkg
    with open(os.path.join(os.path.dirname(pkg.__file__), "csrc", "conv3x3.hip")) as fh:
        table = re.search(r"kTiles\[\] = \{(.*?)\};", fh.read(), re.S).group(1)
    tiles = [tuple(float(v) for v in t.split(",")) for t in re.findall(r"\{([^{}]*)\}", table)]
    assert len(tiles) == 5
    best = None
    for i, (bm, bn, alone, shared, edge) in enumerate(tiles):
        if W > 31 and i == 1:
            continue
        each = -(-(-(-M // bm) * -(-n // bn)) // 256)
        t = 3 * -(-ca // 32) * (alone if each < 2 else each * shared) + each * edge
        if best is None or t < best[0]:
            best = (t, (int(bm), int(bn)))
    return best[1]


def test_the_tile_cases_reach_every_tile():
    reached = set()
    for batch, H, W, _, ca, n, _ in TILE_CASES:
        bm, bn = _tile(batch * H * W, W, ca, n)
        assert batch * H * W % bm and n % bn
        reached.add((bm, bn, W > 31))
    both = {(256, 64), (128, 64), (128, 96), (64, 64)}
    assert reached == {(m, n, w) for m, n in both for w in (False, True)} | {(256, 96, False)}


@pytest.mark.parametrize("batch,H,W,cs,ca,n,ldy", CASES + TILE_CASES)
def test_conv3x3(batch, H, W, cs, ca, n, ldy):
    got, ref, after, before = _conv_case(batch, H, W, cs, ca, 3, 3, 1, 1, cs, n, ldy, True,
                                         poison=True)
    # One rounding to bf16, half a unit of 8 significant bits: up to 2^-8 = 3.9e-3
    # of the largest value (reached at the low end of a binade); the fp32 sums of at
    # most 2232 products add up to 1e-4.
    assert rel_err(got, ref) < 4e-3
    np.testing.assert_array_equal(after, before)


def test_conv3x3_bits_do_not_depend_on_the_batch():
    """An image alone takes 64x64 tiles, the same image in a batch larger ones."""
    from gpu_util import dev
    from paper_2609_10018_amd import ffi
    rng = np.random.default_rng(3)
    hw, c, n, batch = 28, 88, 88, 70
    x = dev(rng.standard_normal((batch, hw, hw, c)), torch.bfloat16)
    w = dev(rng.standard_normal((n, 9 * c)) * 0.05, torch.bfloat16)
    b = dev(rng.standard_normal(n), torch.float32)

    def run(xs):
        y = torch.empty((xs.shape[0], hw, hw, n), dtype=torch.bfloat16, device="cuda")
        ffi.op_conv2d(xs, xs.shape[0], hw, hw, c, c, 3, 3, 1, 1, w, 9 * c, c, b, y, n, n, False)
        return y

    whole = run(x)
    for i in (0, 33, batch - 1):
        assert torch.equal(run(x[i:i + 1].clone())[0], whole[i])
