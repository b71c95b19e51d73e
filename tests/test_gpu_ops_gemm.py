"""The FP32 products on split bf16 operands: independence of the tile size, and infinities."""
import numpy as np
import pytest

import drsynth
from tests.gpu_util import MID

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _clips(n, H, W, seed=0):
    f, m = drsynth.make_clip_batch(range(seed, seed + n), 5, H, W)
    return torch.from_numpy(f).cuda(), torch.from_numpy(m).cuda()


@pytest.mark.parametrize("queries", ["masked", "all"])
def test_small_and_large_tiles_agree_bitwise(queries):
    """Three clips of 5 x 240 x 432 take the 128 x 128 tiles, one of them the 64 x 64 tiles
    (ragged last tiles in both): every output's k order is the same, so the bits are too."""
    from paper_2509_10466_amd import Inpainter
    eng = Inpainter(MID, drsynth.make_weights(MID, 3))
    f, m = _clips(3, 240, 432)
    whole = eng(f, m, "fp32", queries)
    for b in range(3):
        one = eng(f[b:b + 1].contiguous(), m[b:b + 1].contiguous(), "fp32", queries)
        assert torch.equal(one[0], whole[b])


def test_infinite_output_gradient_gives_infinite_weight_gradient():
    """dL/dpred = inf at one pixel value: each decoder weight of that pixel and channel gets
    z * inf = +-inf (no NaN from the split's remainders), every other one stays finite."""
    from paper_2509_10466_amd import Inpainter
    from paper_2509_10466_amd.api import unflatten_params
    eng = Inpainter(MID, drsynth.make_weights(MID, 0))
    f, m = _clips(1, 40, 72)
    pred, saved = eng.train_forward(f, m)
    dpred = torch.zeros_like(pred)
    dpred[0, 2, 9, 6, 1] = float("inf")  # pixel row 9 = 4*2 + 1, column 6 = 4*1 + 2, channel 1
    g = unflatten_params(MID, eng.train_backward(saved, dpred).cpu())["dec.w"]
    saved.close()
    hit = np.zeros(tuple(g.shape), bool)
    hit[:, 1, 1, 2] = True
    assert np.isinf(g.numpy()[hit]).all()
    assert np.isfinite(g.numpy()[~hit]).all()
