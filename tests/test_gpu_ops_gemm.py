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


@pytest.mark.parametrize("precision,clips", [("fp32", 5), ("bf16", 9)])
def test_weight_gradients_of_a_batch_are_the_sum_over_its_clips(precision, clips):
    """The batch's weight gradients take the 128 x 128 tiles (a last chunk and a last step with
    few rows), one clip's the 64 x 64 tiles; only the order of the FP32 sums differs: chunks of
    up to 2048 terms, so 2e-5 of a tensor's largest entry leaves a factor of ten."""
    from paper_2509_10466_amd import Inpainter
    from paper_2509_10466_amd.api import unflatten_params
    eng = Inpainter(MID, drsynth.make_weights(MID, 1))
    eng.train_precision(precision)
    f, m = _clips(clips, 240, 432)
    gen = torch.Generator(device="cuda").manual_seed(0)
    dpred = torch.randn(f.shape, generator=gen, device="cuda")

    def grads(part):
        pred, saved = eng.train_forward(f[part].contiguous(), m[part].contiguous())
        g = eng.train_backward(saved, dpred[part].contiguous()).double().cpu()
        saved.close()
        return g

    whole = unflatten_params(MID, grads(slice(None)))
    summed = unflatten_params(MID, sum(grads(slice(b, b + 1)) for b in range(clips)))
    top = max(float(v.abs().max()) for v in summed.values())
    for name, want in summed.items():
        err = float((whole[name] - want).abs().max())
        assert err <= 2e-5 * float(want.abs().max()) + 1e-7 * top, (name, err)
