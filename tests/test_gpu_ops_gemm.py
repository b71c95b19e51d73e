"""The FP32 products on split bf16 operands: independence of the tile size, and infinities."""
import dataclasses

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


@pytest.mark.parametrize("clips", [1, 3])
def test_infinite_weight_gives_infinite_outputs_of_its_channel_alone(clips):
    """wk[7, 3] and wq[5, 9] infinite, at both tile sizes: K's channel 7 and Q's channel 5 are
    +-inf (no NaN from the split's remainders), every other value has the bits it has without."""
    from paper_2509_10466_amd import Inpainter
    cfg = dataclasses.replace(MID, blocks=1)
    f, m = _clips(clips, 240, 432)
    N, C = clips * 5 * 60 * 108, cfg.dim

    def qkv(wk, wq):
        W = drsynth.make_weights(cfg, 3)
        W["blk0.wk"][7, 3] += np.float32(wk)
        W["blk0.wq"][5, 9] += np.float32(wq)
        eng = Inpainter(cfg, W)
        eng(f, m, "fp32", "all")
        return (eng.inspect("kv", N * 2 * C * 4).view(torch.float32).reshape(N, 2 * C).cpu(),
                eng.inspect("q", N * C * 4).view(torch.float32).reshape(N, C).cpu())

    for want, got, channel in zip(qkv(0, 0), qkv(np.inf, -np.inf), (7, 5)):
        others = [c for c in range(want.shape[1]) if c != channel]
        assert torch.isinf(got[:, channel]).all()
        assert torch.equal(got[:, others], want[:, others]) and torch.isfinite(want).all()


def test_overflowing_query_weight_gradient_is_infinite():
    """One query token, channel 11 of the first LayerNorm's output near 1e25 (its weights zero, so
    the forward does not see it) and an output gradient near 1e25: the query weights' gradients
    (rows through a table) of that input channel are products beyond the FP32 range, +-inf."""
    from paper_2509_10466_amd import Inpainter
    from paper_2509_10466_amd.api import unflatten_params
    cfg = dataclasses.replace(MID, blocks=1)
    W = drsynth.make_weights(cfg, 2, qk_std=0.2)
    W["blk0.ln1.g"][11] = 1e25
    W["blk0.ln1.b"][11] = 0
    for name in ("wq", "wk", "wv"):
        W[f"blk0.{name}"][:, 11] = 0
    eng = Inpainter(cfg, W)
    f, m = _clips(1, 40, 72)
    m.zero_()
    m[0, 1, 8:12, 20:24] = 1
    pred, saved = eng.train_forward(f, m)
    dpred = torch.zeros_like(pred)
    dpred[0, 1, 8:12, 20:24] = 1e25 * torch.randn(4, 4, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    g = unflatten_params(cfg, eng.train_backward(saved, dpred).cpu())["blk0.wq"]
    saved.close()
    others = [c for c in range(cfg.dim) if c != 11]
    assert torch.isinf(g[:, 11]).all()
    assert torch.isfinite(g[:, others]).all() and (g[:, others] != 0).any()


@pytest.mark.parametrize("mode", ["clip", "train"])
def test_weights_that_are_not_numbers_cost_no_more_than_plain_fp32(mode):
    """A diverged network also runs its products as FP32 fused multiply-adds, some 3 times as long
    as the split ones: 8 times as long leaves room (recomputed one result at a time: 33 times for
    the clip, 65 for the training step)."""
    from paper_2509_10466_amd import Inpainter
    cfg = drsynth.NETS["clip240"]
    f, m = _clips(1, 240, 432)
    dpred = torch.ones_like(f)

    def ms(W):
        eng = Inpainter(cfg, W)

        def once():
            if mode == "clip":
                return eng(f, m, "fp32")
            _, saved = eng.train_forward(f, m)
            g = eng.train_backward(saved, dpred)
            saved.close()
            return g

        out = once()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        for _ in range(3):
            once()
        ev[1].record()
        torch.cuda.synchronize()
        eng.close()
        return ev[0].elapsed_time(ev[1]) / 3, out

    W = drsynth.make_weights(cfg, 0)
    finite, out = ms(W)
    assert torch.isfinite(out).all()
    W["blk0.w1"][0, 5] = np.nan
    diverged, out = ms(W)
    print(f"{mode}: {finite:.2f} ms, diverged {diverged:.2f} ms", flush=True)
    assert torch.isnan(out).any()
    assert diverged < 8 * finite
