"""The three bf16 planes that FP32 products are formed from: what the split keeps and what the six
products of a pair leave out, in NumPy on the CPU."""
import numpy as np
import torch


def _bf16(x):
    """Rounded to bf16 (nearest even, subnormals kept)."""
    return torch.from_numpy(x).bfloat16().float().numpy()


def _planes(a):
    a1 = (a.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    r = a - a1
    a2 = _bf16(r)
    return a1, a2, _bf16(r - a2)


def _floats(rng, n, lo, hi):
    """Random significands, exponents lo .. hi - 1."""
    return np.ldexp(rng.uniform(1, 2, n), rng.integers(lo, hi, n)).astype(np.float32) * rng.choice([-1, 1], n).astype(np.float32)


def test_planes_are_the_float_exactly_from_2_to_the_minus_110():
    rng = np.random.default_rng(0)
    a = _floats(rng, 400000, -110, 128)
    a = a[np.isfinite(a)]
    assert np.array_equal(sum(p.astype(np.float64) for p in _planes(a)), a.astype(np.float64))


def test_smaller_values_lose_at_most_2_to_the_minus_134():
    rng = np.random.default_rng(1)
    a = np.concatenate([_floats(rng, 200000, -149, -110), np.float32([0.0, 2.0 ** -149, 2.0 ** -126])])
    lost = np.abs(sum(p.astype(np.float64) for p in _planes(a)) - a.astype(np.float64))
    assert 0 < lost.max() <= 2.0 ** -134


def test_six_products_leave_out_at_most_2_to_the_minus_22():
    """Remainders are largest against the value just above a power of two, where a1 is smallest."""
    rng = np.random.default_rng(2)
    wide = _floats(rng, 400000, -20, 20), _floats(rng, 400000, -20, 20)
    near = [rng.uniform(1, 1.03, 400000).astype(np.float32) for _ in range(2)]
    for a, w in (wide, near):
        pa, pw = ([p.astype(np.float64) for p in _planes(x)] for x in (a, w))
        kept = pa[2] * pw[0] + pa[1] * pw[1] + pa[0] * pw[2] + pa[1] * pw[0] + pa[0] * pw[1] + pa[0] * pw[0]
        exact = a.astype(np.float64) * w.astype(np.float64)
        rel = np.abs(kept - exact) / np.abs(exact)
        assert rel.max() <= 1.001 * 2.0 ** -22
    assert rel.max() > 2.0 ** -23 and rel.mean() < 2.0 ** -24
