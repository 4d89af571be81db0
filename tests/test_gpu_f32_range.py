"""fp32 expert FFN of many rows per expert at both ends of the number range: products that overflow, products just below the largest
float, operands that three bf16 parts cannot hold.  Expected values from 64-bit sums; what the fp32 instruction gives as infinities
has to be infinite, of the same sign, and no no-number."""
import numpy as np
import pytest
import torch

from paper_2605_18643_amd import zeda

pytestmark = pytest.mark.gpu

# wide (N * 2I and N * H at least 16384), 20 rows per expert: two blocks of token rows, the second one ragged
T, H, I, N = 160, 2048, 1024, 8
E = torch.arange(T) // (T // N)


def _ffn(x, wg, wu, wd):
    d = zeda.make_desc(T, H, I, N, 0, 1, "f32")
    off = (torch.arange(N + 1) * (T // N)).to(torch.int32).cuda()
    slots = torch.arange(T, dtype=torch.int32, device="cuda")
    y = torch.full((T, H), float("nan"), device="cuda")
    ws = torch.empty(zeda.expert_ffn_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    zeda.zeda_expert_ffn(d, x.cuda(), wg.cuda(), wu.cuda(), wd.cuda(), off, slots, off[-1:], y, ws)
    torch.cuda.synchronize()
    return ws[: T * I * 4].view(torch.float32).view(T, I).cpu(), y.cpu()


def _sums(tok, w):
    """[T, F]: row t times the weights of its expert, in 64 bits."""
    return torch.bmm(tok.double().view(N, T // N, -1), w.double().transpose(1, 2).contiguous()).view(T, -1)


def _normal(g, *shape, std=1.0):
    return std * torch.randn(*shape, generator=g)


def _err(got, want):
    return float((got.double() - want).norm() / want.norm())


def _layer(seed):
    """Ordinary weights; coordinate 6 of every token is 1 and the gate rows are 0.5 there and 0 elsewhere: every gate is exactly 0.5."""
    g = torch.Generator().manual_seed(seed)
    x, wu, wd = _normal(g, T, H), _normal(g, N, I, H, std=0.03), _normal(g, N, H, I, std=0.03)
    wg = torch.zeros(N, I, H)
    x[:, 6], wg[:, :, 6] = 1.0, 0.5
    return g, x, wg, wu, wd


SILU_HALF = 0.5 / (1.0 + np.exp(-0.5))


def test_overflowing_products_are_infinite():
    """One element of a token times one of a weight row above the largest float, in gate/up and in the down projection."""
    g, x, wg, wu, wd = _layer(1)
    rows, feats = slice(3, T, 5), slice(1, I, 7)
    x[rows, 5] = 1e22 * (1 + torch.rand(len(x[rows]), generator=g)) * torch.where(torch.rand(len(x[rows]), generator=g) < 0.5, -1.0, 1.0)
    wu[:, feats, 5] = 1e21 * (1 + torch.rand(N, len(range(1, I, 7)), generator=g))
    act, _ = _ffn(x, wg, wu, wd)
    got = act[rows, feats]
    assert not torch.isnan(act).any()
    assert torch.isinf(got).all() and torch.equal(got > 0, (x[rows, 5] > 0)[:, None].expand_as(got))
    # activations of 1e22 against weights of 1e21 (the up rows of feature 9 see a coordinate that is 1e22)
    g, x, wg, wu, wd = _layer(2)
    x[rows, 5], wu[:, 9, :], wu[:, 9, 5] = 1e22, 0.0, 2.0
    wu[:, 9, 6] = 0.0
    wd[:, feats, 9] = 1e21 * (1 + torch.rand(N, len(range(1, I, 7)), generator=g))
    act, y = _ffn(x, wg, wu, wd)
    assert (act[rows, 9] > 5e21).all() and not torch.isnan(y).any() and torch.isposinf(y[rows, feats]).all()
    other = torch.ones(T, dtype=torch.bool)
    other[rows] = False
    assert torch.isfinite(y[other]).all()


def test_products_just_below_the_largest_float_stay_finite():
    """Both factors' leading parts may round up: the product of the parts would be infinite."""
    g, x, wg, wu, wd = _layer(3)
    x[:, 5] = 1.84e19 * (1 + 0.002 * torch.rand(T, generator=g))
    wu[:, :, 5] = 1.84e19 * (1 + 0.002 * torch.rand(N, I, generator=g))
    act, _ = _ffn(x, wg, wu, torch.zeros_like(wd))
    want = (SILU_HALF * _sums(x, wu))
    assert torch.isfinite(act).all()
    # (a rounding of the product, of the sums and of the activation, expf: a few last places)
    assert float(((act.double() - want) / want).abs().max()) < 1e-6


@pytest.mark.parametrize("std", [1e-12, 1e-15, 3e-18, 1e-18, 5e-19])
def test_small_tokens_give_small_activations(std):
    """Activations of std^2 / 2, down to 1e-37, times ordinary weights: nothing a float does not hold."""
    g = torch.Generator().manual_seed(4)
    x, wg, wu, wd = _normal(g, T, H, std=std), _normal(g, N, I, H, std=0.03), _normal(g, N, I, H, std=0.03), _normal(g, N, H, I, std=0.03)
    act, y = _ffn(x, wg, wu, wd)
    a, b = _sums(x, wg), _sums(x, wu)
    # Sums of 32 products at 24 bits: 1e-7 as for ordinary numbers.  Activations and products with them below the smallest normal
    # float (1.2e-38) are kept to 2^-150 = 7e-46 each: 4e-8 of activations of 2e-38 (5e-19), 2-norm, and less of their sums.
    assert _err(act, a / (1 + torch.exp(-a)) * b) < 4e-7
    assert _err(y, _sums(act, wd)) < 4e-7


def test_small_tokens_against_large_weights():
    """Products of ordinary size from factors at the ends of the range."""
    g = torch.Generator().manual_seed(5)
    x, wd = _normal(g, T, H, std=1e-36), _normal(g, N, H, I, std=0.03)
    wg, wu = _normal(g, N, I, H, std=0.03e36), _normal(g, N, I, H, std=0.03e36)
    act, y = _ffn(x, wg, wu, wd)
    a, b = _sums(x, wg), _sums(x, wu)
    assert _err(act, a / (1 + torch.exp(-a)) * b) < 1e-6 and _err(y, _sums(act, wd)) < 4e-7


def test_elements_at_the_window_edges():
    """Whole rows at the smallest and the largest magnitude that three parts take (2^-110, 2^60), and outside, against weights that
    give products of ordinary size, and single elements outside: the same precision, and a row's result does not depend on its
    neighbours."""
    g, x, wg, wu, wd = _layer(6)
    wu[:, : I // 2] *= 2.0 ** 50
    wu[:, :, 6] = 0.0  # (coordinate 6 makes the gates, 0.5 for every row)
    base, _ = _ffn(x, wg, wu, wd)
    scale, one = torch.ones(T), torch.zeros(T, dtype=torch.bool)
    for i, p in enumerate((-112, -111, -110, -109, -108, 57, 58, 59, 60)):
        scale[i::11] = 2.0 ** p
    one[9::11] = True
    xs = x * scale[:, None]
    xs[:, 6] = 1.0
    xs[one, 7], xs[one, 8] = 2.0 ** 62, -(2.0 ** -120)
    act, _ = _ffn(xs, wg, wu, wd)
    want = SILU_HALF * _sums(xs, wu)
    for t in range(T):
        for half in (slice(0, I // 2), slice(I // 2, I)):
            assert _err(act[t, half], want[t, half]) < 1e-6, (t, half, float(scale[t]))
    same = (scale == 1) & ~one
    assert same.any() and torch.equal(act[same], base[same])


def test_zeros_are_ordinary():
    """Rows and columns of zeros, as padding has them, and tokens that are zero altogether."""
    g, x, wg, wu, wd = _layer(7)
    x[::3, ::2], x[5::11], wu[:, ::4, 100:300] = 0.0, 0.0, 0.0
    act, y = _ffn(x, wg, wu, wd)
    a, b = _sums(x, wg), _sums(x, wu)
    assert _err(act, a / (1 + torch.exp(-a)) * b) < 1e-6 and _err(y, _sums(act, wd)) < 1e-6
    assert not act[5::11].any() and not y[5::11].any()
