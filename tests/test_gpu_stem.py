"""GPU parity of the fused stems: the dense 7x7/2 stem with its max-pool
(against the two calls it stands for, bit for bit: the same operands in the
same order), the stem on image blocks (against the oracle's split, 3-pixel
BlockPad and convolution, by the convolution bound) and the max-pool of
packed stacks (against pad_halo + maxpool_halo, bit for bit).  Sizes: tiles cut
at either side, maps smaller than a tile, one to four channels, channel
counts that are not multiples of 64, stacks without room for every block."""
from __future__ import annotations

import numpy as np
import pytest
import torch
import torch.nn.functional as F

import oracle
from parity_util import assert_conv_close, log
from paper_2011_12025_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2011_12025_amd._binding as b
    b.lib()
    oracle.set_threads(0)


def cl(t):
    return t.cuda().contiguous(memory_format=torch.channels_last)


def image(seed, N, C, H, W, dtype):
    """Channels-last memory also where one channel makes both formats the same."""
    x = inputs.feature_map(seed, N, C, H, W, dtype).cuda()
    return torch.empty((N, C, H, W), dtype=x.dtype, device="cuda", memory_format=torch.channels_last).copy_(x)


@pytest.mark.parametrize("dtype,N,C,Co,H,W", [
    ("f16", 1, 3, 64, 64, 128), ("bf16", 2, 3, 64, 130, 266), ("f16", 2, 3, 72, 67, 70), ("bf16", 1, 4, 8, 1, 2),
    ("f16", 1, 1, 40, 9, 514), ("bf16", 3, 2, 128, 61, 62),
    ("f16", 24, 3, 64, 131, 386)])  # more 16-row tiles than CUs: the 8-row tiles
def test_stem_pool_equals_its_two_calls(dtype, N, C, Co, H, W):
    import paper_2011_12025_amd as sb
    log(f"[stem pool] {dtype} {N}x{C}x{H}x{W} -> {Co}")
    x = image(190, N, C, H, W, dtype)
    w, b = inputs.conv_weight(190, Co, C, 7, dtype).cuda(), inputs.conv_bias(190, Co, 49 * C, dtype).cuda()
    y = sb.stem_pool(x, w, b)
    ref = sb.maxpool(sb.conv2d(x, w, b, stride=2, padding=3, relu=True), 3, 2, 1)
    torch.cuda.synchronize()
    assert y.shape == ref.shape and torch.equal(y, ref)


def test_stem_pool_infinity_stays_in_its_windows():
    import paper_2011_12025_amd as sb
    x = inputs.feature_map(191, 1, 3, 64, 128, "f16")
    x[0, 1, 31, 61] = float("inf")
    w = inputs.conv_weight(191, 64, 3, 7, "f16")
    y = sb.stem_pool(cl(x), w.cuda()).cpu().float()
    ref = F.max_pool2d(F.conv2d(x.double(), w.double(), stride=2, padding=3).clamp(min=0), 3, 2, 1)
    assert torch.equal(torch.isinf(y), torch.isinf(ref)) and not torch.isnan(y).any()


@pytest.mark.parametrize("dtype,N,C,Co,grid,bs,mask_kind,short,relu", [
    ("f16", 1, 3, 64, (2, 3), 128, "bernoulli", 0, True), ("bf16", 2, 3, 64, (3, 2), 64, "bernoulli", 0, False),
    ("f16", 1, 4, 72, (3, 3), 8, "bernoulli", 0, True), ("bf16", 1, 1, 8, (2, 2), 36, "high", 0, True),
    ("f16", 2, 2, 64, (2, 2), 20, "low", 0, True), ("f16", 1, 3, 64, (3, 4), 64, "bernoulli", 2, True)])
def test_stem_blocks_matches_oracle(dtype, N, C, Co, grid, bs, mask_kind, short, relu):
    import paper_2011_12025_amd as sb
    GH, GW = grid
    H, W = GH * bs, GW * bs
    log(f"[stem blocks] {dtype} {N}x{C} grid {grid} bs={bs} {mask_kind} short={short}")
    mask = {"high": np.ones, "low": np.zeros}.get(mask_kind, lambda *_: None)((N, GH, GW), np.uint8)
    mask = inputs.mask_bernoulli(192, N, GH, GW, 0.5) if mask is None else mask
    x = image(192, N, C, H, W, dtype)
    w, b = inputs.conv_weight(192, Co, C, 7, dtype), inputs.conv_bias(192, Co, 49 * C, dtype)
    nh, nl = max(0, int(mask.sum()) - short), max(0, int((mask == 0).sum()) - short)
    md = torch.from_numpy(mask).cuda()
    ho, lo = sb.stem_blocks(x, md, bs, w.cuda(), b.cuda(), counts=(nh, nl), relu=relu)
    if short:  # blocks without a place count as absent: the three calls know how
        hp, lp = sb.pad_halo(*sb.split(x, md, bs, counts=(nh, nl)), md, bs, H, W, 3)
        hp, lp = hp.cpu().float().numpy(), lp.cpu().float().numpy()
    else:
        hp, lp = oracle.pad_halo(*oracle.split(x.cpu().float().numpy(), mask, bs, dtype), mask, bs, H, W, dtype, 3)
    torch.cuda.synchronize()
    for got, P, name in ((ho, hp, "hi"), (lo, lp, "lo")):
        if P.shape[0] == 0:
            continue
        ref = oracle.conv_block_general(P, 3, w.float().numpy(), 2, 1, b.float().numpy())
        assert_conv_close(got, np.maximum(ref, 0.0) if relu else ref, dtype, 49 * C, f"stem_blocks {name}")


@pytest.mark.parametrize("dtype,N,C,grid,bs,p_low,short", [
    ("f16", 1, 64, (2, 3), 64, 0.5, 0), ("bf16", 2, 8, (3, 3), 4, 0.4, 0), ("f16", 1, 24, (2, 4), 12, 0.6, 1),
    ("bf16", 1, 72, (2, 2), 20, 1.0, 0), ("f16", 1, 16, (3, 2), 32, 0.0, 0)])
def test_maxpool_blocks_equals_its_two_calls(dtype, N, C, grid, bs, p_low, short):
    import paper_2011_12025_amd as sb
    GH, GW = grid
    H, W = GH * bs, GW * bs
    log(f"[maxpool blocks] {dtype} {N}x{C} grid {grid} bs={bs}")
    mask = torch.from_numpy(inputs.mask_bernoulli(193, N, GH, GW, p_low)).cuda()
    nh, nl = (max(0, n - short) for n in sb.count(mask))
    hi, lo = sb.split(image(193, N, C, H, W, dtype), mask, bs, counts=(nh, nl))
    got = sb.maxpool_blocks(hi, lo, mask, bs, H, W)
    ref = sb.maxpool_halo(*sb.pad_halo(hi, lo, mask, bs, H, W, 1), mask, bs, H, W, 1, 3, 2)
    torch.cuda.synchronize()
    for g, r in zip(got, ref):
        assert g.shape == r.shape and torch.equal(g, r)


def test_maxpool_blocks_nan_and_infinity():
    import paper_2011_12025_amd as sb
    H, W, bs = 64, 96, 32
    mask = torch.tensor([[[1, 0, 1], [0, 1, 0]]], dtype=torch.uint8, device="cuda")
    x = image(194, 1, 8, H, W, "f16")
    x[0, 1, 3:12, 5:14] = float("nan")  # whole windows and parts of some, in a high block
    x[0, 2, 20:30, 40:52] = float("nan")  # ... and in a low one
    x[0, 3, 28:36, 26:70] = float("-inf")  # across blocks
    x[0, 4, 33, 33] = float("inf")
    hi, lo = sb.split(x, mask, bs, counts=(3, 3))
    got = sb.maxpool_blocks(hi, lo, mask, bs, H, W)
    ref = sb.maxpool_halo(*sb.pad_halo(hi, lo, mask, bs, H, W, 1), mask, bs, H, W, 1, 3, 2)
    torch.cuda.synchronize()
    for g, r in zip(got, ref):
        assert torch.equal(g, r) and not torch.isnan(g).any()
    assert any(bool((r[:, 1] == float("-inf")).any()) for r in ref)
