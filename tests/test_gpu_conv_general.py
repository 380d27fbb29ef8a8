"""GPU parity of the general convolution kernel where its staging and its tile
plan change: NCHW and channels-last, whole and partial K chunks, channel counts
whose channel tiles are unequal, tiles of 64, 128 and 256 pixels, odd filters,
tensors that are not 16-byte aligned, the three halo samplings; the fused
layer, the packed and the padded convolution share one order of sums, so they
agree bit for bit."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from parity_util import Case, assert_conv_close, log, make_inputs, to_dev, y64_from_stacks, oracle_stages

pytestmark = pytest.mark.gpu

CASES = [
    Case("plane_f32_partial", "f32", 1, 19, 21, 20, 40, 20, seed=200),        # 16 + 3 channels, odd filters
    Case("plane_f16_odd", "f16", 1, 35, 72, 24, 24, 12, seed=201),            # 32 + 3 channels; 48 + 24 out
    Case("plane_bf16_even", "bf16", 2, 64, 130, 24, 48, 24, p_low=0.3, seed=202),
    Case("small_tiles_f32", "f32", 1, 48, 16, 64, 64, 32, seed=203),          # tiles of 64 pixels
    Case("mid_tiles_f16", "f16", 1, 40, 40, 128, 256, 16, seed=204),          # tiles of 128 pixels
    Case("full_tiles_f32", "f32", 1, 32, 24, 264, 480, 24, seed=205),         # tiles of 256 pixels (rows 8 of 24)
    Case("bs256_f32", "f32", 1, 8, 8, 256, 256, 256, seed=206, mask_kind="high"),
    Case("bs4_bf16", "bf16", 2, 72, 8, 32, 32, 4, p_low=0.6, seed=207),
    Case("runs_and_rest_f16", "f16", 2, 24, 40, 84, 60, 12, seed=210),        # 70 blocks: runs of four, then single ones
    Case("all_low_f16", "f16", 1, 72, 40, 96, 64, 16, seed=211, mask_kind="low"),
    Case("all_low_f32", "f32", 1, 20, 72, 64, 128, 32, seed=212, mask_kind="low"),
]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2011_12025_amd._binding as b
    b.lib()
    oracle.set_threads(0)


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
@pytest.mark.parametrize("c", CASES, ids=[c.name for c in CASES])
def test_general_convolution(c, layout):
    import paper_2011_12025_amd as sb
    log(f"[general conv] {c.name} {layout}")
    mask, x, w, b = make_inputs(c)
    ref = oracle_stages(c, mask, x, w, b)
    md, xd, wd = torch.from_numpy(mask).cuda(), to_dev(x, layout), w.cuda()
    bd = None if b is None else b.cuda()
    y = sb.layer(xd, md, c.bs, wd, bd)
    assert_conv_close(y, y64_from_stacks(c, mask, ref["ho64"], ref["lo64"]), c.dtype, 9 * c.C, "layer")
    hi, lo = sb.split(xd, md, c.bs)
    packed = sb.block_conv3x3(hi, lo, md, c.bs, c.H, c.W, wd, bd, layout=1 if layout == "nhwc" else 0)
    hp, lp = sb.pad(hi, lo, md, c.bs, c.H, c.W)
    padded = sb.conv3x3(hp, lp, md, c.bs, c.H, c.W, wd, bd)
    torch.cuda.synchronize()
    for p, q, r in zip(packed, padded, (ref["ho64"], ref["lo64"])):
        assert_conv_close(p, r, c.dtype, 9 * c.C, "packed")
        assert_conv_close(q, r, c.dtype, 9 * c.C, "padded")
    # (channels-last packed stacks of 64 channels run elsewhere)
    if layout == "nchw" or c.C % 64:
        assert all(torch.equal(p, q) for p, q in zip(packed, padded))
        assert torch.equal(sb.combine(*padded, md, c.bs, c.H, c.W), y)


@pytest.mark.parametrize("sampling", ["strided", "zero"])
@pytest.mark.parametrize("dtype,layout", [("f32", "nchw"), ("f16", "nhwc")])
def test_general_convolution_samplings(dtype, layout, sampling):
    """Against the same layer as pad_ex + conv3x3 + combine, bit for bit."""
    import paper_2011_12025_amd as sb
    c = Case("sampling", dtype, 1, 40, 24, 48, 96, 24, seed=208)
    mask, x, w, b = make_inputs(c)
    md, xd, wd, bd = torch.from_numpy(mask).cuda(), to_dev(x, layout), w.cuda(), b.cuda()
    y = sb.layer(xd, md, c.bs, wd, bd, sampling=sampling)
    hp, lp = sb.pad(*sb.split(xd, md, c.bs), md, c.bs, c.H, c.W, sampling=sampling)
    ref = sb.combine(*sb.conv3x3(hp, lp, md, c.bs, c.H, c.W, wd, bd), md, c.bs, c.H, c.W)
    torch.cuda.synchronize()
    assert torch.equal(y, ref)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_general_convolution_unaligned(dtype):
    """Tensors one element past an aligned address take element-wise staging."""
    import paper_2011_12025_amd as sb
    c = Case("unaligned", dtype, 1, 24, 20, 32, 48, 16, seed=209)
    mask, x, w, b = make_inputs(c)
    md, bd = torch.from_numpy(mask).cuda(), b.cuda()
    ref = sb.layer(to_dev(x, "nhwc"), md, c.bs, w.cuda(), bd)
    xd, wd = to_dev(x, "nhwc"), w.cuda().contiguous(memory_format=torch.channels_last)

    def shifted(t):
        buf = torch.zeros(t.numel() + 1, dtype=t.dtype, device="cuda")
        return torch.as_strided(buf, t.shape, t.stride(), 1).copy_(t)

    y = sb.layer(shifted(xd), md, c.bs, shifted(wd), bd)
    torch.cuda.synchronize()
    assert torch.equal(y, ref)
