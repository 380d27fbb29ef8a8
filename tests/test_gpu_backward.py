"""GPU parity of the backward pass against the CPU oracle's transposes.

BlockCombine and BlockSample transposed are bit-exact (a fixed-order fp32
2x2 sum, an exact quarter).  BlockPad transposed sums up to nine gradients per
pixel in fp32 on the GPU and in fp64 in the oracle: within one storage ulp
plus the fp32 rounding of the sum of the magnitudes.  The convolution's data
and weight gradients meet the convolution tolerance (max-norm relative 1e-4
fp32, 2e-2 fp16/bf16, plus the element-wise bound), and so do the whole
layer's gradients (dx, dw, db), on the same seeded inputs."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from parity_util import (NORM_TOL, ULP_SCALE, Case, assert_bitexact, assert_conv_close, f32, log, make_inputs,
                         to_dev)
from paper_2011_12025_amd import inputs

pytestmark = pytest.mark.gpu

TDT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}

CASES = [
    Case("c64_bs32_f16", "f16", 1, 64, 64, 64, 128, 32, seed=160),
    Case("c32_bs16_bf16", "bf16", 2, 32, 48, 32, 64, 16, seed=161),
    Case("ragged_f32", "f32", 2, 12, 20, 18, 30, 6, p_low=0.4, seed=162),
    Case("bs2_f16", "f16", 1, 8, 8, 8, 12, 2, seed=163),
    Case("c128_bs8_f16", "f16", 1, 128, 96, 32, 48, 8, seed=164),
    Case("allhigh_bf16", "bf16", 1, 16, 16, 32, 32, 8, mask_kind="high", seed=165),
    Case("alllow_f16", "f16", 1, 16, 16, 32, 32, 8, mask_kind="low", seed=166),
]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2011_12025_amd._binding as b
    b.lib()
    oracle.set_threads(0)


def up(a, dtype, layout):
    return to_dev(torch.from_numpy(np.ascontiguousarray(a)).to(TDT[dtype]), layout)


def _grad(seed, shape, dtype):
    return inputs.normal(seed, 9, shape, 1.0, dtype).float().numpy()


def _pad_bound(ref, abs_ref, dtype):
    return ULP_SCALE[dtype] * np.abs(ref) + 16 * 2.0 ** -24 * abs_ref + 1e-30


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_module_transposes(c, layout):
    import paper_2011_12025_amd as sb
    mask, x, w, b = make_inputs(c)
    log(f"[backward modules] {c.name} {layout}")
    md = torch.from_numpy(mask).cuda()
    nh, nl = int(mask.sum()), int(mask.size - mask.sum())
    lb = c.bs // 2
    # BlockCombine transposed
    dy = _grad(c.seed, (c.N, c.C, c.H, c.W), c.dtype)
    rh, rl = oracle.combine_backward(dy, mask, c.bs, c.dtype)
    dh, dl = sb.combine_backward(up(dy, c.dtype, layout), md, c.bs, counts=(nh, nl))
    torch.cuda.synchronize()
    assert_bitexact(dh, rh, "combine_backward hi")
    assert_bitexact(dl, rl, "combine_backward lo")
    # BlockSample transposed
    gh = _grad(c.seed + 1, (nh, c.C, c.bs, c.bs), c.dtype)
    gl = _grad(c.seed + 2, (nl, c.C, lb, lb), c.dtype)
    dx = sb.split_backward(up(gh, c.dtype, layout), up(gl, c.dtype, layout), md, c.bs, c.H, c.W)
    torch.cuda.synchronize()
    assert_bitexact(dx, oracle.split_backward(gh, gl, mask, c.bs, c.H, c.W, c.dtype), "split_backward")
    # BlockPad transposed, the three samplings
    ph = _grad(c.seed + 3, (nh, c.C, c.bs + 2, c.bs + 2), c.dtype)
    pl = _grad(c.seed + 4, (nl, c.C, lb + 2, lb + 2), c.dtype)
    for sampling in ["avg", "strided", "zero"]:
        rh, rl = oracle.pad_backward(ph, pl, mask, c.bs, c.H, c.W, c.dtype, sampling)
        ah, al = oracle.pad_backward(np.abs(ph), np.abs(pl), mask, c.bs, c.H, c.W, "f32", sampling)
        gh_, gl_ = sb.pad_backward(up(ph, c.dtype, layout), up(pl, c.dtype, layout), md, c.bs, c.H, c.W,
                                   sampling=sampling)
        torch.cuda.synchronize()
        for got, ref, mag, what in [(gh_, rh, ah, "hi"), (gl_, rl, al, "lo")]:
            g = f32(got)
            assert g.shape == ref.shape
            bad = np.abs(g - ref) > _pad_bound(ref, mag, c.dtype)
            assert not bad.any(), f"pad_backward {sampling} {what}: {bad.sum()} elements off, first " \
                                  f"{np.argwhere(bad)[0]}: {g[bad][0]} vs {ref[bad][0]}"


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_conv_gradients(c, layout):
    import paper_2011_12025_amd as sb
    mask, x, w, b = make_inputs(c)
    log(f"[backward conv] {c.name} {layout}")
    md = torch.from_numpy(mask).cuda()
    hi, lo = oracle.split(x.float().numpy(), mask, c.bs, c.dtype)
    hp, lp = oracle.pad(hi, lo, mask, c.bs, c.H, c.W, c.dtype)
    gho = _grad(c.seed + 5, (hp.shape[0], c.Co, c.bs, c.bs), c.dtype)
    glo = _grad(c.seed + 6, (lp.shape[0], c.Co, c.bs // 2, c.bs // 2), c.dtype)
    wf = w.float().numpy()
    dhp, dlp = sb.conv3x3_backward_data(up(gho, c.dtype, layout), up(glo, c.dtype, layout), md, c.bs, c.H, c.W,
                                        w.cuda())
    torch.cuda.synchronize()
    assert_conv_close(dhp, oracle.conv3x3_backward_data(gho, wf), c.dtype, 9 * c.Co, "dgrad hi")
    assert_conv_close(dlp, oracle.conv3x3_backward_data(glo, wf), c.dtype, 9 * c.Co, "dgrad lo")
    dw, db = sb.conv3x3_backward_weight(up(hp, c.dtype, layout), up(lp, c.dtype, layout), up(gho, c.dtype, layout),
                                        up(glo, c.dtype, layout), md, c.bs, c.H, c.W, bias=True)
    torch.cuda.synchronize()
    rw, rb = oracle.conv3x3_backward_weight([(hp, gho), (lp, glo)])
    npx = hp.shape[0] * c.bs * c.bs + lp.shape[0] * (c.bs // 2) ** 2
    assert_conv_close(dw, rw, c.dtype, npx, "wgrad")
    assert_conv_close(db, rb, c.dtype, npx, "bias grad")


# The implicit GEMM's partial sums take more than the general kernel's padded
# gradients: a workspace that holds only the latter runs the general kernel.
@pytest.mark.parametrize("least", [False, True])
def test_data_gradient_in_either_workspace(least):
    import ctypes

    from paper_2011_12025_amd import _binding as B
    c = Case("c16_co256_bs2", "f16", 1, 16, 256, 12, 20, 2, seed=170)
    mask, _, w, _ = make_inputs(c)
    nh = int(mask.sum())
    nl = mask.size - nh
    n = ctypes.c_size_t(0)
    shape = (B.SB_F16, B.SB_NHWC, 1, c.C, c.H, c.W)
    assert B.lib().segblocks_conv3x3_backward_data_workspace_size(*shape, c.bs, c.Co, nh, nl, ctypes.byref(n)) == 0
    parts = (nh * c.Co * 36 * 2, nl * c.Co * 25 * 2, c.C * c.Co * 9 * 2, mask.size * 2)
    general = sum(-(-p // 256) * 256 for p in parts)
    assert general < n.value
    need = general if least else n.value
    log(f"[backward data] {c.name} nh={nh} nl={nl} workspace {need}")
    gho, glo = _grad(c.seed + 5, (nh, c.Co, 2, 2), c.dtype), _grad(c.seed + 6, (nl, c.Co, 1, 1), c.dtype)
    dho, dlo, dw, dm = up(gho, "f16", "nhwc"), up(glo, "f16", "nhwc"), to_dev(w, "nhwc"), torch.from_numpy(mask).cuda()
    out = [up(np.full((k, c.C, e, e), np.nan, np.float32), "f16", "nhwc") for k, e in ((nh, 4), (nl, 3))]
    ws = torch.full((need + 512,), 255, dtype=torch.uint8, device="cuda")
    off = -ws.data_ptr() % 256
    P = lambda a: ctypes.c_void_p(a.data_ptr())
    rc = B.lib().segblocks_conv3x3_backward_data(P(dho), P(dlo), *shape, P(dm), c.bs, P(dw), c.Co, P(out[0]), P(out[1]),
                                                 nh, nl, ctypes.c_void_p(ws.data_ptr() + off), need,
                                                 ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, B.lib().segblocks_last_error().decode()
    torch.cuda.synchronize()
    assert bool((ws[off + need:] == 255).all()) and bool((ws[:off] == 255).all())
    wf = w.float().numpy()
    assert_conv_close(out[0], oracle.conv3x3_backward_data(gho, wf), "f16", 9 * c.Co, "dgrad hi")
    assert_conv_close(out[1], oracle.conv3x3_backward_data(glo, wf), "f16", 9 * c.Co, "dgrad lo")


@pytest.mark.parametrize("sampling", ["avg", "strided", "zero"])
@pytest.mark.parametrize("c", [CASES[0], CASES[2], CASES[4],
                               Case("stage1_full", "f16", 1, 64, 64, 256, 512, 32, seed=167)],
                         ids=lambda c: c.name)
def test_layer_backward(c, sampling):
    """The whole layer's gradients against the oracle's chain (which rounds
    every stored gradient where the GPU stores it); the last case is the
    benchmark's layer shape."""
    import paper_2011_12025_amd as sb
    mask, x, w, b = make_inputs(c)
    if sampling != "avg" and c.name == "stage1_full":
        pytest.skip("the full-size case runs with average sampling only")
    log(f"[backward layer] {c.name} {sampling}: oracle ...")
    dy = _grad(c.seed + 7, (c.N, c.Co, c.H, c.W), c.dtype)
    rdx, rdw, rdb = oracle.layer_backward(x.float().numpy(), mask, c.bs, w.float().numpy(), b.float().numpy(), dy,
                                          c.dtype, sampling)
    log(f"[backward layer] {c.name} {sampling}: gpu")
    layout = "nhwc"
    dx, dw, db = sb.layer_backward(to_dev(x, layout), torch.from_numpy(mask).cuda(), c.bs, w.cuda(),
                                   up(dy, c.dtype, layout), bias=True, sampling=sampling)
    torch.cuda.synchronize()
    # dx went through two rounded stages after the convolution: max-norm rule
    g = f32(dx).astype(np.float64)
    assert np.all(np.isfinite(g))
    rel = float(np.max(np.abs(g - rdx)) / max(np.max(np.abs(rdx)), 1e-30))
    assert rel <= NORM_TOL[c.dtype], f"dx relative error {rel:.3e}"
    npx = c.N * c.H * c.W
    assert_conv_close(dw, rdw, c.dtype, npx, "dw")
    assert_conv_close(db, rdb, c.dtype, npx, "db")


@pytest.mark.parametrize("sampling", ["avg", "strided", "zero"])
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
@pytest.mark.parametrize("c,short", [(c, 0) for c in CASES] + [(CASES[0], 2), (CASES[2], 3)],
                         ids=lambda v: v.name if isinstance(v, Case) else str(v))
def test_fused_first_and_last_step(c, short, layout, sampling):
    """split_pad and pad_split_backward against the two calls each stands for,
    bit for bit, also with stacks that lack room for some blocks."""
    import paper_2011_12025_amd as sb
    mask, x, w, b = make_inputs(c)
    md, xd = torch.from_numpy(mask).cuda(), to_dev(x, layout)
    lay = 1 if layout == "nhwc" else 0
    nh, nl = (max(0, int(n) - short) for n in (mask.sum(), mask.size - mask.sum()))
    log(f"[fused split/pad] {c.name} {layout} {sampling} {nh}/{nl}")
    got = sb.split_pad(xd, md, c.bs, counts=(nh, nl), layout=lay, sampling=sampling)
    ref = sb.pad(*sb.split(xd, md, c.bs, counts=(nh, nl), layout=lay), md, c.bs, c.H, c.W, layout=lay,
                 sampling=sampling)
    torch.cuda.synchronize()
    for g, r in zip(got, ref):
        assert g.shape == r.shape and torch.equal(g, r)
    lb = c.bs // 2
    gh = up(_grad(c.seed + 5, (nh, c.C, c.bs + 2, c.bs + 2), c.dtype), c.dtype, layout)
    gl = up(_grad(c.seed + 6, (nl, c.C, lb + 2, lb + 2), c.dtype), c.dtype, layout)
    dx = sb.pad_split_backward(gh, gl, md, c.bs, c.H, c.W, layout=lay, sampling=sampling)
    ref = sb.split_backward(*sb.pad_backward(gh, gl, md, c.bs, c.H, c.W, layout=lay, sampling=sampling), md, c.bs, c.H,
                            c.W, layout=lay)
    torch.cuda.synchronize()
    assert torch.equal(dx, ref)
