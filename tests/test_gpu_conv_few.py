"""Convolutions with at most four input channels on their own kernel, against the oracle: ragged pixel groups and channel tiles, strides,
filters whose taps do not fill a chunk, rows of several workgroups, windows of larger tensors, non-finite values, the fused form."""
import math

import numpy as np
import pytest
import torch

from paper_1903_06498_amd import binding as B
from paper_1903_06498_amd import workloads as W
from tests.util import SENTINEL_F, SENTINEL_I, parity, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["bf16", "f32", "i8"])
@pytest.mark.parametrize("shape", [(2, 19, 18, 3, 64, 7, 7, 2, 3), (1, 9, 33, 3, 20, 3, 3, 1, 1), (3, 12, 11, 2, 70, 5, 5, 2, 2), (1, 8, 17, 4, 16, 1, 4, 1, 0),
                                   (1, 21, 40, 2, 33, 5, 3, 3, 1), (2, 7, 7, 3, 129, 7, 7, 1, 3), (1, 3, 3, 3, 5, 2, 2, 1, 0)])
@pytest.mark.parametrize("ty", [0, 1, 3])
def test_few_channels(shape, dt, ty, monkeypatch):
    monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,conv_few=1,conv_few_ty={ty}")
    N, H, Wd, Ci, Co, R, S, s, p = shape
    blk = W.conv2d_block(N, H, Wd, Ci, Co, R, S, s, p, dt, "i32" if dt == "i8" else "f32")
    sb = B.StripeBlock(blk)
    name = sb.info["kernel"]
    sb.close()
    if name.startswith("contract_"):      # fp32 and bf16 blocks whose literal kernel holds 64 sums per output
        monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,conv_few=2,conv_few_ty={ty}")
    info, _ = parity(blk, [W.seeded_tensor((N, H, Wd, Ci), dt, 0), W.seeded_tensor((R, S, Co, Ci), dt, 1)], what=f"few {shape} {dt}", threads=8)
    assert info["kernel"].startswith(f"conv_few_{dt}_c{Ci}"), info["kernel"]


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_non_finite_values(dt, monkeypatch):
    """Infinities and NaN at the border of the image and of the filter: what a constraint removes contributes nothing."""
    blk = W.conv2d_block(1, 13, 20, 3, 20, 5, 5, 2, 2, dt, "f32")
    ins = [W.seeded_tensor(r.sizes, dt, i) for i, r in enumerate(blk.refs[:2])]
    ins[0][0, 0, 0, 1] = math.inf
    ins[0][0, 6, 19, 2] = -math.inf
    ins[1][0, 0, 3, 0] = math.inf
    ins[1][4, 4, 18, 2] = math.nan
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,conv_few=2")
    got, sb = run_gpu(blk, ins, return_block=True)
    assert sb.info["kernel"].startswith("conv_few_"), sb.info["kernel"]
    want = run_gpu(blk, ins, "generic")
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want))
    assert np.array_equal(np.isneginf(got), np.isneginf(want)) and np.isinf(want).any() and np.isnan(want).any()
    fin = np.isfinite(want)
    assert fin.any() and np.allclose(got[fin], want[fin], rtol=1e-5, atol=75 * 2.0 ** -24 * 75)      # 75 products of order 1 in fp32


@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
@pytest.mark.parametrize("Co", [64, 18])
def test_fused_bias_relu(out_dt, Co, monkeypatch):
    """The following statement in the store, inputs and bias behind unaligned addresses, an output with and without whole vectors."""
    monkeypatch.setenv("STRIPE_TUNE", "conv_few=2")
    prog = W.conv_bias_relu_program(2, 30, 26, 3, Co, 7, 7, 2, 3, "bf16", out_dt)
    sb = B.StripeBlock(prog)
    assert sb.info["kernel"].startswith("conv_few_") and "+bias_relu" in sb.info["kernel"] and sb.info["workspace_bytes"] == 0, sb.info
    host = [W.seeded_tensor(r.sizes, r.dtype, i) for i, r in enumerate(r for r in prog.refs if r.dir == "in")]
    held = []
    for t in host:
        big = torch.zeros(t.numel() + 1, dtype=t.dtype, device="cuda")
        big[1:] = t.reshape(-1).cuda()
        held.append(big[1:])
    out = torch.full((2, 15, 13, Co), -7.0, dtype=torch.bfloat16 if out_dt == "bf16" else torch.float32, device="cuda")
    sb.run(held, out)
    sb.close()
    x, f, b = (t.double() for t in host)
    pre = torch.nn.functional.conv2d(x.permute(0, 3, 1, 2), f.permute(2, 3, 0, 1), stride=2, padding=3) + b[:, None, None]
    want = torch.relu(pre).permute(0, 2, 3, 1)
    mag = torch.nn.functional.conv2d(x.abs().permute(0, 3, 1, 2), f.abs().permute(2, 3, 0, 1), stride=2, padding=3).permute(0, 2, 3, 1) + b.abs()
    tol = 148 * 2.0 ** -24 * mag + (2.0 ** -8 * want if out_dt == "bf16" else 0)      # 147 products and the bias in fp32, half a step of bf16
    assert bool(((out.double().cpu() - want).abs() <= tol).all())


def test_window_of_a_larger_image(monkeypatch):
    """An input whose pixels are four channels apart and whose rows are longer: the last pixel's load ends with the operand."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,conv_few=2")
    for dt in ("bf16", "i8", "f32"):
        blk = W.conv2d_block(2, 11, 12, 3, 24, 3, 3, 1, 1, dt, "i32" if dt == "i8" else "f32")
        dense = [W.seeded_tensor((2, 11, 12, 3), dt, 0), W.seeded_tensor((3, 3, 24, 3), dt, 1)]
        want = run_gpu(blk, dense, "generic")
        got, sb = run_gpu(blk, dense, return_block=True)
        assert sb.info["kernel"].startswith("conv_few_"), sb.info["kernel"]
        if dt == "i8":
            assert np.array_equal(got, want)
        else:
            assert np.allclose(got, want, rtol=1e-5, atol=27 * 2.0 ** -24 * 27)


@pytest.mark.parametrize("shape,dt,most", [((4, 51, 51, 3, 24, 7, 7, 1, 3), "bf16", 5.7e-8), ((4, 35, 35, 4, 32, 2, 2, 1, 0), "f32", 6.7e-8),
                                           ((4, 69, 69, 4, 32, 7, 7, 4, 3), "f32", 9.6e-8)])
def test_sums_are_short_chains(shape, dt, most, monkeypatch):
    """The error in 64 bits of a sum grows with its chain of roundings.  224 bf16 products in one chain are 6.6e-8 off in the 2-norm, 16 fp32
    products 7.5e-8, 13 such chains added one after the other 1.01e-7; as four sums of at most 64 products, two of 8 and four of at most 4
    chains 5.0e-8, 6.1e-8 and 9.0e-8."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,conv_few=2")
    N, H, Wd, Ci, Co, R, S, s, p = shape
    g = torch.Generator().manual_seed(5)
    x, f = (torch.randn(n, generator=g).to(torch.bfloat16 if dt == "bf16" else torch.float32) for n in ((N, H, Wd, Ci), (R, S, Co, Ci)))
    got, sb = run_gpu(W.conv2d_block(N, H, Wd, Ci, Co, R, S, s, p, dt, "f32"), [x, f], return_block=True)
    assert sb.info["kernel"].startswith("conv_few_"), sb.info["kernel"]
    want = torch.nn.functional.conv2d(x.double().permute(0, 3, 1, 2), f.double().permute(2, 3, 0, 1), stride=s, padding=p).permute(0, 2, 3, 1).numpy()
    err = np.linalg.norm(got.reshape(want.shape) - want) / np.linalg.norm(want)
    assert err <= most, err


@pytest.mark.parametrize("dt", ["bf16", "i8", "f32"])
@pytest.mark.parametrize("Ci,extra", [(3, 1), (2, 0), (2, 3), (4, 3)])
def test_windows_of_larger_tensors(Ci, extra, dt, monkeypatch):
    """Image, filter and output as windows: pixels `extra` channels further apart, longer rows, origins and ends inside the parents.
    What lies beside the windows (NaN; int8: 127) is read by no sum, what lies beside the output stays: the same bits as from dense
    tensors, which the oracle is asked about too."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,conv_few=2")
    odt = "i32" if dt == "i8" else "f32"
    N, H, Wd, Co, R, S = 2, 11, 21, 22, 3, 5
    dense_ins = [W.seeded_tensor((N, H, Wd, Ci), dt, 0), W.seeded_tensor((R, S, Co, Ci), dt, 1)]
    dense = W.conv2d_block(N, H, Wd, Ci, Co, R, S, 2, 1, dt, odt)
    info, _ = parity(dense, dense_ins, what=f"dense {Ci} {dt}")
    want, sb = run_gpu(dense, dense_ins, return_block=True)
    sb.close()
    block = W.conv2d_block(N, H, Wd, Ci, Co, R, S, 2, 1, dt, odt)
    osz = block.refs[2].sizes
    parents = [(N + 1, H + 3, Wd + 5, Ci + extra), (R + 1, S + 2, Co + 3, Ci + extra), (N + 1, osz[1] + 2, osz[2] + 1, Co + 6)]
    W.embed(block, [(1, 2, 3, extra // 2), (1, 1, 2, extra // 2), (0, 1, 1, 4)], parents)
    ins = []
    for r, t, sizes in zip(block.refs, dense_ins, parents):
        big = torch.full(sizes, 127 if dt == "i8" else math.nan, dtype=t.dtype)
        big[tuple(slice(c, c + n) for c, n in zip(r.access_const, r.sizes))] = t
        ins.append(big)
    got, sb = run_gpu(block, ins, return_block=True)
    assert sb.info["kernel"] == info["kernel"] and sb.info["kernel"].startswith("conv_few_"), (sb.info["kernel"], info["kernel"])
    sb.close()
    image = np.full(int(np.prod(parents[2])), SENTINEL_I if odt == "i32" else np.float32(SENTINEL_F), dtype=got.dtype)
    image[:got.size] = got
    image = image.reshape(parents[2])
    inside = tuple(slice(c, c + n) for c, n in zip((0, 1, 1, 4), osz))
    assert np.array_equal(image[inside], want.reshape(osz))
    image[inside] = SENTINEL_I if odt == "i32" else np.float32(SENTINEL_F)
    assert (image == (SENTINEL_I if odt == "i32" else np.float32(SENTINEL_F))).all()


@pytest.mark.parametrize("dt", ["bf16", "i8", "f32"])
@pytest.mark.parametrize("sy,sx,py,px,R,S", [(1, 3, 2, 0, 5, 3), (3, 1, 0, 3, 2, 7), (2, 1, 1, 2, 3, 4)])
def test_asymmetric_strides_and_pads(sy, sx, py, px, R, S, dt, monkeypatch):
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,conv_few=2")
    N, H, Wd, Ci, Co = 2, 17, 35, 3, 37
    Ho, Wo = (H + 2 * py - R) // sy + 1, (Wd + 2 * px - S) // sx + 1
    bufs = [W.Buffer("I", "in", dt, (N, H, Wd, Ci)), W.Buffer("F", "in", dt, (R, S, Co, Ci)),
            W.Buffer("O", "out", "i32" if dt == "i8" else "f32", (N, Ho, Wo, Co))]
    ya, xa = f"{sy}*y + i - {py}", f"{sx}*x + j - {px}"
    blk = W.flat_block(bufs, dict(n=N, y=Ho, x=Wo, i=R, j=S, c=Ci, k=Co),
                       [(["n", ya, xa, "c"], "assign"), (["i", "j", "k", "c"], "assign"), (["n", "y", "x", "k"], "add")],
                       constraints=[f"{ya} >= 0", f"{H - 1 + py} - {sy}*y - i >= 0", f"{xa} >= 0", f"{Wd - 1 + px} - {sx}*x - j >= 0"])
    info, _ = parity(blk, [W.seeded_tensor((N, H, Wd, Ci), dt, 0), W.seeded_tensor((R, S, Co, Ci), dt, 1)], what=f"{sy} {sx} {py} {px} {dt}")
    assert info["kernel"].startswith(f"conv_few_{dt}_c3"), info["kernel"]
