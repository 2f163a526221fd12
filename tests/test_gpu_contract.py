"""The general matrix-core contraction and the few-rows product against the oracle, at the edges of their tiles and fetch
forms.  Tolerances as in tests/util.py; integers bit-exact, elements no iteration writes untouched."""
import math
import random

import numpy as np
import pytest
import torch

from oracle import stripe_oracle as O
from paper_1903_06498_amd import binding as B
from paper_1903_06498_amd import workloads as W
from tests import brute
from tests.test_contract_fetch import PARTNERS
from tests.util import SENTINEL_I, parity, run_gpu

pytestmark = pytest.mark.gpu
TILES = ["128x128", "64x64", "32x32", "128x64"]


def random_block(seed, dt="i8"):
    inj = seed % 5 != 4
    return brute.random_block(random.Random(9100 + seed), seed % 3 == 2, dt, "i32" if dt == "i8" else "f32", "add", "mul", injective_out=inj,
                              max_range=9, contraction_roles=inj)


@pytest.mark.parametrize("seed", range(64))
def test_random_blocks(seed, monkeypatch):
    """Random small (nested) int8 sum-of-products blocks: negative strides, constraints over several indexes, passed values,
    shared output elements; every tile."""
    monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,contract_tile={seed % 4}")
    blk = random_block(seed)
    nrng = np.random.default_rng(seed)
    ins = [torch.from_numpy(nrng.integers(-3, 4, size=int(np.prod(r.sizes)), dtype=np.int8)) for r in blk.refs[:-1]]
    try:
        gpu, sb = run_gpu(blk, ins, return_block=True)
    except B.StripeError as e:
        assert e.status == 5, str(e)
        pytest.skip(f"rejected at create: {e}")
    res = O.evaluate(blk, [W.to_numpy(t) for t in ins], out=np.full(W.output_extent(blk), SENTINEL_I, np.int64))
    assert np.array_equal(gpu.astype(np.int64), res.out), sb.info["kernel"]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("seed", [s for s in range(60) if s % 5 != 4])
def test_random_float_blocks(seed, dt, monkeypatch):
    """The same in float, where a removed point's factor must not reach the sum: constrained blocks on every tile."""
    monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,contract_tile={seed % 4}")
    blk = random_block(seed, dt)
    try:
        parity(blk, [W.seeded_tensor(r.sizes, dt, i) for i, r in enumerate(blk.refs[:-1])], threads=1, what=f"seed {seed} {dt}")
    except B.StripeError as e:
        assert e.status == 5, str(e)
        pytest.skip(f"rejected at create: {e}")


def test_random_blocks_reach_the_kernel(monkeypatch):
    taken = 0
    for seed in range(64):
        monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,contract_tile={seed % 4}")
        try:
            sb = B.StripeBlock(random_block(seed))
        except B.StripeError:
            continue
        taken += sb.info["kernel"].startswith("contract_")
        sb.close()
    assert taken >= 12, taken


def matmul(M, N, K, dt, layout):
    bufs = [W.Buffer("A", "in", dt, (K, M) if layout == "tn" else (M, K)), W.Buffer("B", "in", dt, (N, K) if layout == "nt" else (K, N)),
            W.Buffer("C", "out", "i32" if dt == "i8" else "f32", (M, N))]
    return W.flat_block(bufs, dict(m=M, n=N, k=K), [(["k", "m"] if layout == "tn" else ["m", "k"], "assign"),
                                                    (["n", "k"] if layout == "nt" else ["k", "n"], "assign"), (["m", "n"], "add")])


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("layout", ["nn", "nt", "tn"])
@pytest.mark.parametrize("M,N,K,tile", [(2, 2, 2, 2), (33, 31, 17, 2), (7, 130, 1025, 2), (65, 63, 129, 1), (129, 127, 67, 0), (130, 65, 193, 3),
                                        (64, 64, 256, 1), (40, 36, 15, 2), (72, 8, 16, 1)])
def test_products(M, N, K, tile, layout, dt, monkeypatch):
    """Edges of tiles, K remainders inside one vector, operands with fewer rows than a vector, unaligned rows."""
    monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,contract_tile={tile},gemm_rows=0,gemm_dma=0")
    blk = matmul(M, N, K, dt, layout)
    ins = [W.seeded_tensor(blk.refs[0].sizes, dt, 0), W.seeded_tensor(blk.refs[1].sizes, dt, 1)]
    info, _ = parity(blk, ins, what=f"{layout} {M}x{N}x{K} {dt}")
    kernel = info["kernel"]
    if tile == 3 and dt != "f32" and kernel.endswith("2"):
        tile = 1        # columns fetched in vectors along the columns: the 128 x 64 tile has none of 2-byte and 1-byte elements
    assert kernel.startswith(f"contract_{dt}_{TILES[tile]}x"), kernel


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("shape", [(2, 19, 13, 3, 20, 5, 2, 2), (1, 9, 11, 8, 70, 3, 1, 1), (3, 7, 8, 13, 5, 1, 2, 0), (1, 14, 30, 24, 33, 7, 1, 3), (1, 6, 7, 9, 12, 3, 1, 1)])
@pytest.mark.parametrize("tile", [0, 1, 2, 3])
def test_convolutions(shape, dt, tile, monkeypatch):
    monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,contract_tile={tile},conv_igemm=0")
    N, H, Wd, Ci, Co, R, s, p = shape
    blk = W.conv2d_block(N, H, Wd, Ci, Co, R, R, s, p, dt, "i32" if dt == "i8" else "f32")
    info, _ = parity(blk, [W.seeded_tensor((N, H, Wd, Ci), dt, 0), W.seeded_tensor((R, R, Co, Ci), dt, 1)], what=f"conv {shape} {dt}")
    assert info["kernel"].startswith(("contract_", "gemm_")), info


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("R,s,Co", [(3, 2, 6), (2, 2, 8), (4, 2, 5), (3, 1, 8), (5, 3, 16), (2, 3, 4)])
def test_transposed_convolutions(R, s, Co, dt, monkeypatch):
    """Shared output elements (R > s), none (R <= s), gaps that stay unwritten (R < s) and rows beyond the last tap."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1")
    N, H, Wd, Ci = 2, 6, 9, 8
    bufs = [W.Buffer("I", "in", dt, (N, H, Wd, Ci)), W.Buffer("F", "in", dt, (R, R, Ci, Co)),
            W.Buffer("O", "out", "i32" if dt == "i8" else "f32", (N, s * (H - 1) + R + 1, s * (Wd - 1) + R + 1, Co))]
    blk = W.flat_block(bufs, dict(n=N, y=H, x=Wd, i=R, j=R, c=Ci, k=Co),
                       [(["n", "y", "x", "c"], "assign"), (["i", "j", "c", "k"], "assign"), (["n", f"{s}*y + i", f"{s}*x + j", "k"], "add")])
    info, _ = parity(blk, [W.seeded_tensor((N, H, Wd, Ci), dt, 0), W.seeded_tensor((R, R, Ci, Co), dt, 1)], what=f"transposed {R} {s} {dt}")
    assert info["kernel"].startswith("contract_"), info


@pytest.mark.parametrize("tile", [0, 1, 2, 3])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_infinities_at_removed_points(dt, tile, monkeypatch):
    """A removed point contributes nothing, also where the other operand is infinite: equal to the literal kernel."""
    blk = W.conv2d_block(1, 9, 8, 6, 10, 3, 3, 1, 1, dt, "f32")
    ins = [W.seeded_tensor((1, 9, 8, 6), dt, 0), W.seeded_tensor((3, 3, 10, 6), dt, 1)]
    ins[0] = ins[0].abs() + 0.5
    ins[1][0, 1, 3, 2] = math.inf
    ins[1][2, 2, 7, 0] = math.nan
    monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,contract_tile={tile}")
    got, sb = run_gpu(blk, ins, return_block=True)
    assert sb.info["kernel"].startswith(f"contract_{dt}_{TILES[tile]}x"), sb.info["kernel"]
    want = run_gpu(blk, ins, "generic")
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want)) and np.isinf(want).any()
    fin = np.isfinite(want)
    assert 0 < fin.sum() and np.allclose(got[fin], want[fin], rtol=1e-5, atol=1e-4)     # 54 products of order 1 in fp32: 54 * 2^-24 * sum |a b|


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("make", PARTNERS)
def test_partner_operand_ends_with_the_polyhedron(make, dt, monkeypatch):
    """Nothing behind an operand enters the result: the operands lie at the front of larger tensors, whose rest is once zero
    and once NaN; the results are the same bits, and the oracle's."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1")
    blk = make(dt)
    ins = [W.seeded_tensor(r.sizes, dt, i) for i, r in enumerate(blk.refs[:2])]
    info, _ = parity(blk, ins, what=make.__name__)
    assert info["kernel"].startswith("contract_"), info
    sb, images = B.StripeBlock(blk), []
    for rest in (0.0, math.nan):
        held = []
        for t in ins:
            big = torch.full((t.numel() + (1 << 20),), rest, dtype=t.dtype, device="cuda")
            big[:t.numel()] = t.reshape(-1).cuda()
            held.append(big)
        out = torch.zeros(W.output_extent(blk), dtype=torch.float32, device="cuda")
        sb.run(held, out)
        images.append(out.view(torch.int32).cpu().numpy())
    sb.close()
    assert np.array_equal(images[0], images[1])


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_rows_of_two_tiles_have_one_owner(dt, monkeypatch):
    """66 rows fetched in vectors along the rows: the last vector starts two (bf16: six) rows before the third tile of 32.  An
    infinity in row 65 has that tile summed again; the rows of the tile before keep the bits they have without it."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,contract_tile=2")
    m, n, k = 66, 40, 200
    bufs = [W.Buffer("A", "in", dt, (k, m)), W.Buffer("B", "in", dt, (k, n)), W.Buffer("C", "out", "f32", (m, n))]
    blk = W.flat_block(bufs, dict(m=m, n=n, k=k), [(["k", "m"], "assign"), (["k", "n"], "assign"), (["m", "n"], "add")],
                       constraints=[f"{k + n - 21} - n - k >= 0"])
    ins = [W.seeded_tensor((k, m), dt, 0), W.seeded_tensor((k, n), dt, 1)]
    clean, sb = run_gpu(blk, ins, return_block=True)
    assert sb.info["kernel"].startswith("contract_") and "_fetch2" in sb.info["kernel"], sb.info
    ins[0][3, 65] = math.inf
    for _ in range(3):
        got = run_gpu(blk, ins)
        assert np.isinf(got.reshape(m, n)[65]).all()
        assert np.array_equal(got.reshape(m, n)[:64].view(np.int32), clean.reshape(m, n)[:64].view(np.int32))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("Ci", [3, 8])
def test_infinities_on_the_tiled_literal_kernel(Ci, dt, monkeypatch):
    """The kernel that few output channels over a large image stay on skips removed points too: infinite filter taps at the
    image's border against the oracle."""
    monkeypatch.setenv("STRIPE_TUNE", "generic_tiled=2")
    blk = W.conv2d_block(1, 9, 8, Ci, 10, 3, 3, 1, 1, dt, "f32")
    ins = [W.seeded_tensor((1, 9, 8, Ci), dt, 0).abs() + 0.5, W.seeded_tensor((3, 3, 10, Ci), dt, 1)]
    ins[1][0, 1, 3, 2] = math.inf
    ins[1][2, 2, 7, 0] = math.nan
    got, sb = run_gpu(blk, ins, "generic", return_block=True)
    assert sb.info["kernel"].startswith("generic_tiled_4x4"), sb.info
    want = O.evaluate(blk, [W.to_numpy(t).ravel() for t in ins]).out
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want)) and np.isinf(want).any()
    fin = np.isfinite(want)
    assert np.allclose(got[fin], want[fin], rtol=1e-5, atol=1e-4)       # 72 products of order 1 in fp32


@pytest.mark.parametrize("tile", [0, 1, 2, 3])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["convolution", "transposed", "both operands"])
def test_non_finite_values_over_several_k_tiles(kind, dt, tile, monkeypatch):
    """Infinities of both signs and NaN in both operands, a reduction of several K tiles that ends inside a vector, more rows and
    columns than one part of a tile: the literal kernel's infinities, NaN and (to rounding) finite values."""
    if kind == "convolution":
        blk = W.conv2d_block(2, 13, 13, 13, 70, 5, 5, 1, 2, dt, "f32")
    elif kind == "transposed":
        bufs = [W.Buffer("I", "in", dt, (2, 9, 9, 36)), W.Buffer("F", "in", dt, (3, 3, 36, 20)), W.Buffer("O", "out", "f32", (2, 19, 19, 20))]
        blk = W.flat_block(bufs, dict(n=2, y=9, x=9, i=3, j=3, c=36, k=20),
                           [(["n", "y", "x", "c"], "assign"), (["i", "j", "c", "k"], "assign"), (["n", "2*y + i", "2*x + j", "k"], "add")])
    else:
        bufs = [W.Buffer("A", "in", dt, (70, 130)), W.Buffer("B", "in", dt, (68, 130)), W.Buffer("C", "out", "f32", (70, 68))]
        blk = W.flat_block(bufs, dict(m=70, n=68, k=130), [(["m", "k"], "assign"), (["n", "k"], "assign"), (["m", "n"], "add")],
                           constraints=["100 - k + m >= 0", "k + n - 20 >= 0"])
    ins = [W.seeded_tensor(r.sizes, dt, i) for i, r in enumerate(blk.refs[:2])]
    for i, t in enumerate(ins):
        flat = t.view(-1)
        for at, v in ((7, math.inf), (flat.numel() // 2, -math.inf), (flat.numel() // 2 + 3, math.inf), (flat.numel() - 2 - i, math.nan)):
            flat[at] = v
    monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,contract_tile={tile}")
    got, sb = run_gpu(blk, ins, return_block=True)
    assert sb.info["kernel"].startswith("contract_"), sb.info["kernel"]
    want = run_gpu(blk, ins, "generic")
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want))
    assert np.array_equal(np.isneginf(got), np.isneginf(want)) and np.isinf(want).any() and np.isnan(want).any()
    fin = np.isfinite(want)
    # sums of at most 325 products of order 1 in fp32: 325 * 2^-24 * sum |a b|
    assert fin.any() and np.allclose(got[fin], want[fin], rtol=1e-5, atol=325 * 2.0 ** -24 * 325)


def test_non_finite_values_do_not_stall(monkeypatch):
    """One infinity in the image costs no multiple of the literal kernel's time (point by point it was 23 times that)."""
    blk = W.conv2d_block(2, 8, 8, 256, 182, 5, 5, 1, 2, "f32", "f32")
    ins = [W.seeded_tensor(r.sizes, "f32", i).cuda() for i, r in enumerate(blk.refs[:2])]
    ins[0].view(-1)[12345] = math.inf
    out, took = torch.zeros(W.output_extent(blk), device="cuda"), {}
    for path in ("auto", "generic"):
        sb = B.StripeBlock(blk, path)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        sb.run(ins, out)
        ev[0].record()
        for _ in range(5):
            sb.run(ins, out)
        ev[1].record()
        torch.cuda.synchronize()
        took[path] = ev[0].elapsed_time(ev[1])
        kernel = sb.info["kernel"]
        assert kernel.startswith("contract_" if path == "auto" else "generic_"), kernel
        sb.close()
    assert took["auto"] < 3 * took["generic"], took


@pytest.mark.parametrize("in_dt,out_dt", [("bf16", "bf16"), ("bf16", "f32"), ("f32", "f32")])
@pytest.mark.parametrize("M,N,K", [(5, 33, 1024), (16, 16, 520), (17, 40, 512), (32, 130, 2064), (8, 1, 1040)])
def test_few_rows(M, N, K, in_dt, out_dt):
    """Both row counts of the kernel, columns beyond the tile, a reduction that ends inside a step; with bias + relu."""
    if K * (2 if in_dt == "bf16" else 4) < 1024:
        K *= 2
    prog = W.linear_bias_relu_program(M, N, K, out_dt, b_transposed=True) if in_dt == "bf16" else None
    blk = matmul(M, N, K, in_dt, "nt")
    ins = [W.seeded_tensor((M, K), in_dt, 0), W.seeded_tensor((N, K), in_dt, 1)]
    info, _ = parity(blk, ins, what="few rows")
    # one column: the index is gone from the block, which is a matrix-vector product and stays on the literal kernel
    assert info["kernel"].startswith("generic_affine_wave_per_output" if N == 1 else "gemm_rows_"), info
    if prog is not None:
        bias = W.seeded_tensor((N,), "f32", 2)
        got, sb = run_gpu(prog, ins + [bias], return_block=True)
        want = torch.relu(ins[0].double() @ ins[1].double().t() + bias.double()).numpy().ravel()
        # fp32 sums of K products, one rounding to bf16 on a bf16 store
        tol = K * 2.0 ** -24 * (ins[0].double().abs() @ ins[1].double().abs().t()).numpy().ravel() + 1e-5 + (2.0 ** -8 * want if out_dt == "bf16" else 0)
        assert np.all(np.abs(got - want) <= tol), sb.info["kernel"]
        assert N == 1 or sb.info["kernel"].endswith("+bias_relu"), sb.info


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("M,pieces", [(7, 64), (7, 129), (7, 257), (16, 1025), (20, 65), (17, 129), (32, 515)])
def test_few_rows_steps(M, pieces, dt, monkeypatch):
    """Reductions of 1 to 17 steps of 64 pieces of 16 bytes, whole and ending inside a step: each number of steps at once."""
    monkeypatch.setenv("STRIPE_TUNE", "gemm_rows=2")
    K = pieces * 16 // {"f32": 4, "bf16": 2, "i8": 1}[dt]
    blk = matmul(M, 37, K, dt, "nt")
    info, _ = parity(blk, [W.seeded_tensor((M, K), dt, 0), W.seeded_tensor((37, K), dt, 1)], what=f"{M} rows, {pieces} pieces")
    assert info["kernel"].startswith("gemm_rows_"), info


def test_few_rows_program_in_static_scratch():
    """Temporary and partial sums of this program are more than the static scratch: run_static takes the kernel that needs none."""
    M, N, K = 32, 1024, 32768
    prog = W.linear_bias_relu_program(M, N, K, "bf16", b_transposed=True)
    ins = [W.seeded_tensor((M, K), "bf16", 0), W.seeded_tensor((N, K), "bf16", 1) / 16, W.seeded_tensor((N,), "f32", 2)]
    sb = B.StripeBlock(prog)
    assert sb.info["workspace_bytes"] > 8 << 20 and "splitk" in sb.info["kernel"], sb.info
    dins = [t.cuda() for t in ins]
    want = torch.relu(ins[0].double() @ ins[1].double().t() + ins[2].double())
    tol = K * 2.0 ** -24 * (ins[0].double().abs() @ ins[1].double().abs().t()) + 2.0 ** -8 * want + 1e-5    # fp32 sums, one rounding to bf16
    for run in (sb.run_static, sb.run):
        out = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
        run(dins, out)
        assert ((out.cpu().double() - want).abs() <= tol).all()
    sb.close()


def error_against_64_bits(blk, ins, want, path="auto"):
    """2-norm of the difference over 2-norm of the result, and the kernel's name."""
    got, sb = run_gpu(blk, ins, path, return_block=True)
    return float(np.linalg.norm(got - want) / np.linalg.norm(want)), sb.info["kernel"]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", [(16, 1000, 576), (17, 300, 1040), (3, 500, 4000)])
def test_few_rows_error(M, N, K, dt):
    """The sums are no less exact than on the literal kernel, whose lanes hold 64 partial sums (both against 64 bits)."""
    blk = matmul(M, N, K, dt, "nt")
    ins = [W.seeded_tensor((M, K), dt, 0), W.seeded_tensor((N, K), dt, 1)]
    want = (ins[0].double() @ ins[1].double().t()).numpy().ravel()
    err, kernel = error_against_64_bits(blk, ins, want)
    before, _ = error_against_64_bits(blk, ins, want, "generic")
    assert kernel.startswith("gemm_rows_") and err <= before, (kernel, err, before)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", [(100, 100, 1001), (250, 250, 333), (13000, 5, 301), (40, 200, 4001)])
def test_products_error(M, N, K, dt, monkeypatch):
    """As test_few_rows_error, for the general contraction in place of the wavefront-per-output kernel."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1")
    blk = matmul(M, N, K, dt, "nt")
    ins = [W.seeded_tensor((M, K), dt, 0), W.seeded_tensor((N, K), dt, 1)]
    want = (ins[0].double() @ ins[1].double().t()).numpy().ravel()
    err, kernel = error_against_64_bits(blk, ins, want)
    before, literal = error_against_64_bits(blk, ins, want, "generic")
    assert kernel.startswith("contract_") and "wave_per_output" in literal and err <= before, (kernel, err, before)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_transposed_convolution_error(dt):
    """The same where the literal kernels add up an output's tuples with atomics (64 input channels, 8 x 13 x 13, 3x3, stride 2)."""
    N, H, C, R = 8, 13, 64, 3
    bufs = [W.Buffer("I", "in", dt, (N, H, H, C)), W.Buffer("F", "in", dt, (R, R, C, C)), W.Buffer("O", "out", "f32", (N, 2 * H + 1, 2 * H + 1, C))]
    blk = W.flat_block(bufs, dict(n=N, y=H, x=H, i=R, j=R, c=C, k=C),
                       [(["n", "y", "x", "c"], "assign"), (["i", "j", "c", "k"], "assign"), (["n", "2*y + i", "2*x + j", "k"], "add")])
    ins = [W.seeded_tensor((N, H, H, C), dt, 0), W.seeded_tensor((R, R, C, C), dt, 1)]
    want = np.zeros((N, 2 * H + 1, 2 * H + 1, C))
    for i in range(R):
        for j in range(R):
            want[:, i:i + 2 * H - 1:2, j:j + 2 * H - 1:2] += (ins[0].double().reshape(-1, C) @ ins[1][i, j].double()).reshape(N, H, H, C).numpy()
    err, kernel = error_against_64_bits(blk, ins, want.ravel())
    before, literal = error_against_64_bits(blk, ins, want.ravel(), "generic")
    assert kernel.startswith("contract_") and "atomic" in literal and err <= before, (kernel, err, before)


def test_few_rows_int8():
    blk = matmul(9, 50, 2048, "i8", "nt")
    info, _ = parity(blk, [W.seeded_tensor((9, 2048), "i8", 0), W.seeded_tensor((50, 2048), "i8", 1)], what="few rows int8")
    assert info["kernel"].startswith("gemm_rows_i8"), info


@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
def test_fused_bias_relu(out_dt):
    """The 3-channel convolution and its pointwise statement as one launch."""
    N, H, Ci, Co, R = 2, 30, 3, 20, 5
    prog = W.conv_bias_relu_program(N, H, H, Ci, Co, R, R, 2, 2, "bf16", out_dt)
    ins = [W.seeded_tensor((N, H, H, Ci), "bf16", 0), W.seeded_tensor((R, R, Co, Ci), "bf16", 1), W.seeded_tensor((Co,), "f32", 2)]
    got, sb = run_gpu(prog, ins, return_block=True)
    assert sb.info["kernel"].startswith("contract_") and "+bias_relu" in sb.info["kernel"] and sb.info["workspace_bytes"] == 0, sb.info
    res = O.evaluate_program(prog, [W.to_numpy(t).ravel() for t in ins], threads=8)
    tol = 75 * 2.0 ** -24 * 75 * float(ins[0].abs().max()) * float(ins[1].abs().max()) + (2.0 ** -8 * np.abs(res.out) if out_dt == "bf16" else 0)
    assert res.touched.all() and np.all(np.abs(got - res.out) <= tol)


def unaligned(t, off):
    """A copy of t on the GPU, `off` elements behind a 256-byte boundary."""
    big = torch.empty(t.numel() + off, dtype=t.dtype, device="cuda")
    big[off:] = t.reshape(-1).cuda()
    return big[off:]


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("kind", ["product", "rows", "convolution"])
def test_unaligned_pointers_on_a_side_stream(kind, dt, monkeypatch):
    """Inputs and output one and three elements behind an aligned address, on another stream than the default one."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,gemm_dma=0")
    if kind == "convolution":
        blk = W.conv2d_block(2, 11, 11, 8, 12, 3, 3, 1, 1, dt, "i32" if dt == "i8" else "f32")
        monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,conv_igemm=0,conv_gemm=0,conv_mfma=0,conv_tuned=0")
    else:
        blk = matmul(9 if kind == "rows" else 70, 44, 1040, dt, "nt")
    ins = [W.seeded_tensor(r.sizes, dt, i) for i, r in enumerate(blk.refs[:2])]
    want = run_gpu(blk, ins, "generic")
    sb = B.StripeBlock(blk)
    assert sb.info["path_name"] == "generic" and sb.info["kernel"].startswith("gemm_rows_" if kind == "rows" else "contract_"), sb.info
    held = [unaligned(t, 1 + 2 * i) for i, t in enumerate(ins)]
    out = torch.zeros(want.size + 3, dtype=torch.int32 if dt == "i8" else torch.float32, device="cuda")[3:]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sb.run(held, out)
    side.synchronize()
    got = out.cpu().numpy()
    sb.close()
    if dt == "i8":
        assert np.array_equal(got, want)
    else:       # two fp32 sums of the same products
        K = 72 if kind == "convolution" else 1040
        bound = 2 * K * 2.0 ** -24 * K * float(ins[0].float().abs().max()) * float(ins[1].float().abs().max())
        assert np.abs(got - want).max() <= bound


@pytest.mark.parametrize("kind", ["product", "rows", "convolution"])
def test_captured_runs(kind, monkeypatch):
    """Recorded in a graph and replayed with other inputs and eager work between the replays."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,gemm_dma=0")
    if kind == "convolution":
        blk = W.conv_bias_relu_program(2, 14, 14, 3, 12, 3, 3, 1, 1, "bf16", "bf16")
    else:
        blk = W.linear_bias_relu_program(9 if kind == "rows" else 70, 44, 1040, "bf16", b_transposed=True)
    dts = [r.dtype for r in blk.refs if r.dir == "in"]
    shapes = [r.sizes for r in blk.refs if r.dir == "in"]
    ins = [W.seeded_tensor(s, d, i).cuda() for i, (s, d) in enumerate(zip(shapes, dts))]
    sb = B.StripeBlock(blk)
    assert sb.info["workspace_bytes"] == 0 and "+bias_relu" in sb.info["kernel"], sb.info
    out, eager = (torch.zeros(blk.refs[-1].sizes, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    sb.run(ins, eager)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sb.run(ins, out)
    for seed in range(3):
        ins[0].copy_(W.seeded_tensor(shapes[0], dts[0], 50 + seed))
        sb.run(ins, eager)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager) and out.any()
    sb.close()


@pytest.mark.parametrize("fused", [False, True])
def test_first_run_of_a_split_product_under_capture(fused):
    """Few rows, few columns and a long reduction run as a split product with a workspace; a first run that is being captured,
    where nothing can be allocated, is recorded on the kernel that needs none."""
    M, N, K = 8, 256, 16384
    blk = W.linear_bias_relu_program(M, N, K, "f32", b_transposed=True) if fused else matmul(M, N, K, "bf16", "nt")
    ins = [W.seeded_tensor((M, K), "bf16", 0), W.seeded_tensor((N, K), "bf16", 1)] + ([W.seeded_tensor((N,), "f32", 2)] if fused else [])
    want = ins[0].double() @ ins[1].double().t()
    if fused:
        want = torch.relu(want + ins[2].double())
    tol = K * 2.0 ** -24 * (ins[0].double().abs() @ ins[1].double().abs().t()) + 1e-5
    sb = B.StripeBlock(blk)
    assert sb.info["workspace_bytes"] > 0 and "splitk" in sb.info["kernel"], sb.info
    dins = [t.cuda() for t in ins]
    out = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sb.run(dins, out)
    eager = torch.zeros_like(out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert ((out.cpu().double() - want).abs() <= tol).all()
        sb.run(dins, eager)          # allocates now, and runs split
        torch.cuda.synchronize()
        assert ((eager.cpu().double() - want).abs() <= tol).all()
    sb.close()


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("layout", ["nn", "nt", "tn"])
@pytest.mark.parametrize("M,N,K,tile", [(1, 17, 33, 4), (1, 130, 700, 5), (15, 17, 31, 4), (16, 16, 64, 4), (19, 33, 4100, 4), (64, 64, 64, 5),
                                        (63, 65, 33, 5), (66, 130, 1025, 5), (9, 300, 2100, 2)])
def test_products_whose_reduction_wavefronts_share(M, N, K, tile, layout, dt, monkeypatch):
    """The tiles on which wavefronts share the reduction out: fewer K tiles than wavefronts, a last pass that only some have, partial
    vectors, one row, rows and columns beside the tile."""
    monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,contract_tile={tile},gemm_rows=0,gemm_dma=0")
    blk = matmul(M, N, K, dt, layout)
    ins = [W.seeded_tensor(blk.refs[0].sizes, dt, 0), W.seeded_tensor(blk.refs[1].sizes, dt, 1)]
    info, _ = parity(blk, ins, what=f"{layout} {M}x{N}x{K} {dt}")
    # one row of few columns whose operand cannot be fetched in vectors: no plain product, which the 64 x 64 form is for
    assert info["kernel"].startswith(f"contract_{dt}_{ {2: '32x32', 4: '16x16', 5: '64x64'}[tile] }x"), info["kernel"]


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("shape", [(2, 19, 13, 3, 20, 5, 2, 2), (1, 9, 11, 8, 70, 3, 1, 1), (1, 7, 7, 72, 17, 7, 1, 3), (1, 6, 7, 9, 12, 3, 1, 1)])
def test_convolutions_on_the_smallest_tile(shape, dt, monkeypatch):
    """Constraints and several reduction indexes on the 16 x 16 tile: tables of more and of fewer K tiles than a wavefront has."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,contract_tile=4,conv_igemm=0")
    N, H, Wd, Ci, Co, R, s, p = shape
    blk = W.conv2d_block(N, H, Wd, Ci, Co, R, R, s, p, dt, "i32" if dt == "i8" else "f32")
    info, _ = parity(blk, [W.seeded_tensor((N, H, Wd, Ci), dt, 0), W.seeded_tensor((R, R, Co, Ci), dt, 1)], what=f"conv {shape} {dt}")
    assert info["kernel"].startswith(f"contract_{dt}_16x16x"), info


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_non_finite_values_on_the_smallest_tile(dt, monkeypatch):
    """A removed point contributes nothing there either: the literal kernel's infinities, NaN and finite values."""
    blk = W.conv2d_block(1, 9, 9, 13, 20, 5, 5, 1, 2, dt, "f32")
    ins = [W.seeded_tensor(r.sizes, dt, i) for i, r in enumerate(blk.refs[:2])]
    for i, t in enumerate(ins):
        flat = t.view(-1)
        for at, v in ((7, math.inf), (flat.numel() // 2, -math.inf), (flat.numel() - 2 - i, math.nan)):
            flat[at] = v
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,contract_tile=4")
    got, sb = run_gpu(blk, ins, return_block=True)
    assert sb.info["kernel"].startswith(f"contract_{dt}_16x16x"), sb.info["kernel"]
    want = run_gpu(blk, ins, "generic")
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want))
    assert np.array_equal(np.isneginf(got), np.isneginf(want)) and np.isinf(want).any() and np.isnan(want).any()
    fin = np.isfinite(want)
    assert fin.any() and np.allclose(got[fin], want[fin], rtol=1e-5, atol=325 * 2.0 ** -24 * 325)     # 325 products of order 1 in fp32


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("layout,M,N,K", [("nn", 1, 349, 1000), ("tn", 1, 128, 960), ("nn", 5, 19, 184), ("tn", 3, 64, 240), ("nt", 33, 56, 26)])
def test_small_products(layout, M, N, K, dt):
    """A row vector times a matrix and products of a few thousand points, chosen without any setting."""
    blk = matmul(M, N, K, dt, layout)
    ins = [W.seeded_tensor(blk.refs[0].sizes, dt, 0), W.seeded_tensor(blk.refs[1].sizes, dt, 1)]
    info, _ = parity(blk, ins, what=f"{layout} {M}x{N}x{K} {dt}")
    assert info["kernel"].startswith("contract_"), info["kernel"]


@pytest.mark.parametrize("kind", ["product", "convolution"])
def test_family_blocks_on_the_contraction_keep_their_pointer_contract(kind):
    """Few tiles and a long reduction: a product and a convolution of the matrix-core families run here, stay blocks of their family, and
    refuse unaligned pointers as before; fused with bias + relu too."""
    if kind == "product":
        blk, prog = W.matmul_block(15, 64, 2432, "bf16", "f32"), None
    else:
        blk, prog = W.conv2d_block(3, 13, 13, 256, 64, 5, 5, 1, 2, "bf16", "f32"), W.conv_bias_relu_program(1, 13, 13, 256, 64, 5, 5, 1, 2, "bf16", "f32")
    ins = [W.seeded_tensor(r.sizes, "bf16", i) for i, r in enumerate(blk.refs[:2])]
    info, _ = parity(blk, ins, what=kind)
    assert info["kernel"].startswith("contract_") and info["path_name"] == ("mfma_gemm" if kind == "product" else "mfma_conv"), info
    sb = B.StripeBlock(blk)
    out = torch.zeros(W.output_extent(blk), device="cuda")
    with pytest.raises(B.StripeError) as e:
        sb.run([unaligned(ins[0], 1), ins[1].cuda()], out)
    assert e.value.status == 8, str(e.value)
    sb.close()
    if prog is not None:
        sb = B.StripeBlock(prog)
        assert sb.info["kernel"].startswith("contract_") and sb.info["kernel"].endswith("+bias_relu") and sb.info["workspace_bytes"] == 0, sb.info
        held = [W.seeded_tensor(r.sizes, r.dtype, i).cuda() for i, r in enumerate(r for r in prog.refs if r.dir == "in")]
        out = torch.zeros((1, 13, 13, 64), device="cuda")
        with pytest.raises(B.StripeError) as e:
            sb.run([held[0], held[1], unaligned(held[2].cpu(), 1)], out)
        assert e.value.status == 8, str(e.value)
        sb.run(held, out)
        sb.close()
        x, f, b = (t.double().cpu() for t in held)
        want = torch.relu(torch.nn.functional.conv2d(x.permute(0, 3, 1, 2), f.permute(2, 3, 0, 1), padding=2) + b[:, None, None]).permute(0, 2, 3, 1)
        err = (out.double().cpu() - want).abs().max()
        assert err <= 6400 * 2.0 ** -24 * float((x.abs().max() * f.abs().max() * 6400).clamp(min=1)), float(err)     # 6400 fp32 additions


@pytest.mark.parametrize("M,N,K,dt,layout", [(130, 136, 128, "bf16", "nn"), (127, 264, 384, "bf16", "nn"), (129, 333, 256, "bf16", "nt"), (33, 9, 128, "bf16", "nt"),
                                             (300, 257, 1024, "i8", "nt"), (33, 8, 256, "i8", "nt"), (1000, 520, 256, "i8", "nt")])
@pytest.mark.parametrize("kb", [64, 128])
def test_ragged_products_on_the_128_wide_tiles(M, N, K, dt, layout, kb, monkeypatch):
    """Rows and columns beside the tile: nothing of them is read past the operand or stored, position-sensitive operands exactly."""
    monkeypatch.setenv("STRIPE_TUNE", f"gemm_t128_ragged=1,gemm_t128_kb={kb},gemm_rows=0,gemm_splitk=0")
    blk = matmul(M, N, K, dt, layout)
    a = ((torch.arange(M)[:, None] * 7 + torch.arange(K)[None, :] * 3) % 251 - 125).to(torch.int8 if dt == "i8" else torch.bfloat16)
    sel = (torch.arange(N) + 37) % K
    b = torch.zeros((K, N), dtype=a.dtype)
    b[sel, torch.arange(N)] = 1
    gpu, sb = run_gpu(blk, [a, b.t().contiguous() if layout == "nt" else b], return_block=True)
    assert "_128x128x" in sb.info["kernel"] and sb.info["kernel"].endswith("_ragged"), sb.info["kernel"]
    assert np.array_equal(gpu.reshape(M, N), a.float()[:, sel].numpy())
    ins = [W.seeded_tensor(blk.refs[0].sizes, dt, 0), W.seeded_tensor(blk.refs[1].sizes, dt, 1)]
    parity(blk, ins, what=f"ragged {M}x{N}x{K} {dt}")


def test_ragged_fused_product_on_the_128_wide_tiles(monkeypatch):
    monkeypatch.setenv("STRIPE_TUNE", "gemm_t128_ragged=1,gemm_rows=0,gemm_splitk=0")
    for M, N, out_dt in ((130, 333, "bf16"), (70, 129, "f32")):
        prog = W.linear_bias_relu_program(M, N, 256, out_dt, b_transposed=True)
        sb = B.StripeBlock(prog)
        assert "_128x128x" in sb.info["kernel"] and "_ragged+bias_relu" in sb.info["kernel"], sb.info["kernel"]
        held = [W.seeded_tensor(r.sizes, r.dtype, i).cuda() for i, r in enumerate(r for r in prog.refs if r.dir == "in")]
        out = torch.full((M, N), -7.0, dtype=torch.bfloat16 if out_dt == "bf16" else torch.float32, device="cuda")
        sb.run(held, out)
        sb.close()
        x, w, b = (t.double().cpu() for t in held)
        want = torch.relu(x @ w.t() + b)
        # 256 products of order up to |x||w| in fp32, then half a step of the output type
        tol = 256 * 2.0 ** -24 * (x.abs() @ w.abs().t() + b.abs()) + (2.0 ** -8 * want if out_dt == "bf16" else 0)
        assert bool(((out.double().cpu() - want).abs() <= tol).all())


@pytest.mark.parametrize("M,N,K", [(12, 323, 8192), (20, 1000, 8192), (2, 16, 8192)])
def test_few_rows_with_an_fp32_output(M, N, K):
    """relu(X W^T + b) in fp32 where the general contraction replaces the few-rows kernel: totals in double precision, so what is left is
    chains of at most 32 products and one rounding of the total."""
    prog = W.linear_bias_relu_program(M, N, K, "f32")
    sb = B.StripeBlock(prog)
    held = [W.seeded_tensor(r.sizes, r.dtype, i).cuda() for i, r in enumerate(r for r in prog.refs if r.dir == "in")]
    out = torch.full((M, N), -7.0, device="cuda")
    sb.run(held, out)
    sb.close()
    x, w, b = (t.double().cpu() for t in held)
    want = torch.relu(x @ w.t() + b)
    tol = 64 * 2.0 ** -24 * (x.abs() @ w.abs().t()) + 2.0 ** -23 * (want.abs() + b.abs())
    assert bool(((out.double().cpu() - want).abs() <= tol).all())


@pytest.mark.parametrize("M,N,K,layout,most", [(401, 320, 2560, "nn", 1.15e-7), (537, 264, 2560, "nt", 1.15e-7), (1905, 640, 3072, "nn", 1.8e-7)])
def test_ragged_products_sum_in_short_chains(M, N, K, layout, most):
    """128-wide tiles need fewer slices of the reduction than 256-wide ones, which must not lengthen the chains of roundings: 256, 256 and
    768 products from zero (1.0e-7, 1.0e-7 and 1.6e-7 off in the 2-norm; in one chain per slice 1.3e-7, 1.3e-7 and 3.4e-7)."""
    g = torch.Generator().manual_seed(7)
    a, b = (torch.randn(s, generator=g).to(torch.bfloat16).cuda() for s in ((M, K), (N, K) if layout == "nt" else (K, N)))
    sb = B.StripeBlock(W.matmul_block(M, N, K, "bf16", "f32", b_transposed=layout == "nt"))
    assert "128x128" in sb.info["kernel"] and "_ragged" in sb.info["kernel"], sb.info["kernel"]
    out = torch.zeros((M, N), device="cuda")
    sb.run([a, b], out)
    sb.close()
    want = a.double() @ (b.double().t() if layout == "nt" else b.double()).contiguous()
    err = float((out.double() - want).norm() / want.norm())
    assert err <= most, err


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("M,N,K,tile,lanes", [(129, 2100, 289, 5, 512), (70, 4100, 1025, 5, 512), (63, 65, 33, 5, 512), (9, 300, 2100, 2, 512), (19, 33, 4100, 4, 1024)])
def test_long_products_whose_reduction_wavefronts_share(M, N, K, tile, lanes, dt, monkeypatch):
    """Both operands k-contiguous, K tiles beyond one per wavefront and a partial last one, on the kernel whose wavefronts stage for
    themselves (its workgroup tells it from the one whose four wavefronts share a K tile)."""
    monkeypatch.setenv("STRIPE_TUNE", f"contract_min=1,contract_tile={tile},gemm_rows=0,gemm_dma=0")
    blk = matmul(M, N, K, dt, "nt")
    info, _ = parity(blk, [W.seeded_tensor((M, K), dt, 0), W.seeded_tensor((N, K), dt, 1)], what=f"{M}x{N}x{K} {dt}", threads=8)
    assert info["kernel"].startswith(f"contract_{dt}_") and info["workgroup_size"] == lanes, info


@pytest.mark.parametrize("layout,M,N,K,dt,most", [("nt", 200, 300, 16, "f32", 6.7e-8), ("nn", 500, 200, 12, "f32", 5.9e-8), ("tn", 300, 700, 9, "f32", 5.3e-8)])
def test_short_fp32_reductions_are_two_chains(layout, M, N, K, dt, most):
    """9 to 16 fp32 products in one chain are 7.3e-8, 6.4e-8 and 5.6e-8 off in the 2-norm at these sizes, as two chains of eight
    6.0e-8, 5.4e-8 and 5.0e-8."""
    error_at_most(layout, M, N, K, dt, most)


def error_at_most(layout, M, N, K, dt, most):
    g = torch.Generator().manual_seed(5)
    a, b = (torch.randn(n, generator=g).to(torch.bfloat16 if dt == "bf16" else torch.float32) for n in ((M, K), (K, N)))
    ins = [a.t().contiguous() if layout == "tn" else a, b.t().contiguous() if layout == "nt" else b]
    got, sb = run_gpu(matmul(M, N, K, dt, layout), ins, return_block=True)
    assert sb.info["kernel"].startswith("contract_"), sb.info["kernel"]
    sb.close()
    want = (a.double() @ b.double()).numpy()
    err = np.linalg.norm(got.reshape(want.shape) - want) / np.linalg.norm(want)
    assert err <= most, (err, most)


# ------------------------------------------------------------------ 32 x 32 tiles whose K tile four wavefronts share (tile 6)
@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("kind", ["nn", "nt", "tn", "conv3", "conv5", "upconv", "upconv2"])
def test_tiles_whose_k_tile_wavefronts_share(kind, dt, monkeypatch):
    """Every way to fetch, one and several K tiles with remainders, tables of a batch and of one K tile, constraints."""
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,contract_tile=6,gemm_rows=0,gemm_dma=0,conv_igemm=0")
    if kind in ("nn", "nt", "tn"):
        for M, N, K in ((33, 68, 129), (1, 17, 300), (70, 40, 1037)):
            blk = matmul(M, N, K, dt, kind)
            info, _ = parity(blk, [W.seeded_tensor(r.sizes, dt, i) for i, r in enumerate(blk.refs[:2])], what=f"{kind} {M}x{N}x{K} {dt}")
            assert info["kernel"].startswith(f"contract_{dt}_32x32x") and info["workgroup_size"] == 256, info
        return
    if kind.startswith("conv"):
        N, H, Wd, Ci, Co, R, s, p = (1, 9, 11, 8, 70, 3, 1, 1) if kind == "conv3" else (2, 13, 12, 11, 37, 5, 2, 2)
        blk = W.conv2d_block(N, H, Wd, Ci, Co, R, R, s, p, dt, "i32" if dt == "i8" else "f32")
    else:
        R, Ci, Co, H = (3, 36, 20, 9) if kind == "upconv" else (2, 19, 33, 7)
        Ho = 2 * (H - 1) + R
        bufs = [W.Buffer("I", "in", dt, (2, H, H, Ci)), W.Buffer("F", "in", dt, (R, R, Ci, Co)), W.Buffer("O", "out", "i32" if dt == "i8" else "f32", (2, Ho, Ho, Co))]
        blk = W.flat_block(bufs, dict(n=2, y=H, x=H, i=R, j=R, c=Ci, k=Co),
                           [(["n", "y", "x", "c"], "assign"), (["i", "j", "c", "k"], "assign"), (["n", "2*y + i", "2*x + j", "k"], "add")])
    info, _ = parity(blk, [W.seeded_tensor(r.sizes, dt, i) for i, r in enumerate(blk.refs[:2])], what=f"{kind} {dt}")
    assert info["kernel"].startswith(f"contract_{dt}_32x32x") and info["workgroup_size"] == 256, info


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("Ci,Co", [(13, 20), (8, 40)])
def test_non_finite_values_where_wavefronts_share_a_k_tile(Ci, Co, dt, monkeypatch):
    """A removed point contributes nothing there either: the literal kernel's infinities, NaN and finite values."""
    blk = W.conv2d_block(1, 9, 9, Ci, Co, 5, 5, 1, 2, dt, "f32")
    ins = [W.seeded_tensor(r.sizes, dt, i) for i, r in enumerate(blk.refs[:2])]
    for i, t in enumerate(ins):
        flat = t.view(-1)
        for at, v in ((7, math.inf), (flat.numel() // 2, -math.inf), (flat.numel() - 2 - i, math.nan)):
            flat[at] = v
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,contract_tile=6")
    got, sb = run_gpu(blk, ins, return_block=True)
    assert sb.info["kernel"].startswith(f"contract_{dt}_32x32x") and sb.info["workgroup_size"] == 256, sb.info
    want = run_gpu(blk, ins, "generic")
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want))
    assert np.array_equal(np.isneginf(got), np.isneginf(want)) and np.isinf(want).any() and np.isnan(want).any()
    fin = np.isfinite(want)
    assert fin.any() and np.allclose(got[fin], want[fin], rtol=1e-5, atol=325 * 2.0 ** -24 * 325)     # 325 products of order 1 in fp32


@pytest.mark.parametrize("seed", range(0, 64, 3))
def test_random_blocks_where_wavefronts_share_a_k_tile(seed, monkeypatch):
    monkeypatch.setenv("STRIPE_TUNE", "contract_min=1,contract_tile=6")
    blk = random_block(seed)
    nrng = np.random.default_rng(seed)
    ins = [torch.from_numpy(nrng.integers(-3, 4, size=int(np.prod(r.sizes)), dtype=np.int8)) for r in blk.refs[:-1]]
    try:
        gpu, sb = run_gpu(blk, ins, return_block=True)
    except B.StripeError as e:
        assert e.status == 5, str(e)
        pytest.skip(f"rejected at create: {e}")
    res = O.evaluate(blk, [W.to_numpy(t) for t in ins], out=np.full(W.output_extent(blk), SENTINEL_I, np.int64))
    assert np.array_equal(gpu.astype(np.int64), res.out), sb.info["kernel"]


@pytest.mark.parametrize("layout,M,N,K,most", [("nn", 49, 2304, 64, 4.0e-8), ("tn", 164, 856, 64, 4.05e-8), ("nn", 381, 960, 64, 4.05e-8), ("tn", 14, 384, 384, 6.7e-8)])
def test_bf16_sums_of_a_k_tile_are_short(layout, M, N, K, most):
    """64 products in one chain are 4.2e-8 off in the 2-norm, 128 at a time 7.0e-8 at K = 384; as sums of 32 that meet in pairs
    3.85e-8 and below 6.5e-8."""
    error_at_most(layout, M, N, K, "bf16", most)
