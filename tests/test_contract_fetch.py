"""The general contraction's memory accesses, followed on the CPU: the planned launch parameters are read back and every
address the kernel forms for a load that its own range tests let through is compared with the operand's declared buffer.
A constraint is tested for one operand only, so the other one meets removed points, where its address may lie anywhere."""
import ctypes as C
import random

import numpy as np
import pytest

from paper_1903_06498_amd import binding as B
from paper_1903_06498_amd import workloads as W
from tests import brute

IDX, TESTS = 4, 2
i4, t24 = C.c_int32 * IDX, (C.c_int32 * IDX) * TESTS


class CtIndex(C.Structure):
    _fields_ = [("n", C.c_int32), ("range", C.c_uint32 * IDX), ("mul", C.c_uint32 * IDX), ("shift", i4)]


class Params(C.Structure):
    _fields_ = ([(x, CtIndex) for x in ("m", "n", "k")] + [(x, i4) for x in ("m_in", "m_out", "n_in", "n_out", "k_a", "k_b")]
                + [(x, t24) for x in ("m_t", "ka_t", "n_t", "kb_t")] + [(x, C.c_int32 * TESTS) for x in ("c_a", "c_b")]
                + [(x, C.c_uint32 * TESTS) for x in ("top_a", "top_b")] + [(x, t24) for x in ("m_ob", "n_ob")] + [("ob", C.c_int32 * TESTS)]
                + [(x, C.c_int32) for x in ("n_ob_used", "tested")] + [(x, C.c_uint32) for x in "MNK"]
                + [(x, C.c_int32) for x in ("a_base", "b_base", "o_base", "mode_a", "mode_b", "k_run")]
                + [(x, C.c_uint32) for x in ("bytes_a", "bytes_b")] + [("vec_out", C.c_int32), ("batch_range", C.c_uint32 * 2)]
                + [(x, C.c_int32 * 2) for x in ("batch_a", "batch_b", "batch_o")] + [("tiles_n", C.c_int32), ("epilogue", C.c_int32)])


def planned(blk, monkeypatch, tune="contract_min=1"):
    """The launch parameters (None where another kernel runs the block) and the kernel's name."""
    monkeypatch.setenv("STRIPE_TUNE", tune)
    try:
        sb = B.StripeBlock(blk)
    except B.StripeError as e:
        assert e.status == 5, str(e)
        return None, "rejected"
    fn = B.lib.stripe_test_contract_params
    fn.restype, fn.argtypes = C.c_size_t, [C.c_void_p, C.c_void_p, C.c_size_t]
    p = Params()
    size = fn(sb.handle, C.byref(p), C.sizeof(p))
    name = sb.info["kernel"]
    sb.close()
    if size == 0:
        return None, name
    assert size == C.sizeof(p), "ContractParams and its mirror here differ"
    return p, name


def declared_bytes(ref):
    return (sum((n - 1) * s for n, s in zip(ref.sizes, ref.strides)) + 1) * {"f32": 4, "bf16": 2, "i8": 1}[ref.dtype]


def parts(ix, total, rows):
    """[index][position] -> value, as the kernel divides a flat position up."""
    v, out = np.asarray(rows, np.int64), []
    for j in range(IDX):
        r = max(int(ix.range[j]), 1) if j < ix.n else 1
        out.append(v % r if j < ix.n else np.zeros_like(v))
        v = v // r
    return out


def check_side(p, esize, side_a, extent):
    """Every load of one operand that its tests let through lies inside its buffer."""
    mode = p.mode_a if side_a else p.mode_b
    rix, total = (p.m, p.M) if side_a else (p.n, p.N)
    rin, rt = (p.m_in, p.m_t) if side_a else (p.n_in, p.n_t)
    ka, kt = (p.k_a, p.ka_t) if side_a else (p.k_b, p.kb_t)
    base, c, top = (p.a_base, p.c_a, p.top_a) if side_a else (p.b_base, p.c_b, p.top_b)
    step = (8 if esize < 4 else 4) if mode == 2 else 1      # rows of one vector
    rows = np.arange(0, total, step)
    if mode == 2:
        rows = np.where(rows + step > total, total - step, rows)
    rv = parts(rix, total, rows)
    ve = {0: 1, 1: 16 // esize, 2: 1, 3: 8 // esize}[mode]
    ks = np.arange(0, p.K, ve)
    kv = parts(p.k, p.K, ks)
    koff = sum(int(ka[j]) * kv[j] for j in range(IDX))
    if mode == 1:
        koff = koff - np.maximum(ks + ve - p.K, 0)
    lost = kv[0] >= p.k_run
    bt = [(int(p.batch_a[j] if side_a else p.batch_b[j]), int(p.batch_range[j])) for j in range(2)]
    size = {0: esize, 1: 16, 2: step * esize, 3: 8}[mode]
    for b0 in range(bt[0][1]):
        for b1 in range(bt[1][1]):
            roff = base + bt[0][0] * b0 + bt[1][0] * b1 + sum(int(rin[j]) * rv[j] for j in range(IDX))
            off = (roff[:, None] + koff[None, :]) * esize
            ok = np.broadcast_to(~lost[None, :], off.shape).copy()
            for t in range(TESTS):
                f = int(c[t]) + sum(int(rt[t][j]) * rv[j] for j in range(IDX))[:, None] + sum(int(kt[t][j]) * kv[j] for j in range(IDX))[None, :]
                ok &= (f >= 0) & (f <= int(top[t]))
            off = off[ok]
            if mode == 3:       # a vector that would end behind the operand is fetched from its last 8 bytes
                off = np.where((off < 0) | (off > extent - 8), extent - 8, off)
            reach = (off >= 0) & (off + size <= extent)
            if mode == 0:       # one element: inside the buffer's range, or outside of it and zero
                reach |= (off >= extent) | (off < 0)
            assert reach.all(), (("A" if side_a else "B"), mode, int(off.min()), int(off.max()) + size, extent)


def check(blk, p):
    esize = {"f32": 4, "bf16": 2, "i8": 1}[blk.refs[0].dtype]
    ext = [declared_bytes(r) for r in blk.refs[:2]]
    # which operand plays A: the buffers' own bounds hold in one of the two assignments
    assert any(p.bytes_a <= ext[s] and p.bytes_b <= ext[1 - s] for s in (0, 1)), (p.bytes_a, p.bytes_b, ext)
    check_side(p, esize, True, p.bytes_a)
    check_side(p, esize, False, p.bytes_b)


def blocked_reduction(dt, m=40):
    """C[m,n] += A[m, i + 6j] * B[i + 6j, n], the last block of k cut off by a constraint; B ends with the polyhedron."""
    bufs = [W.Buffer("A", "in", dt, (m, 120)), W.Buffer("B", "in", dt, (100, 64)), W.Buffer("C", "out", "i32" if dt == "i8" else "f32", (m, 64))]
    return W.flat_block(bufs, dict(m=m, n=64, i=48, j=12), [(["m", "i + 6*j"], "assign"), (["i + 6*j", "n"], "assign"), (["m", "n"], "add")],
                        constraints=["99 - i - 6*j >= 0"])


def triangle(dt, n=96):
    """A[k][m] and B[k][n] of n rows, k below 2n with n - 1 - column - k >= 0: the test is B's, A's rows end at n."""
    bufs = [W.Buffer("A", "in", dt, (n, n)), W.Buffer("B", "in", dt, (2 * n, n)), W.Buffer("C", "out", "i32" if dt == "i8" else "f32", (n, n))]
    return W.flat_block(bufs, dict(m=n, n=n, k=2 * n), [(["k", "m"], "assign"), (["k", "n"], "assign"), (["m", "n"], "add")],
                        constraints=[f"{n - 1} - n - k >= 0"])


def joined_reduction(dt, m=40):
    """C[m,n] += A[m,p,q] * B[p+q, n] with 63 - p - q >= 0: A is dense in p and q, B ends at p + q = 63."""
    bufs = [W.Buffer("A", "in", dt, (m, 64, 64)), W.Buffer("B", "in", dt, (64, 72)), W.Buffer("C", "out", "i32" if dt == "i8" else "f32", (m, 72))]
    return W.flat_block(bufs, dict(m=m, n=72, p=64, q=64), [(["m", "p", "q"], "assign"), (["p + q", "n"], "assign"), (["m", "n"], "add")],
                        constraints=["63 - p - q >= 0"])


def blocked_operand(dt, m=40):
    """A stored in blocks of 16 of k, [7][m][16], against B[100, n]; 99 - 16 o - i >= 0."""
    bufs = [W.Buffer("A", "in", dt, (7, m, 16)), W.Buffer("B", "in", dt, (100, 72)), W.Buffer("C", "out", "i32" if dt == "i8" else "f32", (m, 72))]
    return W.flat_block(bufs, dict(m=m, n=72, o=7, i=16), [(["o", "m", "i"], "assign"), (["16*o + i", "n"], "assign"), (["m", "n"], "add")],
                        constraints=["99 - 16*o - i >= 0"])


PARTNERS = [blocked_reduction, triangle, joined_reduction, blocked_operand]


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("make", PARTNERS)
def test_partner_operand_ends_with_the_polyhedron(make, dt, monkeypatch):
    blk = make(dt)
    p, name = planned(blk, monkeypatch)
    assert name.startswith("contract_"), name
    check(blk, p)


@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
def test_convolutions_keep_their_vectors(dt, monkeypatch):
    """The halo's tests are the input's own: both operands are fetched in vectors, inside their buffers."""
    for (H, ci, co, R, s, pad) in [(14, 16, 24, 3, 1, 1), (15, 3, 20, 5, 2, 2), (9, 24, 33, 3, 2, 1)]:
        blk = W.conv2d_block(2, H, H, ci, co, R, R, s, pad, dt, "i32" if dt == "i8" else "f32")
        p, name = planned(blk, monkeypatch, "contract_min=1,conv_igemm=0,conv_gemm=0,conv_mfma=0,conv_tuned=0")
        if p is not None:
            assert p.mode_a and p.mode_b, name
            check(blk, p)


@pytest.mark.parametrize("R,s", [(3, 2), (5, 3), (3, 1), (4, 2)])
@pytest.mark.parametrize("dt", ["f32", "bf16", "i8"])
def test_transposed_convolutions(R, s, dt, monkeypatch):
    N, H, Ci, Co = 2, 7, 8, 6
    bufs = [W.Buffer("I", "in", dt, (N, H, H, Ci)), W.Buffer("F", "in", dt, (R, R, Ci, Co)),
            W.Buffer("O", "out", "i32" if dt == "i8" else "f32", (N, s * (H - 1) + R, s * (H - 1) + R, Co))]
    blk = W.flat_block(bufs, dict(n=N, y=H, x=H, i=R, j=R, c=Ci, k=Co),
                       [(["n", "y", "x", "c"], "assign"), (["i", "j", "c", "k"], "assign"), (["n", f"{s}*y + i", f"{s}*x + j", "k"], "add")])
    p, name = planned(blk, monkeypatch)
    assert name.startswith("contract_"), name
    check(blk, p)


def test_random_blocks(monkeypatch):
    """Buffers sized by the executed points, so every address behind a constraint is one the operand does not hold."""
    taken = 0
    for seed in range(600):
        rng = random.Random(40000 + seed)
        dt = ["i8", "bf16", "f32"][seed % 3]
        blk = brute.random_block(rng, seed % 4 == 2, dt, "i32" if dt == "i8" else "f32", "add", "mul", injective_out=True,
                                 max_range=9, contraction_roles=True, root_origin=3 if seed % 5 == 0 else 0)
        p, name = planned(blk, monkeypatch)
        if p is None:
            continue
        taken += 1
        check(blk, p)
    assert taken >= 100, taken
