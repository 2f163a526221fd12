"""Host-side checks of the HIP library that need no GPU: it loads, exports every
symbol include/stripe.h declares, and its planner (flatten, bounds proof,
canonical form, kernel-family choice) behaves as documented.  No kernel runs."""
import ctypes
import os
import re

import pytest

from paper_1903_06498_amd import binding as B
from paper_1903_06498_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "stripe.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(stripe_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = declared_functions()
    assert "stripe_block_create" in names and "stripe_block_run" in names
    lib = ctypes.CDLL(B.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in stripe.h but not exported"
    assert set(names) == set(B.EXPORTS)


def test_benchmark_configs_plan_with_the_documented_work_figures():
    want = {"tiny_conv_f32": (294912, 270848, 29184), "gemm_bf16_4096": (4096 ** 3, 4096 ** 3, 134217728),
            "resnet_conv_bf16": (3699376128, 3611820032, 38608896),
            "conv7x7_s2_int8": (1888223232, 1859432448, 53798080), "maxpool_f32": (57802752, 57116672, 128450560)}
    for name, (hull, work, nbytes) in want.items():
        blk = B.StripeBlock(W.config_block(name))
        assert (blk.info["hull_points"], blk.info["work_points"], blk.info["algorithmic_bytes"]) == (hull, work, nbytes), name
        blk.close()
    assert B.StripeBlock(W.config_block("gemm_bf16_4096")).info["path_name"] == "mfma_gemm"
    assert B.StripeBlock(W.config_block("maxpool_f32")).info["path_name"] == "pool"


def test_tiled_and_flat_forms_of_the_worked_example_plan_alike():
    a = B.StripeBlock(W.fig5_flat()).info
    b = B.StripeBlock(W.fig5_tiled()).info
    for key in ("n_idx", "n_out_idx", "n_red_idx", "hull_points", "work_points", "output_elements", "kernel", "grid"):
        assert a[key] == b[key], key
    assert a["work_points"] == 200192 and a["hull_points"] == 12 * 16 * 9 * 8 * 16


def test_non_dividing_tile_with_overflow_constraint_merges_back():
    """x split as 5*xo + xi over a range of 12 (quotient rounded up to 3) with the
    overflow removed by 11 - 5*xo - xi >= 0 plans like the un-tiled block."""
    bufs = [W.Buffer("A", "in", "f32", (12, 7)), W.Buffer("B", "in", "f32", (7,)), W.Buffer("O", "out", "f32", (12,))]
    flat = W.flat_block(bufs, dict(x=12, k=7), [(["x", "k"], "assign"), (["k"], "assign"), (["x"], "add")])
    outer = W.make_level(dict(xo=3), [(["5*xo", "0"], "assign", (5, 7)), (["0"], "assign", (7,)),
                                      (["5*xo"], "add", (5,))], buffers=bufs)
    inner = W.make_level(dict(xi=5, k=7), [(["xi", "k"], "assign"), (["k"], "assign"), (["xi"], "add")],
                         buffers=bufs, passed=dict(xb="5*xo"), parent=outer, constraints=["11 - xb - xi >= 0"],
                         intrinsic="mul")
    outer.child = inner
    tiled = W.make_root(bufs, outer)
    a, b = B.StripeBlock(flat).info, B.StripeBlock(tiled).info
    assert (a["n_idx"], a["hull_points"], a["work_points"]) == (b["n_idx"], b["hull_points"], b["work_points"]) == (2, 84, 84)


def status_of(block, path="auto"):
    try:
        B.StripeBlock(block, path).close()
        return 0
    except B.StripeError as e:
        assert e.detail
        return e.status


def test_out_of_bounds_blocks_are_rejected():
    blk = W.conv2d_block(1, 6, 6, 2, 2, 3, 3, 1, 1, "f32", "f32")
    assert status_of(blk) == 0
    blk.child.cons_coeff, blk.child.cons_const = blk.child.cons_coeff[1:], blk.child.cons_const[1:]
    assert status_of(blk) == 4
    big = W.conv2d_block(64, 300, 300, 16, 16, 3, 3, 1, 1, "f32", "f32")   # too large to enumerate: proven symbolically
    assert status_of(big) == 0
    big.child.cons_coeff, big.child.cons_const = big.child.cons_coeff[:3], big.child.cons_const[:3]
    assert status_of(big) == 4
    tiled = W.fig5_tiled()
    tiled.child.refs[0].sizes = [4, 6, 8]      # the halo view is 5 x 6 x 8
    assert status_of(tiled) == 4


def test_assign_and_multi_writer_rules():
    bufs = [W.Buffer("A", "in", "f32", (4, 3)), W.Buffer("O", "out", "f32", (4,))]
    ok = W.flat_block(bufs, dict(a=4, r=1), [(["a", "r"], "assign"), (["a"], "assign")], intrinsic="copy")
    bad = W.flat_block(bufs, dict(a=4, r=3), [(["a", "r"], "assign"), (["a"], "assign")], intrinsic="copy")
    assert status_of(ok) == 0 and status_of(bad) == 5
    tiled = W.fig5_tiled()
    tiled.child.refs[-1].agg = "assign"          # disjoint output tiles: a legal claim
    assert status_of(tiled) == 0
    bufs2 = [W.Buffer("A", "in", "f32", (6,)), W.Buffer("B", "in", "f32", (3,)), W.Buffer("O", "out", "f32", (8,))]
    scatter = W.flat_block(bufs2, dict(x=6, i=3), [(["x"], "assign"), (["i"], "assign"), (["x + i"], "add")])
    sb = B.StripeBlock(scatter)                  # O[x+i]: several (x, i) tuples share an element -> atomic combine
    assert sb.info["kernel"].endswith("_atomic") and sb.info["output_elements"] == 8
    scatter_assign = W.flat_block(bufs2, dict(x=6, i=3), [(["x"], "assign"), (["i"], "assign"), (["x + i"], "assign")])
    assert status_of(scatter_assign) == 5        # 'assign' tolerates one writer only
    assert status_of(scatter, "mfma_gemm") == 3


def test_malformed_descriptors():
    blk = W.matmul_block(4, 4, 4, "f32", "f32")
    blk.refs[0].dtype = blk.child.refs[0].dtype = "i8"
    assert status_of(blk) == 2                   # integer input, float output
    blk = W.matmul_block(4, 4, 4, "f32", "f32")
    blk.child.refs[1].strides = [1, 4]
    assert status_of(blk) == 2                   # a view must keep its parent's strides
    blk = W.matmul_block(4, 4, 4, "f32", "f32")
    blk.child.intrinsic = "copy"
    assert status_of(blk) == 2
    blk = W.matmul_block(4, 4, 4, "f32", "f32")
    blk.child.ranges[0] = -1
    assert status_of(blk) == 2
    h = ctypes.c_void_p()
    assert B.lib.stripe_block_create(None, ctypes.byref(h)) == 1
    assert B.stripe_last_error() != ""
    assert B.stripe_status_string(4) == "access may leave its buffer or view"


def test_very_large_blocks_plan_or_are_refused_cleanly():
    """Sizes at and beyond the limits: no wrap-around in the planner's arithmetic, a status instead of a crash."""
    big = W.matmul_block(65536, 65536, 65536, "bf16", "f32")          # 2^48 points, 8 GB operands: still a GEMM
    info = B.StripeBlock(big).info
    assert info["path_name"] == "mfma_gemm" and info["hull_points"] == 2 ** 48 and info["grid"] == 256 * 256
    assert status_of(W.matmul_block(2 ** 21, 2 ** 21, 2 ** 21, "bf16", "f32")) == 3      # beyond 2^62 points
    bufs = [W.Buffer("A", "in", "f32", (2 ** 17, 2 ** 16)), W.Buffer("O", "out", "f32", (2 ** 17, 2 ** 16))]
    copy = W.flat_block(bufs, dict(a=2 ** 17, b=2 ** 16), [(["a", "b"], "assign"), (["a", "b"], "assign")], intrinsic="copy")
    info = B.StripeBlock(copy).info                                    # offsets beyond 32 bits: the 64-bit kernel
    assert info["kernel"] == "generic_affine_lane_per_output_i64" and info["grid"] == 2 ** 25
    bufs = [W.Buffer("A", "in", "f32", (2 ** 20, 2 ** 20)), W.Buffer("O", "out", "f32", (2 ** 20, 2 ** 20))]
    huge = W.flat_block(bufs, dict(a=2 ** 20, b=2 ** 20), [(["a", "b"], "assign"), (["a", "b"], "assign")], intrinsic="copy")
    assert status_of(huge) == 3                                        # more workgroups than one launch can hold
    one_index = W.flat_block([W.Buffer("A", "in", "f32", (2 ** 33,)), W.Buffer("O", "out", "f32", (2 ** 33,))], dict(x=2 ** 33),
                             [(["x"], "assign"), (["x"], "assign")], intrinsic="copy")
    assert status_of(one_index) == 2                                   # a single range is limited to 2^31 - 1
    wide = W.maxpool_block(1, 3, 2 ** 30, 4, 3, 2, 1)                  # a row wider than the pooling kernels index
    info = B.StripeBlock(wide).info
    assert info["path_name"] == "generic" and info["work_points"] == -1    # too many points to count, reported as such


def test_forcing_a_family_the_block_does_not_have_is_refused():
    assert status_of(W.config_block("maxpool_f32"), "mfma_gemm") == 3
    assert status_of(W.config_block("gemm_bf16_4096"), "pool") == 3
    assert status_of(W.matmul_block(100, 100, 100, "bf16", "f32"), "mfma_gemm") == 3   # not tile-divisible
    assert B.StripeBlock(W.matmul_block(100, 100, 100, "bf16", "f32")).info["path_name"] == "generic"


def test_tune_override_selects_variants(monkeypatch):
    monkeypatch.setenv("STRIPE_TUNE", "pool_ty=4,pool_nt=1")
    assert B.StripeBlock(W.config_block("maxpool_f32")).info["kernel"] == "pool_max_f32_3x3s2_ty4_nt"
    monkeypatch.delenv("STRIPE_TUNE")
    assert B.StripeBlock(W.config_block("maxpool_f32")).info["kernel"] == "pool_max_f32_3x3s2_ty1x4"


def test_split_reduction_is_planned_for_few_tiles_and_long_k(monkeypatch):
    """Section 2.1: an aggregation may be regrouped.  Few output tiles + long reduction index => slices over
    workgroups, with a workspace of one partial-sum image per slice; large products and short reductions stay whole."""
    sb = B.StripeBlock(W.matmul_block(256, 256, 65536, "bf16", "f32"))
    assert "_splitk" in sb.info["kernel"]
    S = int(sb.info["kernel"].rsplit("_splitk", 1)[1])
    assert S >= 2 and 65536 % (S * 128) == 0
    assert sb.info["workspace_bytes"] == S * 256 * 256 * 4 == B.stripe_block_workspace_size(sb.handle)
    assert sb.info["grid"] == 4 * S                       # four 128 x 128 tiles, S slices each
    with pytest.raises(B.StripeError) as e:
        B.stripe_block_set_workspace(sb.handle, 256, 1024)            # too small
    assert e.value.status == 7
    with pytest.raises(B.StripeError) as e:
        B.stripe_block_set_workspace(sb.handle, 257, 1 << 30)         # misaligned
    assert e.value.status == 2
    B.stripe_block_set_workspace(sb.handle, 0, 0)                     # back to handle-owned memory
    sb.close()
    for shape in [(4096, 4096, 4096), (512, 512, 512), (2048, 2048, 2048)]:
        sb = B.StripeBlock(W.matmul_block(*shape, "bf16", "f32"))
        assert "_splitk" not in sb.info["kernel"] and sb.info["workspace_bytes"] == 0, sb.info["kernel"]
        sb.close()
    monkeypatch.setenv("STRIPE_TUNE", "gemm_splitk=0")
    sb = B.StripeBlock(W.matmul_block(256, 256, 65536, "bf16", "f32"))
    assert "_splitk" not in sb.info["kernel"] and sb.info["workspace_bytes"] == 0
    sb.close()


def test_statement_list_reports_its_workspace():
    prog = W.conv_bias_relu_program(2, 9, 7, 5, 6, 3, 3, 1, 1, "f32", "f32")
    sb = B.StripeBlock(prog)
    assert sb.info["workspace_bytes"] == (2 * 9 * 7 * 6 * 4 + 255) // 256 * 256
    sb.close()
    fused = B.StripeBlock(W.conv_bias_relu_program(1, 7, 20, 64, 64, 3, 3, 1, 1, "bf16", "f32"))
    assert "+bias_relu" in fused.info["kernel"] and fused.info["workspace_bytes"] == 0     # the temporary was scalarised away
    fused.close()


def test_tile_selection_follows_the_cost_model():
    """Section 3.3's model as the library's tile selector: strip heights of the window family (register level, with
    the occupancy correction) and the workgroup tile of the general convolution kernel (LDS level)."""
    kernel = lambda blk: B.StripeBlock(blk).info["kernel"]
    assert kernel(W.config_block("maxpool_f32")).endswith("3x3s2_ty1x4")                # rows shared through L1: 9 rows per 4
    assert kernel(W.maxpool_block(32, 112, 112, 64, 2, 2, 0)).endswith("2x2s2_ty1")     # no sharing: the smallest footprint
    assert kernel(W.maxpool_block(32, 112, 112, 64, 3, 1, 1)).endswith("3x3s1_ty4x4")   # stride 1 shares most: registers and L1
    assert kernel(W.depthwise_conv_block(32, 112, 112, 64, 3, 3, 1, 1, "f32")).endswith("3x3s1_ty3x2")   # four rows would leave three wavefronts per SIMD: the measured best
    assert "256x64x32" in kernel(W.conv2d_block(4, 28, 28, 64, 32, 3, 3, 1, 1, "bf16", "f32"))
    # (the K tile: 128-byte rows = 64 bf16 channels on the 128 x 128 tile where the block has at most one tile per CU)
    assert "128x128x64" in kernel(W.conv2d_block(4, 28, 28, 128, 128, 3, 3, 1, 1, "bf16", "f32"))
    assert "128x128x64" in kernel(W.conv2d_block(4, 28, 28, 64, 96, 3, 3, 1, 1, "bf16", "f32"))
    assert "128x128x32" in kernel(W.conv2d_block(4, 28, 28, 32, 96, 3, 3, 1, 1, "bf16", "f32"))    # 32 channels: 64-byte rows
    assert "256x64x32" in kernel(W.conv2d_block(4, 28, 28, 128, 192, 3, 3, 1, 1, "bf16", "f32"))   # three 64-wide tiles waste nothing
    # the largest tile where its tiles fill one round of workgroups: 196 of them here, 392 there (then 784 smaller ones, two per CU)
    assert "256x128x32" in kernel(W.conv2d_block(32, 28, 28, 128, 192, 3, 3, 1, 1, "bf16", "f32"))
    assert "conv_gemm_bf16_256x256x32" in kernel(W.conv2d_block(16, 56, 56, 128, 256, 3, 3, 1, 1, "bf16", "f32"))   # 196 tiles of 256 x 256: the contraction kernel
    assert "conv_igemm_bf16_128x128x32" in kernel(W.conv2d_block(32, 56, 56, 128, 128, 3, 3, 1, 1, "bf16", "f32"))   # half a 256-wide tile would be padding: 784 tiles of 128 x 128, two per CU


def _two_statements(t_access_write, t_access_read, write_constraints=(), write_range=8):
    """0: T[<t_access_write>] = A[x] * A[x]  (x in 0..write_range-1);   1: O[x] = relu(T[<t_access_read>] + B[x])  (x in 0..7)."""
    bufs = [W.Buffer("A", "in", "f32", (16,)), W.Buffer("B", "in", "f32", (8,)), W.Buffer("T", "temp", "f32", (16,)),
            W.Buffer("O", "out", "f32", (8,))]
    s0 = W.make_level(dict(x=write_range), [(["x"], "assign"), (["x"], "assign"), ([t_access_write], "assign")],
                      buffers=[bufs[0], bufs[0], W.Buffer("T", "out", "f32", (16,))], constraints=list(write_constraints), intrinsic="mul")
    s0.parent_refs = [0, 0, 2]
    s1 = W.make_level(dict(x=8), [([t_access_read], "assign"), (["x"], "assign"), (["x"], "assign")],
                      buffers=[W.Buffer("T", "in", "f32", (16,)), bufs[1], bufs[3]], intrinsic="add_relu")
    s1.parent_refs = [2, 1, 3]
    s0.next = s1
    return W.make_root(bufs, s0)


def test_statement_list_that_reads_unwritten_temporary_elements_is_refused():
    B.StripeBlock(_two_statements("x", "x")).close()                       # writes T[0..7], reads T[0..7]
    with pytest.raises(B.StripeError) as e:
        B.StripeBlock(_two_statements("x", "x", write_range=6))            # writes six elements, reads eight
    assert e.value.status == 2 and "temporary" in str(e.value)
    with pytest.raises(B.StripeError) as e:
        B.StripeBlock(_two_statements("x", "x", write_constraints=["x - 2 >= 0"]))   # T[0], T[1] have no iteration
    assert e.value.status == 2 and "temporary" in str(e.value)


def test_statement_that_reads_its_own_output_through_another_map_is_refused():
    """Definition 2 rule 2: an element written by one iteration may not be read by another.  T[x] = relu(T[x] + B[x])
    is a per-element update; T[x] = relu(T[x + 1] + B[x]) is not."""
    def prog(read_access):
        bufs = [W.Buffer("A", "in", "f32", (16,)), W.Buffer("B", "in", "f32", (8,)), W.Buffer("T", "temp", "f32", (16,)),
                W.Buffer("O", "out", "f32", (8,))]
        s0 = W.make_level(dict(x=16), [(["x"], "assign"), (["x"], "assign"), (["x"], "assign")],
                          buffers=[bufs[0], bufs[0], W.Buffer("T", "out", "f32", (16,))], intrinsic="mul")
        s0.parent_refs = [0, 0, 2]
        s1 = W.make_level(dict(x=8), [([read_access], "assign"), (["x"], "assign"), (["x"], "assign")],
                          buffers=[W.Buffer("T", "in", "f32", (16,)), bufs[1], W.Buffer("T", "out", "f32", (16,))], intrinsic="add_relu")
        s1.parent_refs = [2, 1, 2]
        s2 = W.make_level(dict(x=8), [(["x"], "assign"), (["x"], "assign"), (["x"], "assign")],
                          buffers=[W.Buffer("T", "in", "f32", (16,)), bufs[1], bufs[3]], intrinsic="add")
        s2.parent_refs = [2, 1, 3]
        s0.next, s1.next = s1, s2
        return W.make_root(bufs, s0)
    B.StripeBlock(prog("x")).close()
    with pytest.raises(B.StripeError) as e:
        B.StripeBlock(prog("x + 1"))
    assert e.value.status == 2 and "reads the buffer it writes" in str(e.value)


def test_constraint_coefficient_beyond_32_bits_is_refused_not_truncated():
    """A passed value scaled by 2^20 inside a constraint scaled by 2^12: the flattened coefficient is 2^32."""
    bufs = [W.Buffer("A", "in", "i32", (2, 3)), W.Buffer("O", "out", "i32", (2, 3))]
    outer = W.make_level(dict(x=2), [(["x", "0"], "assign", (1, 3)), (["x", "0"], "assign", (1, 3))], buffers=bufs)
    inner = W.make_level(dict(y=3), [(["0", "y"], "assign"), (["0", "y"], "assign")], buffers=bufs, passed=dict(p="1048576*x"),
                         parent=outer, constraints=["5 - 4096*p - y >= 0"], intrinsic="copy")
    outer.child = inner
    with pytest.raises(B.StripeError) as e:
        B.StripeBlock(W.make_root(bufs, outer))
    assert e.value.status == 3


def test_fusion_keeps_apart_what_the_general_kernel_leaves_unwritten():
    """Padding beyond the filter: some output pixels have no tap inside the image, the convolution writes nothing there
    and the temporary would hold an undefined element: such a list is refused (unwritten temporary) rather than fused."""
    prog = W.conv_bias_relu_program(1, 8, 8, 32, 32, 3, 3, 1, 3, "bf16", "f32")
    with pytest.raises(B.StripeError):
        B.StripeBlock(prog)


@pytest.mark.parametrize("M,N,K,rows", [(8, 4096, 4096, True), (32, 1024, 4096, True), (8, 256, 32768, False), (16, 128, 32768, False),
                                        (32, 1024, 16384, False), (2, 120000, 512, True), (32, 120000, 2048, False), (8, 4096, 8192, True)])
def test_few_row_products_go_to_the_faster_kernel(M, N, K, rows):
    """Few columns with a long reduction keep the split product (8 x 256 x 32768: 16 us split, 47 us on the few-rows kernel),
    very many columns with more than 16 rows the 256-wide tiles."""
    b = B.StripeBlock(W.matmul_block(M, N, K, "bf16", "f32", b_transposed=True))
    assert b.info["kernel"].startswith("gemm_rows_") == rows, b.info["kernel"]
    b.close()


@pytest.mark.parametrize("blk,literal", [
    (W.matmul_block(33, 33, 1001, "f32", "f32", b_transposed=True), True), (W.matmul_block(250, 250, 1001, "f32", "f32", b_transposed=True), False),
    (W.matmul_block(4, 100, 4001, "f32", "f32", b_transposed=True), True), (W.matmul_block(100000, 3, 5, "f32", "f32"), True),
    (W.conv2d_block(1, 16, 16, 12, 12, 5, 5, 1, 2, "f32", "f32"), True), (W.conv2d_block(1, 56, 56, 12, 12, 5, 5, 1, 2, "f32", "f32"), False),
    (W.conv2d_block(27, 184, 184, 3, 8, 3, 3, 1, 1, "f32", "f32"), True), (W.conv2d_block(8, 112, 112, 3, 8, 3, 3, 2, 1, "f32", "f32"), False)])
def test_blocks_stay_on_the_literal_kernel_where_it_is_faster(blk, literal, monkeypatch):
    """Few tiles with a long reduction, short reductions, few columns; a set contract_min overrides the rule, at any value."""
    for tune, want in (("", literal), ("contract_min=65536", False), ("contract_min=65535", False)):
        monkeypatch.setenv("STRIPE_TUNE", tune)
        b = B.StripeBlock(blk)
        assert b.info["kernel"].startswith("generic_") == want, (tune, b.info["kernel"])
        b.close()


def strided_conv(R, S, stride_x, Ho, Wo, Ci, Co, dt):
    """A convolution whose image is as large as its taps reach: stride 1 along y, stride_x along x."""
    H, Wd = Ho + R - 1, stride_x * (Wo - 1) + S
    bufs = [W.Buffer("I", "in", dt, (1, H, Wd, Ci)), W.Buffer("F", "in", dt, (R, S, Co, Ci)), W.Buffer("O", "out", "i32" if dt == "i8" else "f32", (1, Ho, Wo, Co))]
    return W.flat_block(bufs, dict(n=1, y=Ho, x=Wo, i=R, j=S, c=Ci, k=Co),
                        [(["n", "y + i", f"{stride_x}*x + j", "c"], "assign"), (["i", "j", "k", "c"], "assign"), (["n", "y", "x", "k"], "add")])


@pytest.mark.parametrize("R,stride_x,dt", [(26, 600000, "f32"), (26, 688300, "f32"), (28, 800000, "bf16")])
def test_image_rows_that_no_lds_holds(R, stride_x, dt):
    """Few input channels, rows of image of gigabytes between the taps: sizes that 32-bit products wrap into a plausible range.  The
    general contraction's, which holds no image rows; what is planned fits the 160 KB of LDS."""
    b = B.StripeBlock(strided_conv(R, 2, stride_x, 40, 2, 2, 4096, dt))
    assert not b.info["kernel"].startswith("conv_few_") and 0 <= b.info["lds_bytes"] <= 160 * 1024, (b.info["kernel"], b.info["lds_bytes"])
    b.close()


@pytest.mark.parametrize("M,N,K,out_dt,b_transposed", [(64, 136, 1536, "f32", True), (33, 64, 1024, "bf16", False), (15, 320, 8192, "bf16", True),
                                                       (100, 24, 1536, "f32", False), (2, 24, 1536, "f32", False)])
def test_an_output_laid_out_unlike_the_temporary_is_fused(M, N, K, out_dt, b_transposed):
    """Products of few tiles, which the general contraction takes where it can store through the second statement: where it cannot (rows
    of the output further apart than the temporary's), their family's kernel does, in one launch and without a temporary."""
    prog = W.linear_bias_relu_program(M, N, K, out_dt, b_transposed=b_transposed)
    prog.refs[-1].strides = [N + 8, 1]
    prog.child.next.refs[-1].strides = [N + 8, 1]
    b = B.StripeBlock(prog)
    assert "+bias_relu" in b.info["kernel"] and b.info["workspace_bytes"] == 0, b.info
    b.close()


def test_a_fused_product_on_the_contraction_refuses_what_its_family_refuses():
    """Inputs at 16 bytes, the bias at 4, the output at its element: refused before anything is launched, so without a GPU too."""
    for out_dt, esize in (("f32", 4), ("bf16", 2)):
        b = B.StripeBlock(W.linear_bias_relu_program(64, 136, 1536, out_dt))
        assert b.info["kernel"].startswith("contract_") and b.info["path_name"] == "mfma_gemm", b.info
        x, w, bias, out = (1 << 20 << i for i in range(4))      # never touched
        for ptrs in ((x + 2, w, bias, out), (x, w + 8, bias, out), (x, w, bias + 2, out), (x, w, bias, out + esize // 2)):
            with pytest.raises(B.StripeError) as e:
                b.run(ptrs[:3], ptrs[3], stream=0)
            assert e.value.status == 8, (ptrs, str(e.value))
        b.close()


@pytest.mark.parametrize("M,N,K", [(8, 64, 8192), (12, 320, 8192), (16, 128, 8192), (20, 1000, 8192), (8, 4096, 4096)])
def test_few_rows_with_an_fp32_output_keep_totals_in_double(M, N, K):
    """A Linear layer with bias and relu at few rows: the few-rows kernel's totals are in double precision, and those of the general
    contraction where it takes its place (its name says so)."""
    b = B.StripeBlock(W.linear_bias_relu_program(M, N, K, "f32"))
    assert b.info["kernel"].startswith("gemm_rows_") or "_f64" in b.info["kernel"], b.info["kernel"]
    assert b.info["kernel"].endswith("+bias_relu") and b.info["path_name"] == "mfma_gemm", b.info
    b.close()


@pytest.mark.parametrize("N,H,Ci,Co,R,stride,dt,few", [(10, 50, 2, 1008, 3, 3, "f32", False), (7, 127, 3, 103, 2, 1, "f32", False), (5, 142, 2, 344, 3, 1, "i8", False),
                                                      (24, 94, 3, 64, 3, 1, "i8", False), (3, 153, 3, 46, 3, 1, "i8", False), (8, 224, 3, 64, 7, 2, "bf16", True),
                                                      (3, 75, 3, 64, 7, 2, "f32", True), (13, 61, 3, 32, 7, 2, "i8", True)])
def test_few_input_channels_where_their_kernel_is_the_faster_one(N, H, Ci, Co, R, stride, dt, few):
    """Many tiles of output channels and large outputs in single elements stay on the general contraction (2.7, 1.7, 6.6, 3.6 and 1.4 times as
    slow on the few-channels kernel when it took them); the first layers of image networks do not."""
    b = B.StripeBlock(W.conv2d_block(N, H, H, Ci, Co, R, R, stride, 0 if R == 2 else R // 2, dt, "i32" if dt == "i8" else "f32"))
    assert b.info["kernel"].startswith("conv_few_" if few else "contract_"), b.info["kernel"]
    b.close()


@pytest.mark.parametrize("tune", ["", "pool_ty=2", "pool_nt=1,generic_i64=0", "fuse=1"])
def test_a_knob_of_one_family_leaves_the_others_alone(tune, monkeypatch):
    """A ragged product on 128-wide tiles, a first layer of an image network, a product and a convolution of few tiles on the contraction."""
    blocks = [W.matmul_block(2000, 2048, 2048, "i8", "i32", b_transposed=True), W.conv2d_block(8, 224, 224, 3, 64, 7, 7, 2, 3, "bf16", "f32"),
              W.matmul_block(6, 1536, 768, "bf16", "f32"), W.conv2d_block(3, 42, 42, 256, 9, 7, 7, 1, 3, "i8", "i32")]
    monkeypatch.delenv("STRIPE_TUNE", raising=False)
    want = [B.StripeBlock(b).info["kernel"] for b in blocks]
    assert [w.split("_")[0] for w in want] == ["gemm", "conv", "contract", "contract"] and "128x128" in want[0] and "conv_few" in want[1], want
    monkeypatch.setenv("STRIPE_TUNE", tune)
    assert [B.StripeBlock(b).info["kernel"] for b in blocks] == want


@pytest.mark.parametrize("M,N,K,dt,layout,lds", [(1000, 1000, 3000, "bf16", "tn", 7 * 64 * 64 * 4 + 128 * 24),       # the sums on their way to each other are the most
                                                 (56, 64, 4080, "bf16", "nt", 16 * 32 * 256 + 32 * 24)])             # K tiles of 16 wavefronts
def test_lds_of_the_general_contraction(M, N, K, dt, layout, lds):
    """What its kernels declare: it decides how many workgroups a CU holds."""
    bufs = [W.Buffer("A", "in", dt, (K, M) if layout == "tn" else (M, K)), W.Buffer("B", "in", dt, (N, K) if layout == "nt" else (K, N)), W.Buffer("C", "out", "f32", (M, N))]
    b = B.StripeBlock(W.flat_block(bufs, dict(m=M, n=N, k=K), [(["k", "m"] if layout == "tn" else ["m", "k"], "assign"),
                                                               (["n", "k"] if layout == "nt" else ["k", "n"], "assign"), (["m", "n"], "add")]))
    assert b.info["kernel"].startswith("contract_") and b.info["lds_bytes"] == lds, b.info
    b.close()


@pytest.mark.parametrize("N,H,Ci,Co,R,stride", [(1, 20, 4, 16, 2, 1), (2, 35, 3, 32, 2, 1), (4, 35, 4, 64, 2, 2), (2, 49, 3, 64, 3, 1), (7, 19, 3, 48, 3, 2)])
def test_few_input_channels_and_a_short_fp32_reduction(N, H, Ci, Co, R, stride):
    """12 or 16 products, which both kernels sum as two chains of eight, and 27: on the one for few input channels."""
    b = B.StripeBlock(W.conv2d_block(N, H, H, Ci, Co, R, R, stride, 0 if R == 2 else R // 2, "f32", "f32"))
    assert b.info["kernel"].startswith("conv_few_"), b.info["kernel"]
    b.close()


@pytest.mark.parametrize("N,H,Ci,Co,dt,up", [(2, 55, 64, 115, "f32", False), (1, 70, 40, 100, "f32", False), (2, 49, 64, 15, "bf16", True), (1, 49, 64, 29, "f32", True),
                                             (2, 32, 64, 20, "bf16", True)])
def test_convolutions_on_the_tile_whose_k_tile_wavefronts_share(N, H, Ci, Co, dt, up):
    """3x3 convolutions (transposed: the last 4x4) that lost 4 to 42 % of their time when that tile was gone."""
    R = 4 if Co == 20 else 3
    if up:
        Ho = 2 * (H - 1) + R
        bufs = [W.Buffer("I", "in", dt, (N, H, H, Ci)), W.Buffer("F", "in", dt, (R, R, Ci, Co)), W.Buffer("O", "out", "f32", (N, Ho, Ho, Co))]
        blk = W.flat_block(bufs, dict(n=N, y=H, x=H, i=R, j=R, c=Ci, k=Co),
                           [(["n", "y", "x", "c"], "assign"), (["i", "j", "c", "k"], "assign"), (["n", "2*y + i", "2*x + j", "k"], "add")])
    else:
        blk = W.conv2d_block(N, H, H, Ci, Co, R, R, 1, 1, dt, "f32")
    b = B.StripeBlock(blk)
    assert b.info["kernel"].startswith(f"contract_{dt}_32x32x") and b.info["workgroup_size"] == 256, b.info
    b.close()


@pytest.mark.parametrize("M,N,K,tile", [(1857, 3136, 64, "128x128"), (4096, 4096, 64, "128x128"), (2500, 1300, 64, "128x128"), (1024, 3000, 40, "64x64"), (3000, 3000, 200, "64x64")])
def test_int8_products_of_one_k_tile(M, N, K, tile):
    """Many outputs and a short reduction on large tiles (10.6 and 12.4 us, 16.8 and 25.7, 8.8 and 10.6 on 64 x 64), not with few tiles or a longer one."""
    b = B.StripeBlock(W.matmul_block(M, N, K, "i8", "i32"))
    assert b.info["kernel"].startswith(f"contract_i8_{tile}x"), b.info["kernel"]
    b.close()
