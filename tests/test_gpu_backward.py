"""Backward pass of the HIP path (bs_stack_plan_backward / bs_stack_backward through the C ABI)
against the backward oracle on the same seeded inputs.

Tolerance: the kernels accumulate in float32 and round once (the oracle in float64, unrounded):
max|err| <= 1e-5 * max|ref| for float32 and 1e-2 * max|ref| for 16-bit storage, which also
covers the 16-bit rounding of the gradients handed from stage to stage.  The decisions the
gradient depends on (ReLU signs, max-pooling picks) are the forward pass's on both sides."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import backward as bw
from paper_1804_08378_amd import brainslug as bs
from paper_1804_08378_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 1e-2, "f16": 1e-2}
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", TORCH[dtype])


def _inputs(layers, shape, seed, dtype):
    x = wl.activation(shape, seed, dtype)
    res = [wl.activation(s, seed + 1 + i, dtype) for i, s in enumerate(wl.residual_shapes(layers, shape))]
    dy = wl.activation(wl.output_shape(layers, shape), seed + 50, dtype)
    return x, res, dy


def run_gpu(layers, x, res, dy, dtype, need_input=True, need_res=None, **opts):
    st = bs.Stack(layers, x.shape, dtype).plan(**opts).plan_backward()
    stages = bs.bs_stack_backward_num_stages(st.handle)
    # a channels-last plan takes and returns channels_last tensors; what is read back are the logical N, C, H, W values
    mf = torch.channels_last if opts.get("layout") == bs.BS_LAYOUT_NHWC else torch.contiguous_format
    put = lambda a: _dev(a, dtype).contiguous(memory_format=mf)
    gx, gres = st.backward(put(x), [put(r) for r in res], put(dy), need_input, need_res)
    for t in [gx] + list(gres):
        assert t is None or t.is_contiguous(memory_format=mf)
    torch.cuda.synchronize()
    out = None if gx is None else gx.float().cpu().numpy()
    outs = [None if g is None else g.float().cpu().numpy() for g in gres]
    st.close()
    return out, outs, stages


def _close(got, ref, dtype, label):
    assert got.shape == ref.shape, label
    scale = float(np.abs(ref).max()) or 1.0
    err = float(np.abs(got.astype(np.float64) - ref).max())
    print(f"         {label}: max|err|={err:.3e} (bar {TOL[dtype] * scale:.3e})", flush=True)
    assert np.isfinite(got).all(), label
    assert err <= TOL[dtype] * scale, label


def check(layers, shape, dtype, label, seed=0, **opts):
    print(f"[backward] {label} shape={shape} dtype={dtype} opts={opts}", flush=True)
    x, res, dy = _inputs(layers, shape, seed, dtype)
    ref_x, ref_res = bw.backward_stack(layers, x, res, dy, dtype)
    gx, gres, stages = run_gpu(layers, x, res, dy, dtype, **opts)
    _close(gx, ref_x, dtype, label + " grad_x")
    assert len(gres) == len(ref_res)
    for i, (a, b) in enumerate(zip(gres, ref_res)):
        _close(a, b, dtype, f"{label} grad_residual[{i}]")
    return stages


CASES = [(n, d) for n in wl.CONFIG_NAMES for d in wl.build(n)[2]]


@pytest.mark.parametrize("name,dtype", CASES)
def test_named_configurations(name, dtype):
    layers, shape, _ = wl.build(name, 0, 2, False)
    check(layers, shape, dtype, name)


def _stacks(c):
    return {
        "bn_relu_max2": [wl.bn_params(c, 1), wl.relu(), wl.maxpool(2, 2, 0)],
        "bn_relu_max3s2p1": [wl.bn_params(c, 2), wl.relu(), wl.maxpool(3, 2, 1)],
        "bn_add_relu": [wl.bn_params(c, 3), wl.add(), wl.relu()],
        "bn_relu_avg2": [wl.bn_params(c, 4), wl.relu(), wl.avgpool(2, 2)],
        "halo_stress": [wl.bn_params(c, 5), wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1),
                        wl.bn_params(c, 6), wl.relu()],
        "max_bn_relu_x3": sum(([wl.maxpool(3, 1, 1), wl.bn_params(c, 7 + i), wl.relu()] for i in range(3)), []),
        "avg_nopad_div": [wl.relu(), wl.avgpool(3, 2, 1, False), wl.add(), wl.maxpool(2, 1, 0)],
        "rect_windows": [wl.bn_params(c, 9), wl.maxpool((3, 2), (2, 1), (1, 0)), wl.avgpool((2, 3), (1, 2), (1, 1), True)],
        "two_adds": [wl.add(), wl.bn_params(c, 10), wl.leaky_relu(0.1), wl.add(), wl.clamp(-0.5, 1.5)],
        "ceil_avg": [wl.bn_params(c, 11), wl.avgpool(3, 2, 1, True, ceil_mode=True), wl.relu()],
        "ceil_avg_nopad": [wl.avgpool(2, 2, 0, False, ceil_mode=True), wl.bn_params(c, 12)],
        "ceil_max": [wl.leaky_relu(0.2), wl.maxpool(3, 2, 0, ceil_mode=True), wl.add(), wl.relu()],
        "global_avg": [wl.bn_params(c, 13), wl.relu(), wl.avgpool((12, 16), (12, 16), 0)],
        "global_max": [wl.bn_params(c, 14), wl.maxpool((12, 16), (12, 16), 0), wl.relu()],
        "pool_first_then_add": [wl.maxpool(2, 2), wl.add(), wl.bn_params(c, 15), wl.relu(), wl.avgpool(2, 2), wl.add()],
        "stride_gt_kernel": [wl.bn_params(c, 16), wl.maxpool(2, 3, 0), wl.avgpool(1, 2, 0)],
    }


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("name", list(_stacks(3)))
def test_small_stacks_vector_and_ragged_rows(name, dtype):
    layers = _stacks(5)[name]
    check(layers, (3, 5, 12, 16), dtype, name + "/vector rows")     # rows of whole 128-bit vectors
    if not name.startswith("global"):
        check(layers, (2, 5, 13, 11), dtype, name + "/ragged rows", seed=3)  # one cell per lane


def _own_pick_stacks(c):
    return {
        "stem": [wl.bn_params(c, 30), wl.relu(), wl.maxpool(3, 2, 1)],
        "stem_add": [wl.bn_params(c, 31), wl.add(), wl.leaky_relu(0.1), wl.maxpool(3, 2, 1)],
        "max3s1": [wl.bn_params(c, 32), wl.relu(), wl.maxpool(3, 1, 1)],
        "pool_only": [wl.maxpool(3, 2, 1)],
        "two_adds_s1": [wl.add(), wl.bn_params(c, 33), wl.add(), wl.clamp(-0.5, 1.0), wl.maxpool(3, 1, 1)],
        "chain": [wl.maxpool(3, 1, 1), wl.bn_params(c, 34), wl.relu(), wl.maxpool(3, 2, 1), wl.bn_params(c, 35), wl.relu()],
        "avg3s1": [wl.bn_params(c, 37), wl.relu(), wl.avgpool(3, 1, 1, True)],
        "avg3s2_in_range_count": [wl.add(), wl.bn_params(c, 38), wl.avgpool(3, 2, 1, False)],
        "halo_stress": [wl.bn_params(c, 39), wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), wl.bn_params(c, 40), wl.relu()],
    }


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(2, 3, 12, 16), (1, 2, 40, 32), (1, 2, 37, 24), (2, 2, 7, 8), (1, 1, 1, 8), (1, 2, 5, 256),
                                   (1, 1, 9, 264), (2, 1, 70, 16)])
def test_overlapping_max_windows_without_recorded_picks(shape, dtype):
    """3 x 3 max windows (stride 1 and 2, padding 1) on rows of whole vectors: the lanes of a row find the picks
    themselves.  Several chunks of rows, odd heights, one row, rows that fill a wave (64 column blocks) or do not
    fit one (264 float32 columns: recorded picks again).  Against the oracle, and bit for bit against the
    kernel that gathers recorded picks: both sum a cell's windows in the same order."""
    for name, layers in _own_pick_stacks(shape[1]).items():
        label = f"own picks/{name}"
        x, res, dy = _inputs(layers, shape, 7, dtype)
        x[:, :, ::2, 1::3] = 0.5   # ties inside windows
        ref_x, ref_res = bw.backward_stack(layers, x, res, dy, dtype)
        print(f"[backward] {label} shape={shape} dtype={dtype}", flush=True)
        gx, gres, _ = run_gpu(layers, x, res, dy, dtype)
        hx, hres, _ = run_gpu(layers, x, res, dy, dtype, lane_exchange=-1)
        _close(gx, ref_x, dtype, label + " grad_x")
        _close(hx, ref_x, dtype, label + " grad_x (recorded picks)")
        # the operations behind the last pooling join its stage (no gradient rounded to 16 bits in between)
        # (and the average's box sums add in another order than the gather does: no common bits there)
        same_bits = (dtype == "f32" or name not in ("chain", "halo_stress")) and "avg" not in name and name != "halo_stress"
        assert not same_bits or np.array_equal(gx.view(np.uint32), hx.view(np.uint32)), label
        for i, (a, b, c) in enumerate(zip(gres, ref_res, hres)):
            _close(a, b, dtype, f"{label} grad_residual[{i}]")
            assert not same_bits or np.array_equal(a.view(np.uint32), c.view(np.uint32)), label
    st = bs.Stack(_own_pick_stacks(shape[1])["stem"], shape, dtype).plan().plan_backward()
    fits = shape[3] // (4 if dtype == "f32" else 8) <= 64
    assert (bs.bs_stack_backward_workspace_bytes(st.handle) == 0) == fits
    st.close()
    # max pool, BatchNorm, ReLU: one stage where the lanes find the picks, two otherwise
    layers = [wl.maxpool(3, 2, 1), wl.bn_params(shape[1], 36), wl.relu()]
    for opts, want in (({}, 1 if fits else 2), (dict(lane_exchange=-1), 2)):
        st = bs.Stack(layers, shape, dtype).plan(**opts).plan_backward()
        assert bs.bs_stack_backward_num_stages(st.handle) == want
        st.close()
    check(layers, shape, dtype, "own picks/pool_bn_relu", seed=9)


def _strip_stacks(c):
    return {
        "stem": [wl.bn_params(c, 90), wl.relu(), wl.maxpool(3, 2, 1)],
        "incep": [wl.bn_params(c, 91), wl.relu(), wl.maxpool(3, 2, 0)],
        "ceil": [wl.relu(), wl.maxpool(3, 2, 0, ceil_mode=True)],
        "ceil_padded": [wl.maxpool(3, 2, 1, ceil_mode=True), wl.leaky_relu(0.2)],
        "stride1": [wl.bn_params(c, 92), wl.relu(), wl.maxpool(3, 1, 1)],
        "stride1_no_padding": [wl.clamp(-0.5, 0.5), wl.maxpool(3, 1, 0), wl.bn_params(c, 93), wl.relu()],
        "pool_only": [wl.maxpool(3, 2, 1)],
        "halo_stress": [wl.bn_params(c, 94), wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), wl.bn_params(c, 95), wl.relu()],
        "halo_in_range_count": [wl.leaky_relu(0.1), wl.avgpool(3, 1, 1, False), wl.maxpool(3, 2, 1, ceil_mode=True)],
    }


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(2, 5, 3, 3), (1, 64, 4, 4), (2, 8, 9, 5), (1, 3, 7, 8), (2, 16, 21, 9), (1, 70, 37, 17), (3, 2, 70, 16)])
def test_channels_last_strips(shape, dtype):
    """Channels-last 3 x 3 max pooling (alone, or behind a 3 x 3 / 1 average) in the kernels whose lanes walk strips of columns:
    planes narrower than a strip, odd sizes, whole and ragged strips, one and several chunks of rows, ties.  Against the
    oracle, and -- one pooling, nothing handed on in 16 bits -- bit for bit against the kernel that gathers recorded picks
    (both sum a cell's windows in the same order).  Tolerance: test module."""
    nhwc = dict(layout=bs.BS_LAYOUT_NHWC)
    for name, layers in _strip_stacks(shape[1]).items():
        label = f"strips/{name}"
        x, res, dy = _inputs(layers, shape, 23, dtype)
        x[:, :, ::2, 1::3] = 0.5
        print(f"[backward] {label} shape={shape} dtype={dtype}", flush=True)
        ref_x, _ = bw.backward_stack(layers, x, res, dy, dtype)
        gx, _, stages = run_gpu(layers, x, res, dy, dtype, **nhwc)
        assert stages == 1, label
        _close(gx, ref_x, dtype, label)
        if name in ("stem", "incep", "ceil", "stride1", "pool_only"):
            hx, _, _ = run_gpu(layers, x, res, dy, dtype, lane_exchange=-1, **nhwc)
            if dtype == "f16":
                # float32 product, then binary16: the compiler may merge the two roundings into one (v_fma_mixlo_f16) in
                # either kernel, which moves a value by at most one unit in its last place (11-bit significand; 2^-24
                # between subnormal numbers)
                assert (np.abs(gx - hx) <= 2.0 ** -10 * np.abs(hx) + 2.0 ** -24).all(), label
            else:
                assert np.array_equal(gx, hx), label


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(1, 1, 3, 3), (2, 3, 4, 5), (1, 2, 9, 7), (2, 5, 13, 11), (1, 3, 37, 35), (1, 1, 5, 261), (2, 2, 70, 18)])
def test_row_major_strips(shape, dtype):
    """The same kernels on row-major tensors whose rows are no whole vectors (and on windows without padding): tensors
    shorter than one lane's run of columns, the first and last rows of a tensor, ragged strips, chunks of rows."""
    for name, layers in _strip_stacks(shape[1]).items():
        label = f"row strips/{name}"
        x, res, dy = _inputs(layers, shape, 29, dtype)
        x[:, :, ::2, 1::3] = 0.5
        print(f"[backward] {label} shape={shape} dtype={dtype}", flush=True)
        ref_x, _ = bw.backward_stack(layers, x, res, dy, dtype)
        gx, _, stages = run_gpu(layers, x, res, dy, dtype)
        assert stages == 1, label
        _close(gx, ref_x, dtype, label)
        if name in ("stem", "incep", "ceil", "stride1", "pool_only"):
            hx, _, _ = run_gpu(layers, x, res, dy, dtype, lane_exchange=-1)
            if dtype == "f16":  # as in test_channels_last_strips
                assert (np.abs(gx - hx) <= 2.0 ** -10 * np.abs(hx) + 2.0 ** -24).all(), label
            else:
                assert np.array_equal(gx, hx), label


def test_channels_last_strips_with_infinities_and_offsets_beyond_4_gib():
    """Windows of nothing but -infinity hand their gradient to their first cell inside the plane (the recorded pick);
    a channel slice whose pixels lie so far apart that byte offsets need more than 32 bits."""
    nhwc = dict(layout=bs.BS_LAYOUT_NHWC)
    for pool in (wl.maxpool(3, 2, 1), wl.maxpool(3, 2, 0), wl.maxpool(3, 1, 1)):
        x = wl.activation((1, 6, 9, 11), 3)
        x[:, ::2] = -np.inf
        x[:, 1, :4, :5] = -np.inf
        dy = wl.activation(wl.output_shape([pool], x.shape), 4)
        gx, _, _ = run_gpu([pool], x, [], dy, "f32", **nhwc)
        hx, _, _ = run_gpu([pool], x, [], dy, "f32", lane_exchange=-1, **nhwc)
        assert np.isfinite(gx).all() and np.array_equal(gx, hx), pool
    c, h, w, ct = 8, 9, 8, 1 << 24          # 72 pixels of 64 MiB: 4.5 GiB
    if torch.cuda.mem_get_info()[0] < (12 << 30):
        pytest.skip("needs 12 GiB of free device memory")
    layers = [wl.bn_params(c, 1), wl.relu(), wl.maxpool(3, 2, 1)]
    x, _, dy = _inputs(layers, (1, c, h, w), 5, "f32")
    st = bs.Stack(layers, (1, c, h, w), "f32").plan(**nhwc).plan_backward()
    put = lambda a: _dev(a, "f32").contiguous(memory_format=torch.channels_last)
    xd, dyd = put(x), put(dy)
    dense, _ = st.backward(xd, [], dyd)
    big = torch.empty(h * w * ct, dtype=torch.float32, device="cuda")
    big.view(h * w, ct)[:, ct - c:] = xd.permute(0, 2, 3, 1).reshape(h * w, c)
    gx = torch.empty_like(xd, memory_format=torch.channels_last)
    ws = st.workspace("cuda", backward=True)
    bs.bs_stack_backward_strided(st.handle, big.data_ptr() + 4 * (ct - c), h * w * ct, [], None, dyd.data_ptr(), 0, gx.data_ptr(), 0, [],
                                 ws.data_ptr() if ws is not None else 0, bs.bs_stack_backward_workspace_bytes(st.handle),
                                 torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(gx, dense)
    st.close()


def _run_time_lists(c):
    six = [wl.bn_params(c, 96), wl.leaky_relu(0.3), wl.clamp(-1.5, 2.0), wl.bn_params(c, 97), wl.leaky_relu(0.1), wl.bn_params(c, 98)]
    return {
        "leaky": [wl.bn_params(c, 99), wl.leaky_relu(0.1), wl.maxpool(3, 2, 1, True)],
        "six": six + [wl.maxpool(3, 2, 0, True)],
        "six_stride1": six + [wl.maxpool(3, 1, 1, True)],
        "six_behind": [wl.relu(), wl.maxpool(3, 2, 1, True)] + six,
        "relu": [wl.relu(), wl.maxpool(3, 2, 1, True)],
        "none": [wl.maxpool(3, 2, 0, True)],
        "none_stride1": [wl.maxpool(3, 1, 1, True)],
        "two_six": six + [wl.avgpool(3, 1, 1, False), wl.maxpool(3, 2, 1)] + six,
        "two_relu": [wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), wl.relu()],
        "two_counted": [wl.bn_params(c, 100), wl.relu(), wl.avgpool(3, 1, 1, False), wl.maxpool(3, 2, 1), wl.bn_params(c, 101), wl.relu()],
        "two_none": [wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1)],
    }


@pytest.mark.parametrize("layout,shape,dtype", [(l, s, d) for d in ("f32", "bf16", "f16") for l, s in (
    ("nhwc", (2, 6, 21, 19)), ("nhwc", (1, 16, 12, 24)), ("nhwc", (2, 3, 9, 61)), ("nchw", (2, 6, 21, 19)), ("nchw", (1, 2, 24, 13)),
    ("nchw", (1, 6, 425, 431)), ("nhwc", (1, 7, 425, 431)))] + [("nhwc", (1, 24, 425, 431), "f32")])
def test_strips_with_lists_read_at_run_time(layout, shape, dtype):
    """Lists of any length (more operations than the kernels hold the parameters of), a ReLU alone and none, divisors that leave out
    padding; with the picks of the forward pass and without: small stages gather kept picks, whose sums have the same order."""
    opts = dict(layout=bs.BS_LAYOUT_NHWC) if layout == "nhwc" else {}
    mf = torch.channels_last if opts else torch.contiguous_format
    for name, layers in _run_time_lists(shape[1]).items():
        label = f"run-time lists/{layout}/{name}"
        x, _, dy = _inputs(layers, shape, 31, dtype)
        x[:, :, ::2, 1::3] = 0.5
        print(f"[backward] {label} shape={shape} dtype={dtype}", flush=True)
        ref_x, _ = bw.backward_stack(layers, x, [], dy, dtype)
        st = bs.Stack(layers, shape, dtype).plan(**opts).plan_backward()
        assert bs.bs_stack_backward_num_stages(st.handle) == 1, label
        xd, dyd = (_dev(a, dtype).contiguous(memory_format=mf) for a in (x, dy))
        gx, _ = st.backward(xd, [], dyd)
        _close(gx.float().cpu().numpy(), ref_x, dtype, label)
        if st.n_idx:
            _, idx = st.run(xd)
            hx, _ = st.backward(xd, [], dyd, indices=idx)
            if dtype == "f16":  # as in test_channels_last_strips
                assert bool(((gx.float() - hx.float()).abs() <= 2.0 ** -10 * hx.float().abs() + 2.0 ** -24).all()), label
            else:
                assert torch.equal(gx, hx), label
        st.close()


def test_row_major_strips_with_offsets_beyond_4_gib():
    """Images so far apart that byte offsets need more than 32 bits, one and two pooling levels, lists compiled in and not."""
    n, c, h, w, stride = 3, 2, 9, 11, 700 << 20
    if torch.cuda.mem_get_info()[0] < (12 << 30):
        pytest.skip("needs 12 GiB of free device memory")
    big = torch.empty(2 * stride + c * h * w, dtype=torch.float32, device="cuda")
    for layers in ([wl.bn_params(c, 1), wl.relu(), wl.maxpool(3, 2, 1)], [wl.leaky_relu(0.1), wl.maxpool(3, 1, 1)],
                   [wl.bn_params(c, 2), wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), wl.bn_params(c, 3), wl.relu()],
                   [wl.avgpool(3, 1, 1, False), wl.maxpool(3, 2, 1)]):
        x, _, dy = _inputs(layers, (n, c, h, w), 5, "f32")
        st = bs.Stack(layers, (n, c, h, w), "f32").plan().plan_backward()
        xd, dyd = _dev(x, "f32"), _dev(dy, "f32")
        dense, _ = st.backward(xd, [], dyd)
        big.as_strided((n, c * h * w), (stride, 1)).copy_(xd.reshape(n, -1))
        gx = torch.empty_like(xd)
        ws = st.workspace("cuda", backward=True)
        bs.bs_stack_backward_strided(st.handle, big.data_ptr(), stride, [], None, dyd.data_ptr(), 0, gx.data_ptr(), 0, [],
                                     ws.data_ptr() if ws is not None else 0, bs.bs_stack_backward_workspace_bytes(st.handle),
                                     torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(gx, dense), [l["kind"] for l in layers]
        st.close()


def _two_level_stacks(c):
    return {
        "halo_stress": [wl.bn_params(c, 70), wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), wl.bn_params(c, 71), wl.relu()],
        "in_range_count": [wl.bn_params(c, 72), wl.relu(), wl.avgpool(3, 1, 1, False), wl.maxpool(3, 2, 1), wl.bn_params(c, 73), wl.relu()],
        "pools_only": [wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1)],
        "leaky_clamp": [wl.bn_params(c, 74), wl.leaky_relu(0.2), wl.avgpool(3, 1, 1, False), wl.maxpool(3, 2, 1), wl.clamp(-0.3, 0.6),
                        wl.bn_params(c, 75)],
        "no_list_behind": [wl.clamp(-1.0, 1.5), wl.bn_params(c, 76), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1)],
    }


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(2, 3, 56, 56), (1, 2, 12, 16), (1, 2, 61, 24), (2, 2, 7, 8), (1, 1, 1, 8), (1, 1, 2, 8), (1, 2, 5, 256),
                                   (2, 1, 70, 16), (1, 1, 90, 72)])
def test_two_pooling_levels_in_one_backward_kernel(shape, dtype):
    """Average pooling 3 x 3 / 1 / 1, then max pooling 3 x 3 / 2 / 1, with element-wise lists in front and behind: one
    stage, one kernel, no workspace -- the plane between the poolings and its gradient stay in registers.  One, two
    and more chunks of rows, odd and tiny heights, rows that fill a wave; both divisors of the average; ties in the
    max windows.  Against the oracle and against the plan of separate stages."""
    for name, layers in _two_level_stacks(shape[1]).items():
        label = f"two levels/{name}"
        x, res, dy = _inputs(layers, shape, 13, dtype)
        x[:, :, ::3, 1::4] = 0.25   # equal values: ties between neighbouring averages
        ref_x, _ = bw.backward_stack(layers, x, res, dy, dtype)
        print(f"[backward] {label} shape={shape} dtype={dtype}", flush=True)
        st = bs.Stack(layers, shape, dtype).plan().plan_backward()
        assert bs.bs_stack_backward_num_stages(st.handle) == 1 and bs.bs_stack_backward_workspace_bytes(st.handle) == 0, label
        st.close()
        gx, _, _ = run_gpu(layers, x, res, dy, dtype)
        hx, _, _ = run_gpu(layers, x, res, dy, dtype, lane_exchange=-1)
        _close(gx, ref_x, dtype, label + " grad_x")
        _close(hx, ref_x, dtype, label + " grad_x (separate stages)")
    # an Add in front of the average, or an operation between the poolings: stages of their own
    c = shape[1]
    for layers in ([wl.add(), wl.avgpool(3, 1, 1), wl.maxpool(3, 2, 1)], [wl.avgpool(3, 1, 1), wl.relu(), wl.maxpool(3, 2, 1)],
                   [wl.bn_params(c, 77), wl.avgpool(3, 1, 1), wl.maxpool(3, 1, 1)]):
        st = bs.Stack(layers, shape, dtype).plan().plan_backward()
        assert bs.bs_stack_backward_num_stages(st.handle) == 2
        st.close()
        check(layers, shape, dtype, "two levels/not fused", seed=17)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_disjoint_two_by_two_windows(dtype):
    c = 6
    for pool in (wl.maxpool(2, 2), wl.avgpool(2, 2), wl.avgpool(2, 2, 0, False)):
        layers = [wl.add(), wl.bn_params(c, 1), wl.leaky_relu(0.1), wl.add(), wl.relu(), pool, wl.bn_params(c, 2), wl.relu()]
        check(layers, (3, c, 12, 16), dtype, f"2x2 windows that tile the plane ({pool['kind']})")
        check(layers, (2, c, 13, 16), dtype, f"odd height: the general kernel ({pool['kind']})", seed=2)
        check(layers, (2, c, 12, 12), dtype, f"rows of 12: {'whole vectors' if dtype == 'f32' else 'the general kernel'}", seed=4)
    # ties: equal values in a window (after ReLU most windows of a negative plane are all zero)
    layers = [wl.relu(), wl.maxpool(2, 2)]
    x = -np.abs(wl.activation((2, c, 8, 16), 0, dtype))
    x[:, :, ::3, ::5] = 1.0
    dy = wl.activation((2, c, 4, 8), 1, dtype)
    ref, _ = bw.backward_stack(layers, x, [], dy, dtype)
    got, _, _ = run_gpu(layers, x, [], dy, dtype)
    _close(got, ref, dtype, "ties")
    # without the ReLU every tie goes to the first cell of the window
    x = np.zeros((1, c, 8, 16), np.float32)
    ref, _ = bw.backward_stack([wl.maxpool(2, 2)], x, [], dy[:1], dtype)
    got, _, _ = run_gpu([wl.maxpool(2, 2)], x, [], dy[:1], dtype)
    assert np.array_equal(got, ref.astype(np.float32))


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (1, 3, 1, 2), (2, 5, 3, 3), (1, 7, 13, 11), (3, 9, 1, 19), (2, 30, 29, 37), (1, 51, 64, 65), (2, 1, 33, 3)])
def test_channels_last_elementwise_over_the_whole_tensor(shape, dtype):
    """Channels that are no whole vectors: vectors over the whole tensor whose elements take their own channels' parameters, a rest
    of single elements; fewer channels than a vector holds, tensors smaller than one vector; lists of every kind, up to four Adds."""
    c = shape[1]
    for layers in ([wl.bn_params(c, 1), wl.relu()], [wl.bn_params(c, 2), wl.add(), wl.relu()], [wl.add(), wl.bn_params(c, 3)],
                   [wl.leaky_relu(0.1), wl.bn_params(c, 4), wl.clamp(-1.0, 1.0)], [wl.add(), wl.bn_params(c, 5), wl.add(), wl.relu(), wl.add(), wl.add()]):
        check(layers, shape, dtype, f"channels-last, flat, {[l['kind'] for l in layers]}", seed=6, layout=bs.BS_LAYOUT_NHWC)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
@pytest.mark.parametrize("shape", [(2, 8, 2, 3), (1, 8, 3, 2), (3, 16, 13, 9), (2, 8, 7, 16), (1, 24, 6, 31), (2, 8, 10, 14), (1, 3, 65, 67)])
def test_disjoint_windows_beside_a_row_or_column_left_over(shape, layout, dtype):
    """2 x 2 windows on planes that they do not tile: a lane owns a cell of the plane, the ones that the edge cuts get a gradient
    of zero.  Lists of each kind (compiled in, read at run time, none, one Add), and every tie to the first place."""
    c = shape[1]
    o = {"layout": bs.BS_LAYOUT_NHWC} if layout == "nhwc" else {}
    for pool in (wl.maxpool(2, 2), wl.avgpool(2, 2), wl.maxpool(2, 2, ceil_mode=True)):
        for layers in ([wl.bn_params(c, 1), wl.relu(), pool], [wl.leaky_relu(0.1), pool], [pool, wl.bn_params(c, 2)], [wl.add(), wl.relu(), pool]):
            check(layers, shape, dtype, f"2x2 windows beside a rest, {layout}, {[l['kind'] for l in layers]}", seed=3, **o)
    layers = [wl.maxpool(2, 2)]
    for fill in (0.0, -np.inf):
        x = np.full(shape, fill, np.float32)
        dy = wl.activation(wl.output_shape(layers, shape), 5, dtype)
        ref = np.zeros(shape, np.float32)
        ref[:, :, 0:2 * dy.shape[2]:2, 0:2 * dy.shape[3]:2] = dy
        got, _, _ = run_gpu(layers, x, [], dy, dtype, **o)
        assert np.array_equal(got, ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("name", list(_stacks(3)))
def test_channels_last_plans(name, dtype):
    """The same gradients from channels-last tensors: channel counts that give whole 128-bit vectors
    for both element sizes (16), for float32 only (12) and for neither (5)."""
    for c, shape in ((16, (2, 16, 12, 16)), (12, (2, 12, 13, 11)), (5, (3, 5, 12, 16))):
        if name.startswith("global") and shape[2:] != (12, 16):
            continue
        check(_stacks(c)[name], shape, dtype, f"{name}/channels-last C={c}", seed=c, layout=bs.BS_LAYOUT_NHWC)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_channels_last_disjoint_two_by_two_windows(dtype):
    for c in (8, 24, 6):
        for pool in (wl.maxpool(2, 2), wl.avgpool(2, 2)):
            layers = [wl.add(), wl.bn_params(c, 1), wl.leaky_relu(0.1), wl.add(), wl.relu(), pool, wl.bn_params(c, 2), wl.relu()]
            check(layers, (3, c, 12, 10), dtype, f"channels-last 2x2 windows C={c} ({pool['kind']})", layout=bs.BS_LAYOUT_NHWC)
            check(layers, (2, c, 7, 10), dtype, f"channels-last odd height C={c} ({pool['kind']})", seed=2, layout=bs.BS_LAYOUT_NHWC)
    layers = [wl.relu(), wl.maxpool(2, 2)]  # ties
    x = -np.abs(wl.activation((2, 8, 8, 6), 0, dtype))
    x[:, ::3, ::3, ::5] = 1.0
    dy = wl.activation((2, 8, 4, 3), 1, dtype)
    ref, _ = bw.backward_stack(layers, x, [], dy, dtype)
    got, _, _ = run_gpu(layers, x, [], dy, dtype, layout=bs.BS_LAYOUT_NHWC)
    _close(got, ref, dtype, "channels-last ties")


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_planes_that_are_no_whole_number_of_vectors(dtype):
    """Element-wise stages on 14 x 14 and 7 x 7 planes: vectors run over the whole tensor and may begin in
    one plane (channel, image) and end in the next."""
    for c, shape in ((5, (2, 5, 14, 14)), (8, (3, 8, 7, 7)), (3, (8, 3, 3, 3))):
        layers = [wl.bn_params(c, 1), wl.add(), wl.leaky_relu(0.2), wl.bn_params(c, 2), wl.add(), wl.relu()]
        check(layers, shape, dtype, f"vectors over plane boundaries {shape}")
    # behind a pooling stage as well (the element-wise stage after the pool is the flat one)
    layers = [wl.bn_params(6, 3), wl.relu(), wl.maxpool(2, 2), wl.bn_params(6, 4), wl.add(), wl.relu()]
    check(layers, (4, 6, 28, 28), dtype, "flat stage behind a pooling stage")


def _random_stack(rng, c, h, w):
    """A random valid stack of 1..9 layers (all layer kinds, odd windows, strides, padding, ceil mode, up to four
    residual operands); every pooling output at least 1 x 1."""
    layers, adds = [], 0
    kinds = ["bn", "relu", "leaky", "clamp", "add", "max", "max", "avg", "avg"]
    for _ in range(int(rng.integers(1, 10))):
        kind = rng.choice(kinds)
        if kind in ("max", "avg"):
            k = (int(rng.integers(1, 6)), int(rng.integers(1, 6)))
            st = (int(rng.integers(1, 4)), int(rng.integers(1, 4)))
            p = (int(rng.integers(0, k[0] // 2 + 1)), int(rng.integers(0, k[1] // 2 + 1)))
            ceil = bool(rng.integers(0, 3) == 0)
            ho, wo = wl.pool_out(h, k[0], st[0], p[0], ceil), wl.pool_out(w, k[1], st[1], p[1], ceil)
            if h + 2 * p[0] < k[0] or w + 2 * p[1] < k[1] or ho < 1 or wo < 1:
                continue
            layers.append(wl.maxpool(k, st, p, False, ceil_mode=ceil) if kind == "max"
                          else wl.avgpool(k, st, p, bool(rng.integers(0, 2)), ceil_mode=ceil))
            h, w = ho, wo
        elif kind == "bn":
            layers.append(wl.bn_params(c, int(rng.integers(0, 1000))))
        elif kind == "relu":
            layers.append(wl.relu())
        elif kind == "leaky":
            layers.append(wl.leaky_relu(float(rng.choice([0.01, 0.1, 0.3]))))
        elif kind == "clamp":
            layers.append(wl.clamp(float(rng.choice([-1.0, 0.0, -0.25])), float(rng.choice([0.5, 1.0, 6.0]))))
        elif adds < 4:
            layers.append(wl.add())
            adds += 1
    return layers or [wl.relu()]


@pytest.mark.parametrize("seed", range(8))
def test_random_stacks_match_the_oracle(seed):
    """Seeded random stacks on random small shapes, all three storage types, both memory layouts."""
    rng = np.random.default_rng(5000 + seed)
    for case in range(10):
        n, c = int(rng.integers(1, 4)), int(rng.choice([1, 3, 4, 5, 8, 16]))
        h = int(rng.choice([5, 7, 8, 12, 16, 20, 24, 31]))
        w = int(rng.choice([5, 8, 9, 12, 16, 24, 32, 40]))
        dtype = ("f32", "bf16", "f16")[(seed + case) % 3]
        layers = _random_stack(rng, c, h, w)
        opts = [dict(), dict(layout=bs.BS_LAYOUT_NHWC), dict(jit=-1)][int(rng.integers(0, 3))]
        check(layers, (n, c, h, w), dtype, f"random/{seed}.{case} {[l['kind'] for l in layers]}", seed=100 * seed + case, **opts)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_sixteen_bit_rows_of_four_mod_eight(dtype):
    """28 x 28 and 12-wide planes with 16-bit storage: one 64-bit vector per lane (2 x 2 windows owned whole,
    the 3 x 3 gathers with the window compiled in, the generic gather), not one cell per lane."""
    c = 6
    for layers in ([wl.bn_params(c, 1), wl.relu(), wl.maxpool(2, 2)],
                   [wl.add(), wl.bn_params(c, 2), wl.relu(), wl.avgpool(2, 2), wl.bn_params(c, 3)],
                   [wl.bn_params(c, 4), wl.relu(), wl.maxpool(3, 2, 1)],
                   [wl.avgpool(3, 1, 1, True), wl.add(), wl.maxpool(3, 1, 1), wl.relu()],
                   [wl.leaky_relu(0.1), wl.maxpool((2, 4), (2, 4)), wl.add()]):
        check(layers, (2, c, 28, 28), dtype, f"28 x 28 {[l['kind'] for l in layers]}")
        check(layers, (3, c, 10, 12), dtype, f"10 x 12 {[l['kind'] for l in layers]}", seed=5)


def test_long_lists_are_cut_into_stages():
    c = 4
    # 20 element-wise operations (more than one argument block holds), 6 Adds (more than one stage's residual slots)
    layers = []
    for i in range(6):
        layers += [wl.bn_params(c, 20 + i), wl.add(), wl.leaky_relu(0.3)]
    layers += [wl.relu(), wl.clamp(-1.0, 2.0)]
    stages = check(layers, (2, c, 8, 8), "f32", "20 element-wise operations, 6 Adds")
    assert stages >= 2
    layers = layers + [wl.maxpool(2, 2)] + layers
    check(layers, (2, c, 8, 8), "f32", "the same around a pooling operation")


def test_gradients_that_are_not_wanted_are_not_written():
    layers = [wl.bn_params(4, 1), wl.add(), wl.relu(), wl.maxpool(2, 2), wl.add(), wl.leaky_relu(0.1)]
    shape = (2, 4, 8, 8)
    x, res, dy = _inputs(layers, shape, 0, "f32")
    ref_x, ref_res = bw.backward_stack(layers, x, res, dy)
    gx, gres, _ = run_gpu(layers, x, res, dy, "f32", need_input=False, need_res=[True, False])
    assert gx is None and gres[1] is None
    _close(gres[0], ref_res[0], "f32", "only grad_residual[0]")
    gx, gres, _ = run_gpu(layers, x, res, dy, "f32", need_input=True, need_res=[False, True])
    assert gres[0] is None
    _close(gx, ref_x, "f32", "grad_x")
    _close(gres[1], ref_res[1], "f32", "grad_residual[1]")


def test_single_stage_stacks_need_no_workspace_and_max_pooling_does():
    st = bs.Stack([wl.bn_params(8, 1), wl.add(), wl.relu()], (2, 8, 8, 8), "f32").plan().plan_backward()
    assert bs.bs_stack_backward_num_stages(st.handle) == 1 and bs.bs_stack_backward_workspace_bytes(st.handle) == 0
    st.close()
    st = bs.Stack([wl.bn_params(8, 1), wl.relu(), wl.avgpool(2, 2)], (2, 8, 8, 8), "f32").plan().plan_backward()
    assert bs.bs_stack_backward_num_stages(st.handle) == 1 and bs.bs_stack_backward_workspace_bytes(st.handle) == 0
    st.close()
    # disjoint 2 x 2 windows: the kernel finds the picks itself
    st = bs.Stack([wl.bn_params(8, 1), wl.relu(), wl.maxpool(2, 2)], (2, 8, 8, 8), "f32").plan().plan_backward()
    assert bs.bs_stack_backward_num_stages(st.handle) == 1 and bs.bs_stack_backward_workspace_bytes(st.handle) == 0
    st.close()
    # overlapping 3 x 3 windows on rows of whole vectors: the same, the lanes of a row exchanging picks in their edge columns
    st = bs.Stack([wl.bn_params(8, 1), wl.relu(), wl.maxpool(3, 2, 1)], (2, 8, 8, 8), "f32").plan().plan_backward()
    assert bs.bs_stack_backward_num_stages(st.handle) == 1 and bs.bs_stack_backward_workspace_bytes(st.handle) == 0
    st.close()
    # ... on other rows as well, as strips of columns
    st = bs.Stack([wl.bn_params(8, 1), wl.relu(), wl.maxpool(3, 2, 1)], (2, 8, 8, 10), "f32").plan().plan_backward()
    assert bs.bs_stack_backward_num_stages(st.handle) == 1 and bs.bs_stack_backward_workspace_bytes(st.handle) == 0
    st.close()
    # ... and with recorded picks where those kernels do not apply or are switched off
    for layers, shape, opts in (([wl.bn_params(8, 1), wl.relu(), wl.maxpool(3, 2, 1)], (2, 8, 8, 8), dict(lane_exchange=-1)),
                                ([wl.bn_params(8, 1), wl.relu(), wl.maxpool(3, 2, 1)], (2, 8, 8, 10), dict(lane_exchange=-1)),
                                ([wl.bn_params(8, 1), wl.add(), wl.relu(), wl.maxpool(3, 2, 1)], (2, 8, 8, 10), {}),
                                ([wl.bn_params(8, 1), wl.relu(), wl.maxpool(5, 2, 2)], (2, 8, 8, 8), {})):
        st = bs.Stack(layers, shape, "f32").plan(**opts).plan_backward()
        out = wl.output_shape(layers, shape)
        assert bs.bs_stack_backward_workspace_bytes(st.handle) >= int(np.prod(out)) * 4  # the picks
        st.close()


def test_argument_errors():
    layers = [wl.bn_params(8, 1), wl.relu(), wl.maxpool(3, 2, 1)]
    st = bs.Stack(layers, (2, 8, 8, 8), "f32").plan(lane_exchange=-1)  # recorded picks: a workspace
    x = torch.zeros(2, 8, 8, 8, device="cuda")
    dy = torch.zeros(2, 8, 4, 4, device="cuda")
    gx = torch.empty_like(x)
    with pytest.raises(bs.BrainSlugError) as e:  # no backward plan yet
        bs.bs_stack_backward(st.handle, x.data_ptr(), [], None, dy.data_ptr(), gx.data_ptr(), [], 0, 0, 0)
    assert e.value.status == bs.STATUS_BY_NAME["BS_ERR_NOT_PLANNED"]
    st.plan_backward()
    n = bs.bs_stack_backward_workspace_bytes(st.handle)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    with pytest.raises(bs.BrainSlugError) as e:
        bs.bs_stack_backward(st.handle, x.data_ptr(), [], None, dy.data_ptr(), gx.data_ptr(), [], ws.data_ptr(), n - 1, 0)
    assert e.value.status == bs.STATUS_BY_NAME["BS_ERR_WORKSPACE"]
    with pytest.raises(bs.BrainSlugError) as e:  # the gradient over the input
        bs.bs_stack_backward(st.handle, x.data_ptr(), [], None, dy.data_ptr(), x.data_ptr(), [], ws.data_ptr(), n, 0)
    assert e.value.status == bs.STATUS_BY_NAME["BS_ERR_ALIAS"]
    with pytest.raises(bs.BrainSlugError) as e:
        bs.bs_stack_backward(st.handle, x.data_ptr() + 4, [], None, dy.data_ptr(), gx.data_ptr(), [], ws.data_ptr(), n, 0)
    assert e.value.status == bs.STATUS_BY_NAME["BS_ERR_ALIGN"]
    with pytest.raises(bs.BrainSlugError) as e:
        bs.bs_stack_backward(st.handle, 0, [], None, dy.data_ptr(), gx.data_ptr(), [], ws.data_ptr(), n, 0)
    assert e.value.status == bs.STATUS_BY_NAME["BS_ERR_NULL"]
    # a new forward plan drops the backward plan
    st.plan(lane_exchange=-1)
    assert bs.bs_stack_backward_num_stages(st.handle) == -1
    st.close()


@pytest.mark.parametrize("dtype,layout", [("f32", 0), ("f16", 0), ("bf16", 1)])
def test_saved_indices_replace_the_recomputation(dtype, layout):
    """The picks kept from the forward pass (index outputs of bs_stack_run) give the same gradient as the
    recomputed ones, bit for bit; for picks of an inner pooling layer they are simply not needed."""
    mf = torch.channels_last if layout else torch.contiguous_format
    for layers, shape in (([wl.bn_params(8, 1), wl.relu(), wl.maxpool(3, 2, 1, True)], (2, 8, 16, 16)),
                          ([wl.maxpool(3, 1, 1, True), wl.bn_params(8, 2), wl.relu(), wl.maxpool(3, 2, 1, True)], (2, 8, 16, 16))):
        x, res, dy = _inputs(layers, shape, 3, dtype)
        st = bs.Stack(layers, shape, dtype).plan(layout=layout).plan_backward()
        put = lambda a: _dev(a, dtype).contiguous(memory_format=mf)
        xd, dyd = put(x), put(dy)
        _, idx = st.run(xd, [])
        a, _ = st.backward(xd, [], dyd)
        b, _ = st.backward(xd, [], dyd, indices=idx)
        c, _ = st.backward(xd, [], dyd, indices=[None] * (len(idx) - 1) + [idx[-1]])
        torch.cuda.synchronize()
        assert torch.equal(a, b) and torch.equal(a, c)
        ref, _ = bw.backward_stack(layers, x, [], dy, dtype)
        _close(b.float().cpu().numpy(), ref, dtype, "saved indices")
        # wrong picks are trusted, and only misroute: everything to cell 0 of each plane
        zeros = [torch.zeros_like(t) for t in idx]
        z, _ = st.backward(xd, [], dyd, indices=zeros)
        torch.cuda.synchronize()
        assert torch.isfinite(z.float()).all()
        st.close()


def test_forward_and_backward_can_be_captured_in_a_hip_graph_and_replayed():
    """bs_stack_backward only enqueues kernels (its recomputation passes included): a training step's
    forward and backward pass of a two-stage stack are captured once and replayed with new operands,
    eager calls in between; every replay matches the oracle."""
    c = 6
    layers = [wl.bn_params(c, 5), wl.add(), wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), wl.bn_params(c, 6), wl.relu()]
    shape, oshape = (2, c, 24, 32), (2, c, 12, 16)
    st = bs.Stack(layers, shape, "f32").plan().plan_backward()
    assert bs.bs_stack_backward_num_stages(st.handle) == 2  # BatchNorm, ReLU behind the max pooling join its stage
    x_s, r_s, dy_s = (torch.zeros(sh, device="cuda") for sh in (shape, shape, oshape))
    out, _ = st.alloc_outputs("cuda", False)
    gx, gr = torch.empty_like(x_s), torch.empty_like(r_s)
    n = bs.bs_stack_backward_workspace_bytes(st.handle)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    st.workspace("cuda")

    def step():
        stream = torch.cuda.current_stream().cuda_stream
        st.run(x_s, [r_s], out=out, indices=[])
        bs.bs_stack_backward(st.handle, x_s.data_ptr(), [r_s.data_ptr()], None, dy_s.data_ptr(), gx.data_ptr(), [gr.data_ptr()],
                             ws.data_ptr(), n, stream)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()  # warm-up outside the capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):
        x, r, dy = wl.activation(shape, 70 + rep), wl.activation(shape, 80 + rep), wl.activation(oshape, 90 + rep)
        x_s.copy_(torch.from_numpy(x)); r_s.copy_(torch.from_numpy(r)); dy_s.copy_(torch.from_numpy(dy))
        gx.zero_(); gr.zero_(); ws.zero_()
        graph.replay()
        torch.cuda.synchronize()
        ref_x, (ref_r,) = bw.backward_stack(layers, x, [r], dy)
        _close(gx.cpu().numpy(), ref_x, "f32", f"replay {rep} grad_x")
        _close(gr.cpu().numpy(), ref_r, "f32", f"replay {rep} grad_residual")
        a, (b,) = st.backward(x_s, [r_s], dy_s)  # eager call between the replays
        torch.cuda.synchronize()
        assert torch.equal(a, gx) and torch.equal(b, gr)
    del graph
    st.close()


def _slice_stacks(c, h, w):
    return {
        "bn_add_relu": [wl.bn_params(c, 60), wl.add(), wl.relu()],                                   # element-wise
        "max2": [wl.bn_params(c, 61), wl.relu(), wl.maxpool(2, 2)],                                  # windows that tile the plane
        "stem": [wl.bn_params(c, 62), wl.relu(), wl.maxpool(3, 2, 1)],                               # lanes walk the rows
        "avg3s1": [wl.bn_params(c, 63), wl.relu(), wl.avgpool(3, 1, 1)],                             # gather, compiled window
        "max5": [wl.relu(), wl.maxpool(5, 2, 2)],                                                    # gather, recorded picks
        "halo_stress": [wl.bn_params(c, 64), wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), wl.bn_params(c, 65), wl.relu()],
        "head": [wl.bn_params(c, 66), wl.relu(), wl.avgpool((h, w), (h, w), 0)],
    }


@pytest.mark.parametrize("layout", [bs.BS_LAYOUT_NCHW, bs.BS_LAYOUT_NHWC])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(2, 8, 12, 16), (3, 16, 7, 7), (2, 8, 13, 11)])
def test_gradients_of_channel_slices_are_read_and_written_in_place(shape, dtype, layout):
    """bs_stack_backward_strided: the input, the upstream gradient and the input's gradient as channel
    slices of larger tensors (eight channels on either side).  The same bits as the dense call, the oracle's
    values, and nothing outside the slices touched (guard values in the gradient buffer, NaN around the inputs)."""
    n, c, h, w = shape
    td = TORCH[dtype]
    mf = torch.channels_last if layout == bs.BS_LAYOUT_NHWC else torch.contiguous_format
    stride_of = bs.batch_stride_nhwc if layout == bs.BS_LAYOUT_NHWC else bs.batch_stride
    for name, layers in _slice_stacks(c, h, w).items():
        print(f"[backward] slices/{name} shape={shape} dtype={dtype} layout={layout}", flush=True)
        x, res, dy = _inputs(layers, shape, 11, dtype)
        ref_x, ref_res = bw.backward_stack(layers, x, res, dy, dtype)
        st = bs.Stack(layers, shape, dtype).plan(layout=layout).plan_backward()
        put = lambda a: _dev(a, dtype).contiguous(memory_format=mf)
        xd, dyd, resd = put(x), put(dy), [put(r) for r in res]
        dense_gx, dense_gres = st.backward(xd, resd, dyd)
        big = lambda t, fill: torch.full((n, t.shape[1] + 16) + tuple(t.shape[2:]), fill, dtype=td, device="cuda").contiguous(memory_format=mf)
        big_x, big_dy, guard = big(xd, float("nan")), big(dyd, float("nan")), 4321.0
        big_gx = big(xd, guard)
        big_x[:, 8:8 + c] = xd
        big_dy[:, 8:8 + c] = dyd
        xs, dys, gxs = big_x[:, 8:8 + c], big_dy[:, 8:8 + c], big_gx[:, 8:8 + c]
        gres = [torch.empty_like(r) for r in resd]
        ws = st.workspace("cuda", backward=True)
        nws = bs.bs_stack_backward_workspace_bytes(st.handle)
        bs.bs_stack_backward_strided(st.handle, xs.data_ptr(), stride_of(xs), [r.data_ptr() for r in resd], None, dys.data_ptr(),
                                     stride_of(dys), gxs.data_ptr(), stride_of(gxs), [g.data_ptr() for g in gres],
                                     ws.data_ptr() if nws else 0, nws, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(gxs, dense_gx), name
        for a, b in zip(gres, dense_gres):
            assert torch.equal(a, b), name
        _close(gxs.float().cpu().numpy(), ref_x, dtype, f"slices/{name} grad_x")
        assert bool((big_gx[:, :8] == guard).all()) and bool((big_gx[:, 8 + c:] == guard).all()), name
        # strides that are no channel slice, and outputs over inputs, are refused
        with pytest.raises(bs.BrainSlugError) as e:
            bs.bs_stack_backward_strided(st.handle, xs.data_ptr(), c * h * w - 8, [r.data_ptr() for r in resd], None, dys.data_ptr(),
                                         stride_of(dys), gxs.data_ptr(), stride_of(gxs), [g.data_ptr() for g in gres],
                                         ws.data_ptr() if nws else 0, nws, 0)
        assert e.value.status == bs.STATUS_BY_NAME["BS_ERR_SHAPE"]
        with pytest.raises(bs.BrainSlugError) as e:
            bs.bs_stack_backward_strided(st.handle, xs.data_ptr(), stride_of(xs), [r.data_ptr() for r in resd], None, dys.data_ptr(),
                                         stride_of(dys), xs.data_ptr(), stride_of(xs), [g.data_ptr() for g in gres],
                                         ws.data_ptr() if nws else 0, nws, 0)
        assert e.value.status == bs.STATUS_BY_NAME["BS_ERR_ALIAS"]
        st.close()


@pytest.mark.parametrize("shape,layout", [((160, 24, 49, 51), bs.BS_LAYOUT_NHWC), ((1100, 7, 33, 38), bs.BS_LAYOUT_NHWC), ((80, 32, 47, 43), bs.BS_LAYOUT_NCHW),
                                          ((20, 5, 224, 222), bs.BS_LAYOUT_NCHW), ((40, 96, 56, 56), bs.BS_LAYOUT_NCHW)])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_two_levels_in_small_and_large_tensors(shape, layout, dtype):
    """The kernels of two pooling levels choose strips of four or eight columns, and chunks of rows, by the tensor's size: images of a large tensor have the gradients
    that they have in a small one, bit for bit (every sum has one order)."""
    c = shape[1]
    layers = [wl.bn_params(c, 910), wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), wl.bn_params(c, 911), wl.relu()]
    mf = torch.channels_last if layout == bs.BS_LAYOUT_NHWC else torch.contiguous_format
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(shape, generator=gen, device="cuda").to(dt).contiguous(memory_format=mf)
    got = []
    for images in (shape[0], 2):
        st = bs.Stack(layers, (images, *shape[1:]), dtype).plan(layout=layout)
        st.plan_backward()
        part = x[:images].contiguous(memory_format=mf)
        y, _ = st.run(part)
        if not got:
            dy = torch.randn(tuple(y.shape), generator=gen, device="cuda").to(dt).contiguous(memory_format=mf)
        gx, _ = st.backward(part, [], dy[:images].contiguous(memory_format=mf))
        got.append(gx[:2].clone())
        st.close()
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("shape,layout", [((160, 24, 49, 51), bs.BS_LAYOUT_NHWC), ((1100, 7, 33, 38), bs.BS_LAYOUT_NHWC), ((80, 32, 47, 43), bs.BS_LAYOUT_NCHW)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_two_levels_round_alike_in_strips_of_any_width(shape, layout, dtype):
    """All images of a large tensor (strips of eight columns) against the same images in quarters (strips of four): the gradients' last product and its conversion to
    16 bits are two roundings in every column, also where an instruction exists that does both in one."""
    c = shape[1]
    layers = [wl.bn_params(c, 910), wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), wl.bn_params(c, 911), wl.relu()]
    mf = torch.channels_last if layout == bs.BS_LAYOUT_NHWC else torch.contiguous_format
    dt = torch.float16 if dtype == "f16" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn(shape, generator=gen, device="cuda").to(dt).contiguous(memory_format=mf)
    dy = None

    def gradient(part, images):
        nonlocal dy
        st = bs.Stack(layers, tuple(part.shape), dtype).plan(layout=layout)
        st.plan_backward()
        if dy is None:
            dy = torch.randn(tuple(st.run(part)[0].shape), generator=gen, device="cuda").to(dt).contiguous(memory_format=mf)
        gx = st.backward(part, [], dy[images].clone(memory_format=mf))[0].clone()
        st.close()
        return gx

    whole = gradient(x, slice(None))
    q = shape[0] // 4
    for i in range(0, shape[0], q):
        part = slice(i, i + q)
        assert torch.equal(whole[part], gradient(x[part].clone(memory_format=mf), part)), i  # (clones begin at aligned addresses)


def test_repeated_calls_give_identical_bits():
    """A gather has one summation order: two runs agree bit for bit (no atomics anywhere)."""
    layers = _stacks(6)["halo_stress"]
    x, res, dy = _inputs(layers, (4, 6, 28, 28), 1, "f32")
    a, _, _ = run_gpu(layers, x, res, dy, "f32")
    b, _, _ = run_gpu(layers, x, res, dy, "f32")
    assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("name,dtype,layout", [("vgg_a", "f32", 0), ("vgg_c", "bf16", 0), ("resnet_tail", "f16", 0), ("halo_stress", "f32", 0), ("halo_stress", "bf16", 0),
                                               ("resnet_stem", "f16", 0), ("vgg_a", "f32", 1), ("resnet_stem", "f16", 1),
                                               ("resnet_tail", "bf16", 1), ("densenet_trans", "f32", 1)])
def test_benchmark_sizes_on_sampled_images(name, dtype, layout):
    """Whole tensors at the benchmark sizes on the GPU, in the launch configuration the benchmark times,
    row-major and channels-last; images are independent, so the oracle checks a sample of them (first,
    one inside, last) in full."""
    layers, shape, _ = wl.build(name, 0, None, False)
    print(f"[backward] {name} full size shape={shape} dtype={dtype} layout={layout}", flush=True)
    td = TORCH[dtype]
    mf = torch.channels_last if layout else torch.contiguous_format
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda sh: torch.randn(sh, device="cuda", generator=g).to(td).contiguous(memory_format=mf)
    x = rnd(shape)
    out_shape = wl.output_shape(layers, shape)
    dy = rnd(out_shape)
    res = [rnd(s) for s in wl.residual_shapes(layers, shape)]
    st = bs.Stack(layers, shape, dtype).plan(layout=layout).plan_backward()
    gx, gres = st.backward(x, res, dy)
    torch.cuda.synchronize()
    for n in (0, shape[0] // 2 + 1, shape[0] - 1):
        sl = slice(n, n + 1)
        ref_x, ref_res = bw.backward_stack(layers, x[sl].float().cpu().numpy(), [r[sl].float().cpu().numpy() for r in res],
                                           dy[sl].float().cpu().numpy(), dtype)
        _close(gx[sl].float().cpu().numpy(), ref_x, dtype, f"{name} image {n} grad_x")
        for i, r in enumerate(ref_res):
            _close(gres[i][sl].float().cpu().numpy(), r, dtype, f"{name} image {n} grad_residual[{i}]")
    st.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(2, 3, 7, 5), (1, 6, 3, 3), (1, 2, 4, 1), (3, 16, 30, 9), (5, 7, 191, 170), (9, 64, 65, 62)])
def test_picks_found_as_greatest_keys(shape, dtype):
    """[BatchNorm -> ReLU or ReLU, max pooling 3 x 3] in the strip kernels whose maxima are keys of value and place: one and two channels per
    lane (odd and even channel counts), strips of two and of four columns (the small and the large shapes), planes narrower than a strip,
    equal maxima (the first in row-major order gets the gradient), windows of nothing but zeros (no gradient), infinite maxima."""
    c = shape[1]
    big = int(np.prod(shape)) > 100000
    for (s, p), lead in zip(((2, 1), (2, 0), (1, 1), (1, 0)), ([wl.bn_params(c, 41), wl.relu()], [wl.relu()], [wl.relu()], [wl.bn_params(c, 42), wl.relu()])):
        if shape[2] + 2 * p < 3 or shape[3] + 2 * p < 3 or (big and (s, p) in ((2, 0), (1, 0))):
            continue
        layers = lead + [wl.maxpool(3, s, p)]
        rng = np.random.default_rng(7)
        x = rng.choice(np.array([-2.0, -0.5, 0.0, 0.5, 0.5, 1.5], np.float32), shape)
        x[:, :, : shape[2] // 3] = -1.0  # ReLU cuts off whole windows
        x.flat[:: 97] = np.inf
        dy = rng.integers(-8, 9, wl.output_shape(layers, shape)).astype(np.float32)  # sums of these are exact
        ref, _ = bw.backward_stack(layers, x, [], dy, dtype)
        for opts in (dict(layout=bs.BS_LAYOUT_NHWC), dict()):
            gx, _, stages = run_gpu(layers, x, [], dy, dtype, **opts)
            assert stages == 1
            _close(gx, ref, dtype, f"keys {shape} {dtype} s{s} p{p} {opts}")


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(2, 8, 13, 11), (1, 5, 4, 31), (1, 16, 33, 9)])
def test_windows_of_averages_that_round_to_zero(shape, dtype):
    """ReLU, average, maximum in one kernel on cells so small that every average rounds to 0 while the cells are positive: a window's
    gradient goes to its first cell inside the plane all the same, also in the windows that begin above it."""
    tiny = {"f32": 2.0 ** -149, "bf16": 2.0 ** -133, "f16": 2.0 ** -24}[dtype]
    bn = wl.bn_params(shape[1], 51)
    bn["beta"] = np.abs(bn["beta"]) + 2.0 + np.abs(bn["mean"] * bn["gamma"]) / np.sqrt(bn["var"] + bn["eps"])  # the ReLU behind it passes everything
    bn["beta"] = bn["beta"].astype(np.float32)
    layers = [wl.relu(), wl.avgpool(3, 1, 1, True), wl.maxpool(3, 2, 1), bn, wl.relu()]
    rng = np.random.default_rng(11)
    x = np.full(shape, -1.0, np.float32)
    x[:, :, ::3, ::3] = tiny  # one in nine: no average reaches half the smallest value
    dy = rng.integers(-8, 9, wl.output_shape(layers, shape)).astype(np.float32)
    ref, _ = bw.backward_stack(layers, x, [], dy, dtype)
    assert np.abs(ref[:, :, 0]).max() > 0.0
    for opts in (dict(layout=bs.BS_LAYOUT_NHWC), dict()):
        gx, _, stages = run_gpu(layers, x, [], dy, dtype, **opts)
        assert stages == 1
        _close(gx, ref, dtype, f"averages of 0, {shape} {dtype} {opts}")
