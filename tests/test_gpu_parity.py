"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element, on the
same seeded inputs.  Integer products bit-exact (with counted rounding flips of value-pruned
sets, see compare.py); fp32 tensors within 1e-4 * max|tensor| of the fp64 oracle."""
import dataclasses
import sys

import numpy as np
import pytest

import compare as cmp
from oracle.oracle import Oracle
from paper_2303_04670_amd import evconv as ev
from paper_2303_04670_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-4


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def run_stream(net, x0, inputs, kind, check_nodes_at=None, tol=TOL, exact_sets=False, max_flips=0,
               fp32_oracle=False, label="", frobenius=False):
    """kind: 'frame' or 'increment'.  check_nodes_at: steps (1-based) at which every node is
    compared (None = every step); outputs and the input stage are compared at every step."""
    gpu = ev.EvConvNet(net)
    ora = Oracle(net, fp32_state=fp32_oracle)
    rep = cmp.Report()
    gpu.reset(_dev(x0))
    ora.reset(x0)
    cmp.compare_outputs(gpu, ora, rep, tol)
    for i in range(len(net.nodes)):
        if ora.tensor(i, 0).size:
            z = gpu.state(i, ev.STATE_Z).astype(np.float64)
            zr = ora.z(i)
            assert np.abs(z - zr).max() <= tol * max(np.abs(zr).max(), 1e-30), f"reset: node {i} z"
    for step, inp in enumerate(inputs, 1):
        if kind == "frame":
            gpu.step_frame(_dev(inp))
            ora.step_frame(inp)
        else:
            gpu.step(_dev(inp))
            ora.step_increment(inp)
        cmp.compare_input_stage(gpu, ora, rep)
        cmp.compare_outputs(gpu, ora, rep, tol)
        if check_nodes_at is None or step in check_nodes_at:
            for i in range(len(net.nodes)):
                cmp.compare_node(gpu, ora, i, rep, tol=tol, exact_sets=exact_sets, frobenius=frobenius)
        if step % 10 == 0:
            _say(f"[{label}] step {step}: flips {rep.flips} max rel z err {rep.max_rel_z:.2e} y err {rep.max_rel_y:.2e}")
    _say(f"[{label}] done: flips {rep.flips} (allowed {max_flips}) max rel z err {rep.max_rel_z:.2e} y err {rep.max_rel_y:.2e}"
         + (f" increment err (own norm) {rep.max_rel_inc:.2e}" if frobenius else ""))
    assert rep.flips <= max_flips, f"{rep.flips} rounding flips of value-pruned sets: {rep.flips_by_node}"
    gpu.destroy()
    return rep


def test_workload1_single_conv_10_steps():
    _say("workload 1: single conv3x3 16->16 on 16x64x64, 10 increments at 2 %")
    net = wl.net_single_conv()
    x0, incs = wl.stream_line_increments()
    rep = run_stream(net, x0, incs, "increment", label="w1", max_flips=2)
    assert rep.nodes_checked == 10


def test_workload2_conv_stack_100_steps():
    _say("workload 2: 4-layer conv stack on 5x180x240, 100 frames at 1-5 %")
    net = wl.net_conv_stack()
    frames = list(wl.stream_voxel(1002, 180, 240, 100, wl.density_sweep_1_5))
    run_stream(net, frames[0], frames[1:], "frame", check_nodes_at={1, 2, 3, 25, 50, 75, 100}, label="w2",
               max_flips=8)


@pytest.mark.parametrize("seed", [7, 8, 9])
def test_every_op_small_ragged_graph(seed):
    _say(f"small graph touching every op, seed {seed}")
    kw = {} if seed == 7 else dict(in_c=2, h=9, w=19, bias=(seed == 8))
    net = wl.net_random_small(seed, **kw)
    rng = np.random.default_rng(seed)
    x0 = rng.standard_normal((net.in_c, net.in_h, net.in_w)).astype(np.float32)
    frames, x = [], x0
    for t in range(12):
        m = rng.random((net.in_h, net.in_w)) < (0.02 + 0.08 * (t % 4))
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m[None]).astype(np.float32)
        frames.append(x)
    run_stream(net, x0, frames, "frame", label=f"small{seed}", max_flips=4)


def test_unet_reduced_all_nodes_every_step():
    _say("UNet depth net, reduced 5x64x96 width 8, 30 frames, all nodes every step")
    net = wl.net_unet_depth(1003, h=64, w=96, width=8)
    frames = list(wl.stream_voxel(1003, 64, 96, 30, 0.02, n_prim=6))
    run_stream(net, frames[0], frames[1:], "frame", label="unet-small", max_flips=40)


def test_unet_full_width_reduced_size_matrix_core_layers():
    _say("UNet depth net, full width (32..256 channels) on 5x64x96: matrix-core conv layers, all nodes every step")
    net = wl.net_unet_depth(1003, h=64, w=96)
    g = ev.EvConvNet(net)
    names = [g.kernel_name(i) for i in range(len(net.nodes))]
    g.destroy()
    assert names.count("conv_mfma_f32") == 10 and names[0] == "conv_narrow_mfma_f32" and names[-1] == "conv_pointwise_f32", names
    assert names.count("fused_into_conv_epilogue") == 6, names   # 2 residual adds + 4 skip adds
    # the three x2 up-samplings: only the last one's stored tensor (32 x 48) has tiles away from the border
    assert names.count("fused_into_conv_gather") == 2 and names.count("fused_into_conv_weights") == 1, names
    frames = list(wl.stream_voxel(1003, 64, 96, 20, 0.02, n_prim=6))
    run_stream(net, frames[0], frames[1:], "frame", label="unet-wide", max_flips=40)


def test_unet_full_width_without_epilogue_fusion():
    """The same graph with ADD nodes run by their own kernels instead of the conv epilogues."""
    _say("UNet depth net, full width on 5x64x96, ADD nodes unfused")
    net = wl.net_unet_depth(1003, h=64, w=96)
    g = ev.EvConvNet(net, flags=ev.FLAG_NO_FUSION)
    names = [g.kernel_name(i) for i in range(len(net.nodes))]
    g.destroy()
    assert not any(nm.startswith("fused_into_") for nm in names), names
    frames = list(wl.stream_voxel(1003, 64, 96, 8, 0.02, n_prim=6))
    run_stream(net, frames[0], frames[1:], "frame", label="unet-wide-unfused", max_flips=40)


def test_unet_bf16_matrix_core_variant_reduced():
    """bf16-weight variant: increments are rounded to bf16 in the gather, weights are bf16, fp32
    accumulation.  Oracle: the same bf16-rounded weights held exactly in fp64, unrounded
    increments.  Bar: 2e-2 relative (Frobenius) per accumulated tensor and increment."""
    _say("UNet depth net bf16 variant, full width on 5x64x96, 20 frames")
    net = wl.net_unet_depth(1003, h=64, w=96, bf16=True)
    g = ev.EvConvNet(net)
    names = [g.kernel_name(i) for i in range(len(net.nodes))]
    g.destroy()
    assert names.count("conv_mfma_bf16") == 10, names
    frames = list(wl.stream_voxel(1003, 64, 96, 20, 0.02, n_prim=6))
    run_stream(net, frames[0], frames[1:], "frame", label="unet-bf16", tol=2e-2, frobenius=True, max_flips=200)


def test_matrix_core_conv_shapes_bf16():
    _say("bf16 matrix-core conv variants")
    for k, s, ci, co in [(3, 1, 32, 32), (3, 2, 16, 64), (5, 1, 64, 32), (5, 2, 48, 96), (7, 2, 16, 32), (1, 1, 32, 64), (3, 1, 68, 32), (5, 2, 20, 32),
                         (3, 1, 69, 32), (5, 2, 21, 32), (3, 1, 18, 64), (5, 1, 35, 64),   # c_in % 4 != 0
                         (3, 1, 32, 16), (3, 1, 37, 28)]:                                   # c_out % 32 != 0
        b = wl._NetBuilder(f"conv{k}s{s}", ci, 21, 27, 100 + k * 10 + s, bf16=True, bias=True)
        b.conv(-1, co, k, s, act=wl.ACT_RELU, out=1)
        net = b.finish()
        rng = np.random.default_rng(k + s)
        x0 = rng.standard_normal((ci, 21, 27)).astype(np.float32)
        incs = []
        for t in range(4):
            m = rng.random((21, 27)) < (0.03 if t < 3 else 1.0)
            incs.append(rng.standard_normal(x0.shape).astype(np.float32) * m[None])
        g = ev.EvConvNet(net)
        assert g.kernel_name(0) == "conv_mfma_bf16"
        g.destroy()
        run_stream(net, x0, incs, "increment", label=f"bf16 k{k}s{s}", tol=2e-2, frobenius=True, max_flips=20)


def test_narrow_input_conv_shapes():
    """First-layer kernel (2-8 input channels, taps x channels <= 128): strides, tap counts, one or
    two blocks of output channels, output channel counts that are not multiples of 32."""
    _say("narrow-input conv variants")
    for k, s, ci, co in [(5, 1, 5, 32), (3, 2, 4, 64), (7, 2, 2, 64), (3, 1, 8, 96), (1, 1, 3, 32),
                         (5, 1, 5, 16), (3, 1, 4, 48), (3, 2, 6, 100), (5, 2, 3, 24)]:
        b = wl._NetBuilder(f"narrow{k}s{s}", ci, 21, 27, 200 + k * 10 + s, bias=True)
        b.conv(-1, co, k, s, act=wl.ACT_RELU, out=1)
        net = b.finish()
        rng = np.random.default_rng(k + s + ci)
        x0 = rng.standard_normal((ci, 21, 27)).astype(np.float32)
        incs = []
        for t in range(4):
            m = rng.random((21, 27)) < (0.03 if t < 3 else 1.0)
            incs.append(rng.standard_normal(x0.shape).astype(np.float32) * m[None])
        g = ev.EvConvNet(net)
        assert g.kernel_name(0) == "conv_narrow_mfma_f32", (k, s, ci, co, g.kernel_name(0))
        g.destroy()
        run_stream(net, x0, incs, "increment", label=f"narrow k{k}s{s} {ci}->{co}", max_flips=2)


def test_matrix_core_conv_shapes():
    """Every (kernel, stride, channel-chunk) variant of the matrix-core conv on ragged sizes, with
    bias, dense and sparse increments."""
    _say("matrix-core conv variants: k in {1,3,5,7}, stride {1,2}, c_in in {16,32,48,64}")
    for k, s, ci, co in [(3, 1, 32, 32), (3, 2, 16, 64), (5, 1, 64, 32), (5, 2, 48, 96), (7, 2, 16, 32), (1, 1, 32, 64),
                         (3, 1, 68, 32), (5, 1, 20, 32), (3, 2, 36, 64),      # ragged channel chunks
                         (3, 1, 69, 32), (5, 2, 21, 32), (3, 1, 18, 64), (5, 1, 35, 64), (1, 1, 17, 32),  # c_in % 4 != 0
                         (3, 1, 32, 16), (5, 2, 16, 48), (3, 1, 37, 28), (3, 2, 64, 100),    # c_out % 32 != 0
                         (3, 1, 12, 32), (5, 1, 9, 64), (3, 2, 10, 20)]:                      # fewer than 16 input channels
        b = wl._NetBuilder(f"conv{k}s{s}", ci, 21, 27, 100 + k * 10 + s, bias=True)
        b.conv(-1, co, k, s, act=wl.ACT_RELU, out=1)
        net = b.finish()
        rng = np.random.default_rng(k + s)
        x0 = rng.standard_normal((ci, 21, 27)).astype(np.float32)
        incs = []
        for t in range(4):
            m = rng.random((21, 27)) < (0.03 if t < 3 else 1.0)
            incs.append(rng.standard_normal(x0.shape).astype(np.float32) * m[None])
        g = ev.EvConvNet(net)
        assert g.kernel_name(0) == "conv_mfma_f32"
        g.destroy()
        run_stream(net, x0, incs, "increment", label=f"mfma k{k}s{s}", max_flips=2)


def test_flow_net_reduced_concat_upsample():
    _say("flow encoder-decoder, reduced 4x64x64 width 8, density sweep, all nodes every step")
    net = wl.net_flow(1005, h=64, w=64, width=8)
    g = ev.EvConvNet(net)
    names = [g.kernel_name(i) for i in range(len(net.nodes))]
    g.destroy()
    # every decoder's up-sampling is read by its concatenation alone: interpolated there, never stored
    ups = [i for i, n in enumerate(net.nodes) if n.op == wl.OP_UPSAMPLE2X]
    assert ups and all(names[i] == "fused_into_concat_gather" for i in ups), names
    frames = list(wl.stream_count_timestamp(1005, 64, 64, densities=[0.001, 0.01, 0.05, 0.2], steps_per=4))
    run_stream(net, frames[0], frames[1:], "frame", label="flow-small", max_flips=8)


def test_delayed_flow_net_reduced():
    """Delayed-integration encoder-decoder: decoders fed by skips only, upsampled decoder outputs
    and predictions concatenated at full resolution, two final convolutions."""
    _say("delayed-integration flow net, reduced 4x64x96 width 8, all nodes every step")
    net = wl.net_flow_delayed(1006, h=64, w=96, width=8, d_width=32)
    frames = list(wl.stream_count_timestamp(1006, 64, 96, densities=[0.001, 0.01, 0.05, 0.2], steps_per=4))
    run_stream(net, frames[0], frames[1:], "frame", label="delayed-small", max_flips=8)


def test_resnet_reduced_pool_gap_linear():
    _say("ResNet-18-style classifier, reduced 2x64x64 width 8")
    net = wl.net_resnet18(1004, h=64, w=64, n_classes=11, width=8)
    frames = list(wl.stream_histogram(1004, 64, 64, steps=16))
    run_stream(net, frames[0], frames[1:], "frame", label="resnet-small", max_flips=8)


def test_edge_cases_zero_full_corner_special_values():
    _say("edge cases: zero increment, every site active, corner pixels, -0.0, denormal, NaN-free inf-free")
    net = wl.net_conv_stack(77, h=21, w=27)
    rng = np.random.default_rng(77)
    x0 = rng.standard_normal((5, 21, 27)).astype(np.float32)
    incs = []
    incs.append(np.zeros_like(x0))                                   # nothing changes
    incs.append(rng.standard_normal(x0.shape).astype(np.float32))    # everything changes
    for (y, x) in [(0, 0), (0, 26), (20, 0), (20, 26)]:              # single corner pixels
        d = np.zeros_like(x0)
        d[2, y, x] = 1.25
        incs.append(d)
    d = np.zeros_like(x0)
    d[:, 3, 3] = -0.0                                                 # negative zero: inactive
    d[1, 10, 10] = np.float32(1e-42)                                  # denormal: active
    incs.append(d)
    incs.append(np.zeros_like(x0))
    rep = run_stream(net, x0, incs, "increment", label="edge", exact_sets=False, max_flips=4)
    # explicit expectations on the input stage for the special values
    gpu = ev.EvConvNet(net)
    gpu.reset(_dev(x0))
    gpu.step(_dev(d))
    assert list(gpu.site_list(-1)) == [10 * 27 + 10]
    gpu.step(_dev(np.zeros_like(x0)))
    assert gpu.site_list(-1).size == 0
    for i in range(4):
        assert gpu.site_list(i).size == 0
        assert not gpu.state(i, ev.STATE_OCC_TOUCHED).any()
    gpu.destroy()


def _nan_aware_compare(gpu, ora, net, tol=TOL):
    """Sets bit-exact; NaN and infinite elements at the same places with the same sign; finite
    elements within tol of the tensor's largest finite magnitude."""
    for i in range(len(net.nodes)):
        c, h, w = ora.shape(i)
        s_gpu = cmp.words_to_mask(gpu.state(i, ev.STATE_OCC), h, w)
        t_gpu = cmp.words_to_mask(gpu.state(i, ev.STATE_OCC_TOUCHED), h, w)
        np.testing.assert_array_equal(s_gpu, ora.mask(i, cmp.SET_ACTIVE), err_msg=f"node {i} active set")
        np.testing.assert_array_equal(t_gpu, ora.mask(i, cmp.SET_TOUCHED), err_msg=f"node {i} touched set")
        np.testing.assert_array_equal(gpu.site_list(i), ora.site_list(i))
        pairs = [(gpu.state(i, ev.STATE_DY).astype(np.float64), ora.dy(i), "increment")]
        if ora.z(i).size:
            pairs.append((gpu.state(i, ev.STATE_Z).astype(np.float64), ora.z(i), "accumulated tensor"))
        for got, ref, what in pairs:
            with np.errstate(invalid="ignore"):
                got = np.where(s_gpu[:, :, None] == 1, got, 0.0) if what == "increment" else got
                np.testing.assert_array_equal(np.isnan(got), np.isnan(ref), err_msg=f"node {i} {what}: NaN positions")
                inf = np.isinf(ref)
                np.testing.assert_array_equal(np.isinf(got), inf, err_msg=f"node {i} {what}: infinities")
                np.testing.assert_array_equal(got[inf], ref[inf], err_msg=f"node {i} {what}: sign of infinities")
                fin = np.isfinite(ref)
                scale = max(np.abs(ref[fin]).max(), 1e-30)
                assert np.abs(got[fin] - ref[fin]).max() <= tol * scale, f"node {i} {what}"


@pytest.mark.parametrize("acts", ["relu", "linear"])
def test_nan_and_inf_increments_are_active_and_propagate(acts):
    """The zero test is `!= 0` on the fp32 value, so a NaN or an infinite increment makes its site
    active; the values then follow IEEE arithmetic through the layers: a conv output that reads
    the site becomes NaN / +-inf (a sum of opposite infinities: NaN), relu(NaN) = 0 on both sides,
    so behind a ReLU the increment is 0 - relu(z_old) and the accumulated tensor stays NaN until a
    refresh; without activation the NaN reaches the output.  Narrow-input, matrix-core and
    vector kernels (5 -> 32 -> 32 -> 64 -> 64 channels, strides 1, 2, 2, 1)."""
    _say(f"edge case: NaN and +-inf increments, {acts} stack")
    net = wl.net_conv_stack(78, h=21, w=27)
    if acts == "linear":
        for nd in net.nodes:
            nd.act = wl.ACT_NONE
    rng = np.random.default_rng(78)
    x0 = rng.standard_normal((5, 21, 27)).astype(np.float32)
    d1 = np.zeros_like(x0)
    d1[1, 4, 5] = np.nan
    d1[3, 15, 20] = np.inf
    d1[0, 15, 2] = -np.inf
    d1[2, 9, 9] = 0.5                       # an ordinary change beside them
    d2 = (rng.standard_normal(x0.shape) * (rng.random((1, 21, 27)) < 0.05)).astype(np.float32)
    gpu, ora = ev.EvConvNet(net), Oracle(net)
    gpu.reset(_dev(x0))
    ora.reset(x0)
    for t, d in enumerate((d1, d2, np.zeros_like(x0))):
        gpu.step(_dev(d))
        ora.step_increment(d)
        np.testing.assert_array_equal(gpu.site_list(-1), ora.site_list(-1), err_msg=f"step {t}: input list")
        if t == 0:
            assert {4 * 27 + 5, 15 * 27 + 20, 15 * 27 + 2, 9 * 27 + 9} == set(gpu.site_list(-1).tolist())
        _nan_aware_compare(gpu, ora, net)
    z0 = gpu.state(0, ev.STATE_Z)
    assert np.isnan(z0[4, 5]).all() and np.isinf(z0[15, 20]).any()
    if acts == "linear":
        import torch
        torch.cuda.synchronize()
        assert torch.isnan(gpu.outputs()[0]["y"]).any()
    # a refresh (regular forward pass of the cached frame, which now holds the NaN) is not a cure
    # for the input; a reset on a clean frame is
    gpu.reset(_dev(x0))
    ora.reset(x0)
    gpu.step(_dev(d2))
    ora.step_increment(d2)
    _nan_aware_compare(gpu, ora, net)
    gpu.destroy()


def test_layer_statistics_equal_the_oracles_counters():
    """evconv_get_stats against the oracle: sizes of the touched and active sets, touched tiles,
    and the executed / dense operation counts (2 x the oracle's tile-level and nominal dense
    multiply-accumulate counts, which tests/test_oracle_macs.py pins against hand counts)."""
    _say("layer statistics (set sizes, touched tiles, executed and dense FLOPs) vs the oracle's counters")
    cases = [(wl.net_single_conv(), None), (wl.net_unet_depth(1003, h=64, w=96), list(wl.stream_voxel(1003, 64, 96, 4, 0.02, n_prim=6)))]
    for net, frames in cases:
        gpu, ora = ev.EvConvNet(net), Oracle(net)
        if frames is None:
            x0, incs = wl.stream_line_increments()
            steps = [("increment", d) for d in incs[:4]]
        else:
            x0, steps = frames[0], [("frame", f) for f in frames[1:]]
        gpu.reset(_dev(x0))
        ora.reset(x0)
        checked = 0
        for kind, a in steps:
            (gpu.step_frame if kind == "frame" else gpu.step)(_dev(a))
            (ora.step_frame if kind == "frame" else ora.step_increment)(a)
            for i, nd in enumerate(net.nodes):
                if gpu.kernel_name(i) in ("fused_into_conv_gather", "fused_into_conv_weights", "fused_into_concat_gather"):
                    continue
                st = gpu.stats(i)
                c, h, w = ora.shape(i)
                s_ref, t_ref = ora.mask(i, cmp.SET_ACTIVE), ora.mask(i, cmp.SET_TOUCHED)
                assert (st.n_sites, st.n_tiles) == (h * w, -(-h // 8) * -(-w // 8))
                assert st.n_touched == int(t_ref.sum()), f"node {i} touched"
                # (the value-pruned set may differ by a flip where fp32 summation order decides whether a
                # saturating sigmoid moves at all; the other counters are integer functions of the input set)
                assert abs(st.n_active - int(s_ref.sum())) <= (2 if nd.act == wl.ACT_SIGMOID else 0), f"node {i} active"
                assert st.n_touched_tiles == int(np.count_nonzero(cmp.tile_words(t_ref)[0])), f"node {i} touched tiles"
                if nd.op in (wl.OP_CONV2D, wl.OP_LINEAR):
                    m = ora.macs(i, (8, 8))
                    assert st.flops_executed == 2.0 * m["tile"], f"node {i} executed"
                    assert st.flops_dense == 2.0 * m["dense_nominal"], f"node {i} dense"
                    assert m["site"] <= m["tile"] and m["site"] <= m["dense"] <= m["dense_nominal"]
                    checked += 1
        assert checked >= 4
        gpu.destroy()


def test_delay_of_an_add_that_follows_its_conv_is_not_fused():
    """0 convA(x), 1 convB(x), 2 DELAY of node 3, 3 ADD(0, 1), 4 ADD(3, 2) -> output.  The ADD
    could run in convB's epilogue, but the DELAY between them must see the ADD's buffers as the
    previous step left them; the planner therefore leaves this ADD to its own kernel.  Checked
    against the oracle with the default plan and with every fusion switched off."""
    _say("DELAY of a later ADD placed between the ADD and the conv that could host it")
    b = wl._NetBuilder("delay_add", 16, 24, 40, 41)
    ca = b.conv(-1, 32, 3, act=wl.ACT_NONE)
    cb = b.conv(-1, 32, 3, act=wl.ACT_NONE)
    d = b.delay(32, like=ca)
    add = b.simple(wl.OP_ADD, ca, cb)
    b.close_delay(d, add)
    b.simple(wl.OP_ADD, add, d, out=1)
    net = b.finish()
    rng = np.random.default_rng(41)
    x = rng.standard_normal((16, 24, 40)).astype(np.float32)
    frames = [x]
    for t in range(6):
        m = rng.random((1, 24, 40)) < 0.05
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    g = ev.EvConvNet(net)
    assert g.kernel_name(cb) == "conv_mfma_f32" and g.kernel_name(add) == "elementwise", \
        [g.kernel_name(i) for i in range(len(net.nodes))]
    g.destroy()
    for flags in (0, ev.FLAG_NO_FUSION):
        gpu, ora, rep = ev.EvConvNet(net, flags=flags), Oracle(net), cmp.Report()
        gpu.reset(_dev(frames[0]))
        ora.reset(frames[0])
        for f in frames[1:]:
            gpu.step_frame(_dev(f))
            ora.step_frame(f)
            cmp.compare_outputs(gpu, ora, rep)
            for i in range(len(net.nodes)):
                cmp.compare_node(gpu, ora, i, rep)
        assert rep.flips <= 4
        gpu.destroy()


def test_pooling_windows_other_than_3x3_and_a_global_mean_over_many_ragged_tiles():
    """Max-pool with 2 x 2 / stride 2 / no padding and with 5 x 5 / stride 1 / padding 2 windows
    (the kernel has a path of its own for 3 x 3), and a global mean over a 27 x 43 map (4 x 6 tiles,
    ragged last row and column, most of them inactive at any step) feeding a linear layer; sparse
    and dense steps, a refresh in between."""
    _say("max-pool 2x2 / 5x5 and a global mean over ragged tiles")
    b = wl._NetBuilder("pools", 6, 27, 43, 57)
    c0 = b.conv(-1, 32, 3, act=wl.ACT_RELU)
    p5 = b.simple(wl.OP_MAXPOOL, c0, k=5, stride=1, pad=2)
    g = b.simple(wl.OP_GAP, p5)
    b.linear(g, 10, out=1)
    p2 = b.simple(wl.OP_MAXPOOL, c0, k=2, stride=2, pad=0)
    b.conv(p2, 16, 3, act=wl.ACT_RELU, out=1)
    net = b.finish()
    rng = np.random.default_rng(57)
    x = rng.standard_normal((6, 27, 43)).astype(np.float32)
    frames = [x]
    for t in range(8):
        dens = 1.0 if t == 4 else 0.02
        m = rng.random((1, 27, 43)) < dens
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    gpu, ora, rep = ev.EvConvNet(net), Oracle(net), cmp.Report()
    assert gpu.kernel_name(g) == "global_avgpool" and gpu.kernel_name(p2) == "maxpool"
    gpu.reset(_dev(frames[0]))
    ora.reset(frames[0])
    for t, f in enumerate(frames[1:]):
        if t == 6:
            gpu.reset(_dev(f))
            ora.reset(f)
        else:
            gpu.step_frame(_dev(f))
            ora.step_frame(f)
        cmp.compare_outputs(gpu, ora, rep)
        for i in range(len(net.nodes)):
            cmp.compare_node(gpu, ora, i, rep)
    assert rep.flips <= 4
    gpu.destroy()


@pytest.mark.parametrize("hw", [(20, 28), (40, 56)], ids=["few_workgroups_8_waves", "more_workgroups_4_waves"])
def test_fp32_blocks_of_16_output_channels_with_ragged_channel_counts(hw):
    """Small maps make the fp32 matrix-core conv take blocks of 16 output channels (eight waves
    per workgroup on the smaller map, four on the larger).  Output channel counts that are not
    multiples of 16, a residual ADD + ReLU folded into the epilogue, a stride-2 layer and a 1 x 1
    layer; sparse steps, one dense step, a refresh."""
    _say(f"16-channel blocks of the fp32 matrix-core conv, {hw[0]} x {hw[1]}")
    h, w = hw
    b = wl._NetBuilder("nb16", 12, h, w, 77)
    c0 = b.conv(-1, 40, 3, act=wl.ACT_RELU)
    c1 = b.conv(c0, 40, 3, act=wl.ACT_NONE)
    r = b.simple(wl.OP_ADD, c1, c0, act=wl.ACT_RELU)
    c2 = b.conv(r, 24, 5, stride=2, act=wl.ACT_RELU)
    c3 = b.conv(c2, 72, 1, pad=0, act=wl.ACT_RELU)
    b.conv(c3, 16, 3, act=wl.ACT_NONE, out=1)
    net = b.finish()
    rng = np.random.default_rng(77)
    x = rng.standard_normal((12, h, w)).astype(np.float32)
    frames = [x]
    for t in range(7):
        m = rng.random((1, h, w)) < (1.0 if t == 3 else 0.03)
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    gpu, ora, rep = ev.EvConvNet(net), Oracle(net), cmp.Report()
    assert all(gpu.kernel_name(i) == "conv_mfma_f32" for i in (c0, c1, c2, c3)), [gpu.kernel_name(i) for i in range(len(net.nodes))]
    assert gpu.kernel_name(r) == "fused_into_conv_epilogue"
    gpu.reset(_dev(frames[0]))
    ora.reset(frames[0])
    for t, f in enumerate(frames[1:]):
        if t == 5:
            gpu.reset(_dev(f))
            ora.reset(f)
        else:
            gpu.step_frame(_dev(f))
            ora.step_frame(f)
        cmp.compare_outputs(gpu, ora, rep)
        for i in range(len(net.nodes)):
            cmp.compare_node(gpu, ora, i, rep)
    assert rep.flips <= 4
    gpu.destroy()


def test_auto_mode_times_both_modes_and_keeps_the_state():
    """AUTO runs windows of incremental and of dense-recompute steps, then holds the faster mode;
    whatever it picks, the state follows the same frames (Eq.2), so outputs and accumulated
    tensors stay within the fp32 bar of the oracle at every step; a net with an active
    sparsification layer stays incremental."""
    _say("AUTO mode: state parity through the mode switches")
    net = wl.net_unet_depth(1003, h=64, w=96)
    frames = list(wl.stream_voxel(1003, 64, 96, 16, 0.02, n_prim=6))
    gpu, ora, rep = ev.EvConvNet(net), Oracle(net), cmp.Report()
    gpu.set_mode(ev.MODE_AUTO)
    gpu.reset(_dev(frames[0]))
    ora.reset(frames[0])
    seen = []
    for f in frames[1:]:
        seen.append(gpu.current_mode())
        gpu.step_frame(_dev(f))
        ora.step_frame(f)
        cmp.compare_outputs_value_only(gpu, ora, rep)
        for i, nd in enumerate(net.nodes):
            if nd.op == wl.OP_CONV2D:
                z, zr = gpu.state(i, ev.STATE_Z).astype(np.float64), ora.z(i)
                assert np.abs(z - zr).max() <= TOL * np.abs(zr).max(), f"node {i}"
    assert seen[:8] == [ev.MODE_INCREMENTAL] * 4 + [ev.MODE_DENSE_RECOMPUTE] * 4, seen
    assert all(m in (ev.MODE_INCREMENTAL, ev.MODE_DENSE_RECOMPUTE) for m in seen[8:])
    with pytest.raises(ev.EvConvError):
        gpu.set_mode(3)
    gpu.destroy()
    sp = wl.net_unet_depth(1003, h=32, w=48, width=8, sparsify=True)
    sp.sparsify_tp = 0.1
    g = ev.EvConvNet(sp)
    g.set_mode(ev.MODE_AUTO)
    g.reset(_dev(frames[0][:, :32, :48].copy()))
    for f in frames[1:10]:
        assert g.current_mode() == ev.MODE_INCREMENTAL
        g.step_frame(_dev(f[:, :32, :48].copy()))
    g.destroy()


def test_fixed_step_of_a_first_node_sparsification_layer_survives_create_on_a_side_stream():
    """evconv_create clears the workspace on the net's stream and uploads a fixed rounding step
    with a blocking copy; on a non-blocking stream the two must still be ordered."""
    import torch
    net = _sp_only_net(8, 64, 96, k=0.375)
    side = torch.cuda.Stream()
    for _ in range(3):
        with torch.cuda.stream(side):
            g = ev.EvConvNet(net, stream=side)
        assert float(g.state(0, ev.STATE_STEP)[0]) == 0.375
        g.destroy()


def test_elementwise_kernels_bit_exact_against_fp32_oracle():
    """Activation increment (Eq.12-14) and addition (Eq.11) are single-rounded fp32 operations, so
    the GPU must match the oracle's binary32 mode bit for bit (tol = 0, exact sets)."""
    _say("bit-exact elementwise: ACT(relu) and ADD+relu nets against the binary32 oracle")
    nodes = [wl.Node(wl.OP_ACT, wl.ACT_RELU, -1, -2, 4, 4),
             wl.Node(wl.OP_ADD, wl.ACT_RELU, 0, -1, 4, 4),
             wl.Node(wl.OP_ADD, wl.ACT_NONE, 1, 0, 4, 4, is_output=1)]
    net = wl.Net("elementwise", 4, 19, 23, nodes, np.zeros(0, np.float32))
    rng = np.random.default_rng(5)
    x0 = rng.standard_normal((4, 19, 23)).astype(np.float32)
    frames, x = [], x0
    for t in range(8):
        m = rng.random((19, 23)) < 0.2
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m[None]).astype(np.float32)
        frames.append(x)
    run_stream(net, x0, frames, "frame", tol=0.0, exact_sets=True, fp32_oracle=True, label="ew-bits")


def test_reset_equals_stepped_state_and_dense_recompute_mode():
    """Refresh equivalence on the GPU: after k steps, reset(x_t) and DENSE_RECOMPUTE give the same
    accumulated tensors and output as the incremental path (within fp32 tolerance)."""
    _say("refresh equivalence and dense-recompute mode")
    net = wl.net_unet_depth(21, h=32, w=48, width=8)
    frames = list(wl.stream_voxel(21, 32, 48, 12, 0.05, n_prim=4))
    a, b, c = ev.EvConvNet(net), ev.EvConvNet(net), ev.EvConvNet(net)
    a.reset(_dev(frames[0]))
    c.reset(_dev(frames[0]))
    c.set_mode(ev.MODE_DENSE_RECOMPUTE)
    for f in frames[1:]:
        a.step_frame(_dev(f))
        c.step_frame(_dev(f))
    b.reset(_dev(frames[-1]))
    import torch
    torch.cuda.synchronize()
    for i, nd in enumerate(net.nodes):
        if nd.op == wl.OP_CONV2D or nd.act != wl.ACT_NONE:
            za, zb, zc = (n.state(i, ev.STATE_Z) for n in (a, b, c))
            s = np.abs(zb).max()
            assert np.abs(za - zb).max() <= TOL * s, f"node {i}"
            np.testing.assert_array_equal(zb, zc)
    ya, yb, yc = (n.outputs()[0]["y"].cpu().numpy() for n in (a, b, c))
    assert np.abs(ya - yb).max() <= TOL
    np.testing.assert_array_equal(yb, yc)


@pytest.mark.parametrize("width,h,w", [(8, 40, 56), (32, 64, 96)])
def test_run_to_run_bit_reproducible(width, h, w):
    """width 8: the vector-ALU kernels; width 32: the matrix-core kernels (partial sums of up to
    eight waves, fused epilogue adds, folded up-sampling, occupancy words OR-ed by several
    workgroups)."""
    _say(f"determinism: the same stream twice gives identical bits (width {width})")
    net = wl.net_unet_depth(31, h=h, w=w, width=width)
    frames = list(wl.stream_voxel(31, h, w, 10, 0.03, n_prim=4))
    res = []
    for _ in range(2):
        g = ev.EvConvNet(net)
        g.reset(_dev(frames[0]))
        for f in frames[1:]:
            g.step_frame(_dev(f))
        import torch
        torch.cuda.synchronize()
        stored = [i for i in range(len(net.nodes)) if not g.kernel_name(i).endswith(("_gather", "_weights"))]
        res.append([g.state(i, ev.STATE_DY).copy() for i in stored] +
                   [g.outputs()[0]["y"].cpu().numpy()] + [g.site_list(i) for i in stored])
        g.destroy()
    for u, v in zip(*res):
        np.testing.assert_array_equal(u, v)


@pytest.mark.gpu
@pytest.mark.parametrize("n_streams", [1, 3])
def test_outputs_are_fresh_aliases_of_the_same_memory(n_streams):
    """Every call of outputs() returns tensors of its own over the streams' memory: changing one's
    shape or autograd state leaves the next call's alone, values written by a step show in all."""
    import torch
    net = wl.net_single_conv(5, 16, 24, 40)
    gpu = ev.EvConvNet(net, n_streams=n_streams)
    shape = (net.in_c, net.in_h, net.in_w) if n_streams == 1 else (n_streams, net.in_c, net.in_h, net.in_w)
    gen = torch.Generator().manual_seed(3)
    gpu.reset(torch.randn(shape, generator=gen).cuda())
    first = [gpu.outputs(s) for s in range(n_streams)]
    with torch.inference_mode():
        gpu.step(torch.randn(shape, generator=gen).cuda())
        inside = gpu.outputs(0)[0]["y"]
    second = [gpu.outputs(s) for s in range(n_streams)]
    ptrs = set()
    for a, b in zip(first, second):
        for key in ("y", "dy", "idx", "count"):
            assert a[0][key] is not b[0][key] and a[0][key].data_ptr() == b[0][key].data_ptr()
            assert torch.equal(a[0][key], b[0][key])
        ptrs.add(a[0]["y"].data_ptr())
    assert len(ptrs) == n_streams and inside.data_ptr() == first[0][0]["y"].data_ptr()
    first[0][0]["y"].unsqueeze_(0).requires_grad_()
    third = gpu.outputs(0)[0]["y"]
    assert not third.requires_grad and tuple(third.shape) == tuple(second[0][0]["y"].shape)
    third.add_(1.0)
    assert second[0][0]["y"]._version == 0
    gpu.destroy()


def test_step_before_reset_is_an_error():
    net = wl.net_single_conv(3, c=4, h=8, w=8)
    g = ev.EvConvNet(net)
    with pytest.raises(ev.EvConvError) as e:
        g.step(_dev(np.zeros((4, 8, 8), np.float32)))
    assert e.value.status == ev.ERR_STATE
    # a node index out of range is refused by the C ABI itself (called directly, past the binding)
    import ctypes
    buf = np.zeros(64, np.float32)
    for node in (1, 7, -2):
        st = ev.lib().evconv_get_state_stream(g._h, 0, node, ev.STATE_Z, buf.ctypes.data_as(ctypes.c_void_p), buf.nbytes)
        assert st != 0, node
    g.destroy()


@pytest.mark.timeout(600)
def test_workload4_resnet18_full_size():
    """Full-size ResNet-18-style classifier on 2x224x224 event histograms, density ramp 0.5-5 %:
    max-pool, strided convs with 1x1 projection shortcuts, global mean, linear head."""
    _say("workload 4: ResNet-18 2x224x224, 100 frames, density 0.5 -> 5 %")
    net = wl.net_resnet18()
    gen = wl.stream_histogram(1004, 224, 224, steps=100)
    x0 = next(gen)
    run_stream(net, x0, gen, "frame", check_nodes_at={1, 2, 50, 100}, label="w4", max_flips=64)


@pytest.mark.timeout(900)
def test_workload5_flow_net_full_size_density_sweep():
    """Full-size optical-flow encoder-decoder on 4x256x256 (concat skips, flow head per scale):
    100 consecutive steps, ten at each of ten log-spaced increment densities between 0.1 % and
    20 % (the GPU alone runs the 1000-step sweep in bench.py --sweep; the oracle takes 0.6 s per
    step of this net).  Outputs and the input stage at every step, every node at one step per
    density."""
    _say("workload 5: flow encoder-decoder 4x256x256, 10 densities 0.1 .. 20 %, 10 steps each")
    net = wl.net_flow()
    dens = [float(d) for d in np.geomspace(0.001, 0.2, 10)]
    gen = wl.stream_count_timestamp(1005, 256, 256, densities=dens, steps_per=10)
    x0 = next(gen)
    run_stream(net, x0, gen, "frame", check_nodes_at=set(range(5, 101, 10)) | {1, 100}, label="w5", max_flips=64)


@pytest.mark.timeout(600)
def test_delayed_flow_net_full_size():
    _say("delayed-integration flow net 4x256x256, densities 0.1 / 1 / 5 %, 4 steps each")
    net = wl.net_flow_delayed()
    gen = wl.stream_count_timestamp(1006, 256, 256, densities=[0.001, 0.01, 0.05], steps_per=4)
    x0 = next(gen)
    run_stream(net, x0, gen, "frame", check_nodes_at={1, 6, 11}, label="delayed-full", max_flips=64)


@pytest.mark.timeout(900)
def test_workload3_unet_bf16_full_size_100_steps():
    """Workload 3, bf16-weight variant, full size, 100 consecutive frames: 2e-2 relative."""
    _say("workload 3 (bf16 weights): UNet depth net 5x256x352, 100 frames at 2 %")
    net = wl.net_unet_depth(bf16=True)
    gen = wl.stream_voxel(1003, 256, 352, 100, 0.02)
    x0 = next(gen)
    run_stream(net, x0, gen, "frame", check_nodes_at={1, 50, 100}, label="w3-bf16", tol=2e-2, frobenius=True,
               max_flips=800)   # (measured: 378, all at the 1-channel sigmoid head and behind ReLU zero crossings)


@pytest.mark.timeout(900)
def test_workload3_unet_full_size_100_steps():
    """Full-size UNet depth net (5x256x352), 100 consecutive frames at 2 % changed pixels, in the
    configuration bench.py times.  Outputs and the input stage are compared at every step, every
    node at steps 1, 2, 50 and 100."""
    _say("workload 3: UNet depth net 5x256x352, 100 frames at 2 %")
    net = wl.net_unet_depth()
    gen = wl.stream_voxel(1003, 256, 352, 100, 0.02)
    x0 = next(gen)
    # The 1-channel sigmoid head decides "increment == 0" on differences of saturating values of
    # the order 1e-8; fp32 drift against the fp64 oracle flips that decision at a few sites per
    # thousand.  Every other node must agree on every site.
    rep = run_stream(net, x0, gen, "frame", check_nodes_at={1, 2, 50, 100}, label="w3",
                     max_flips=600)   # (measured: 170 over the 100 steps)
    assert set(rep.flips_by_node) <= {"node 20 active"}, rep.flips_by_node


# --------------------------------------------------------------------------- sparsification layer

def _sp_only_net(c, h, w, k=None, tp=0.0):
    w_arr = np.zeros(0, np.float32)
    k_off = -1
    if k is not None:
        w_arr, k_off = np.asarray([k], np.float32), 0
    nodes = [wl.Node(wl.OP_SPARSIFY, wl.ACT_NONE, -1, -2, c, c, 1, 1, 0, k_off, -1, 1)]
    return wl.Net("sp_only", c, h, w, nodes, w_arr, sparsify_tp=tp)


@pytest.mark.parametrize("k,tp", [(0.3, 0.0), (None, 0.25)])
def test_sparsification_layer_bit_exact_against_fp32_oracle(k, tp):
    """Eq.3-8 are single-rounded fp32 operations on an input both sides see bit-identically, so
    the residual, the emitted increments and the lists must match the binary32 oracle exactly;
    with k = t_p * RMS both sides must also arrive at the identical 8-bit step."""
    _say(f"sparsification layer alone, k={k} tp={tp}: bit-exact vs the binary32 oracle")
    net = _sp_only_net(8, 21, 27, k=k, tp=tp)
    rng = np.random.default_rng(3)
    x0 = rng.standard_normal((8, 21, 27)).astype(np.float32)
    frames, x = [], x0
    for t in range(12):
        m = rng.random((21, 27)) < 0.3
        x = (x + 0.2 * rng.standard_normal(x.shape).astype(np.float32) * m[None]).astype(np.float32)
        frames.append(x)
    g, o = ev.EvConvNet(net), Oracle(net, fp32_state=True)
    g.reset(_dev(x0))
    o.reset(x0)
    assert float(g.state(0, ev.STATE_STEP)[0]) == o.step_size(0) > 0
    g.destroy()
    run_stream(net, x0, frames, "frame", tol=0.0, exact_sets=True, fp32_oracle=True, label="sp-bits")


def test_sparsified_conv_net_exact_arithmetic():
    """Two convolutions with a sparsification layer between them, on values chosen so that every
    sum is exact in binary32 (dyadic weights and inputs, k = 0.5): the rounding decisions cannot
    differ, so the GPU must equal the fp64 oracle on every tensor and every list."""
    _say("conv -> sparsify -> conv with exact arithmetic")
    b = wl._NetBuilder("sp_exact", 4, 19, 23, 5, sparsify=True, sparsify_k=0.5)
    x = b.conv(-1, 32, 3, 1)
    b.conv(x, 32, 3, 1, out=1)
    net = b.finish()
    rng = np.random.default_rng(6)
    wts = net.weights.copy()
    for nd in net.nodes:
        if nd.op == wl.OP_CONV2D:
            n = nd.c_out * nd.c_in * 9
            wts[nd.w_off:nd.w_off + n] = rng.integers(-2, 3, n) / 4.0
    net.weights = wts
    x0 = (rng.integers(-8, 9, (4, 19, 23)) / 4.0).astype(np.float32)
    incs = [((rng.integers(-4, 5, x0.shape) / 4.0) * (rng.random((1, 19, 23)) < 0.1)).astype(np.float32)
            for _ in range(8)]
    g = ev.EvConvNet(net)
    assert g.kernel_name(2) == "conv_mfma_f32"
    g.destroy()
    rep = run_stream(net, x0, incs, "increment", tol=1e-7, exact_sets=True, label="sp-exact")
    assert rep.flips == 0


def test_sparsification_layers_folded_into_conv_epilogues_exact_arithmetic():
    """Sparsification layers whose input comes from a matrix-core conv, directly or through an ADD
    folded into that conv, run inside its epilogue.  Exact arithmetic again (dyadic weights and
    inputs, k = 0.5), so the GPU must equal the fp64 oracle on every tensor and every list, with
    the layers folded and with every fusion switched off."""
    _say("sparsification layers inside conv epilogues (behind the conv and behind a folded ADD), exact arithmetic")
    b = wl._NetBuilder("sp_fused_exact", 16, 21, 27, 5, sparsify=True, sparsify_k=0.5)
    c1 = b.conv(-1, 32, 3)
    c2 = b.conv(c1, 32, 3)                       # its layer reads c1: behind the conv stage
    c3 = b.conv(c2, 32, 3, act=wl.ACT_NONE)      # its layer reads c2
    a = b.simple(wl.OP_ADD, c1, c3, act=wl.ACT_RELU)   # folded into c3's epilogue
    b.conv(a, 32, 3, out=1)                      # its layer reads the ADD: behind the folded ADD stage
    net = b.finish()
    rng = np.random.default_rng(8)
    wts = net.weights.copy()
    for nd in net.nodes:
        if nd.op == wl.OP_CONV2D:
            n = nd.c_out * nd.c_in * 9
            wts[nd.w_off:nd.w_off + n] = rng.integers(-1, 2, n) / 8.0
    net.weights = wts
    x0 = (rng.integers(-8, 9, (16, 21, 27)) / 4.0).astype(np.float32)
    incs = [((rng.integers(-4, 5, x0.shape) / 4.0) * (rng.random((1, 21, 27)) < 0.1)).astype(np.float32)
            for _ in range(8)]
    incs.append(np.zeros_like(x0))
    sp_nodes = [i for i, nd in enumerate(net.nodes) if nd.op == wl.OP_SPARSIFY]
    assert len(sp_nodes) == 3
    g = ev.EvConvNet(net)
    names = [g.kernel_name(i) for i in range(len(net.nodes))]
    g.destroy()
    assert all(names[i] == "fused_into_conv_epilogue" for i in sp_nodes), names
    assert names[a] == "fused_into_conv_epilogue"
    for flags in (0, ev.FLAG_NO_FUSION):
        gpu, ora, rep = ev.EvConvNet(net, flags=flags), Oracle(net), cmp.Report()
        gpu.reset(_dev(x0))
        ora.reset(x0)
        for d in incs:
            gpu.step(_dev(d))
            ora.step_increment(d)
            cmp.compare_outputs(gpu, ora, rep, 1e-7)
            for i in range(len(net.nodes)):
                cmp.compare_node(gpu, ora, i, rep, tol=1e-7, exact_sets=True)
        # a refresh clears the residuals and leaves the layers' buffers holding values
        gpu.set_refresh_period(1)
        gpu.step(_dev(incs[0]))
        for i in sp_nodes:
            assert not gpu.state(i, ev.STATE_Z).any(), f"residual of node {i} after a refresh"
        assert rep.flips == 0
        gpu.destroy()


def test_sparsified_unet_properties_and_speed_of_convergence():
    """Lossy path on a reduced UNet with t_p = 0.3: what must hold whatever the rounding
    decisions were - residual bounded by k/2, emitted increments multiples of k, fewer active
    sites than the lossless run, output a bounded approximation of the regular forward pass,
    and a refresh returns to the regular forward pass."""
    _say("sparsified UNet (t_p = 0.3): residual bound, quantised increments, sparsity, refresh")
    base = wl.net_unet_depth(1003, h=64, w=96)
    sp = wl.net_unet_depth(1003, h=64, w=96, sparsify=True)
    sp.sparsify_tp = 0.3
    # small-valued increments (what the layer is for): a dense frame plus faint changes at 2 % of
    # the pixels per step
    rng = np.random.default_rng(11)
    frames = [rng.standard_normal((5, 64, 96)).astype(np.float32)]
    for _ in range(12):
        m = rng.random((1, 64, 96)) < 0.02
        frames.append((frames[-1] + 0.05 * rng.standard_normal(frames[0].shape).astype(np.float32) * m).astype(np.float32))
    ga, gs = ev.EvConvNet(base), ev.EvConvNet(sp)
    ga.reset(_dev(frames[0]))
    gs.reset(_dev(frames[0]))
    act_a = act_s = 0
    for f in frames[1:]:
        ga.step_frame(_dev(f))
        gs.step_frame(_dev(f))
        act_a += sum(ga.stats(i).n_active for i, nd in enumerate(base.nodes) if nd.op == wl.OP_CONV2D)
        act_s += sum(gs.stats(i).n_active for i, nd in enumerate(sp.nodes) if nd.op == wl.OP_CONV2D)
        for i, nd in enumerate(sp.nodes):
            if nd.op != wl.OP_SPARSIFY:
                continue
            k = float(gs.state(i, ev.STATE_STEP)[0])
            assert k > 0
            d = gs.state(i, ev.STATE_Z)
            assert d.min() >= -0.5 * k * (1 + 1e-5) and d.max() <= 0.5 * k * (1 + 1e-5), f"node {i}"
            m = cmp.words_to_mask(gs.state(i, ev.STATE_OCC), *gs.shape(i)[1:]).astype(bool)
            y = gs.state(i, ev.STATE_DY)[m]
            if y.size:
                assert np.abs(y / k - np.rint(y / k)).max() < 1e-3, f"node {i}: increments not multiples of k"
    assert act_s < 0.8 * act_a, (act_s, act_a)
    import torch
    torch.cuda.synchronize()
    ya = ga.outputs()[0]["y"].cpu().numpy()
    ys = gs.outputs()[0]["y"].cpu().numpy()
    assert 0 < np.abs(ya - ys).max() < 0.2          # sigmoid output in (0, 1)
    gs.reset(_dev(frames[-1]))
    ga.reset(_dev(frames[-1]))
    torch.cuda.synchronize()
    # a refresh is a regular forward pass, the layer is the identity there: the same function.  (Not
    # the same roundings: the plain net's up-sampling convs run with folded weights, this net's
    # convs read a sparsification layer and do not.)
    np.testing.assert_allclose(ga.outputs()[0]["y"].cpu().numpy(), gs.outputs()[0]["y"].cpu().numpy(), rtol=0, atol=1e-5)
    ga.destroy()
    gs.destroy()


# --------------------------------------------------------------------------- elementwise multiply

def test_multiply_increment_bit_exact_against_fp32_oracle():
    """Eq.15-17 as single-rounded binary32 operations: two 1x1 selector convolutions (exact: weights
    1, 0 and 0, 3) feed the product, so its inputs are bit-identical on both sides and the product
    increments, both accumulators and the OR-ed sets must match bit for bit."""
    _say("bit-exact elementwise multiply against the binary32 oracle")
    w = np.asarray([1.0, 0.0, 0.0, 3.0], np.float32)
    nodes = [wl.Node(wl.OP_CONV2D, wl.ACT_NONE, -1, -2, 2, 1, 1, 1, 0, 0, -1, 0),
             wl.Node(wl.OP_CONV2D, wl.ACT_NONE, -1, -2, 2, 1, 1, 1, 0, 2, -1, 0),
             wl.Node(wl.OP_MUL, wl.ACT_NONE, 0, 1, 1, 1, 1, 1, 0, -1, -1, 1),
             wl.Node(wl.OP_MUL, wl.ACT_NONE, 2, 2, 1, 1, 1, 1, 0, -1, -1, 1)]
    net = wl.Net("mul_bits", 2, 21, 27, nodes, w)
    rng = np.random.default_rng(8)
    x0 = rng.standard_normal((2, 21, 27)).astype(np.float32)
    frames, x = [], x0
    for t in range(10):
        m = rng.random((2, 21, 27)) < 0.2          # channels change independently
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    run_stream(net, x0, frames, "frame", tol=0.0, exact_sets=True, fp32_oracle=True, label="mul-bits")
    g, o = ev.EvConvNet(net), Oracle(net, fp32_state=True)
    g.reset(_dev(x0))
    o.reset(x0)
    for f in frames[:4]:
        g.step_frame(_dev(f))
        o.step_frame(f)
    for i in (2, 3):
        np.testing.assert_array_equal(g.state(i, ev.STATE_Z2), o.z2(i).astype(np.float32))
        np.testing.assert_array_equal(g.state(i, ev.STATE_Z), o.z(i).astype(np.float32))
    g.destroy()


@pytest.mark.parametrize("width,h,w", [(8, 37, 45), (32, 64, 96)])
def test_gated_network_sigmoid_tanh_products(width, h, w):
    """Gate structure of ConvLSTM / ConvGRU cells (sigmoid gate x tanh candidate, update gate x
    block input, a square) against the fp64 oracle; width 32 runs the matrix-core convolutions."""
    _say(f"gated network width {width} on 5x{h}x{w}: multiply increments, tanh, all nodes every step")
    net = wl.net_gated(1007, in_c=5, h=h, w=w, width=width)
    frames = list(wl.stream_voxel(1007, h, w, 12, 0.03, n_prim=6))
    run_stream(net, frames[0], frames[1:], "frame", label=f"gated-{width}", max_flips=16)


# --------------------------------------------------------------------------- refresh policy

@pytest.mark.parametrize("kind", ["frame", "increment"])
def test_refresh_period_runs_a_regular_forward_pass_every_nth_step(kind):
    """"Drift Errors": with period 3 the 3rd and 6th step are regular forward passes.  The net
    with the policy must be bit-identical to one that is reset by hand at those steps, and equal
    to the oracle's forward pass of the same frame."""
    _say(f"refresh period 3, {kind} input")
    net = wl.net_unet_depth(1003, h=32, w=48, width=8)
    frames = list(wl.stream_voxel(5, 32, 48, 7, 0.05, n_prim=4))
    a, b = ev.EvConvNet(net), ev.EvConvNet(net)
    a.set_refresh_period(3)
    a.reset(_dev(frames[0]))
    b.reset(_dev(frames[0]))
    ora = Oracle(net)
    out = ora.outputs[0]
    import torch
    torch.cuda.synchronize()
    y_before = a.outputs()[0]["y"].cpu().numpy()
    for t in range(1, 8):
        inp = frames[t] if kind == "frame" else (frames[t] - frames[t - 1]).astype(np.float32)
        (a.step_frame if kind == "frame" else a.step)(_dev(inp))
        if t % 3 == 0:
            cur = b.state(-1, ev.STATE_X_PREV) + inp if kind == "increment" else frames[t]
            b.reset(_dev(cur.astype(np.float32)))
        else:
            (b.step_frame if kind == "frame" else b.step)(_dev(inp))
        import torch
        torch.cuda.synchronize()
        ya, yb = a.outputs()[0]["y"].cpu().numpy(), b.outputs()[0]["y"].cpu().numpy()
        np.testing.assert_array_equal(ya, yb, err_msg=f"step {t}")
        for i in (3, 12, 18):
            np.testing.assert_array_equal(a.state(i, ev.STATE_Z), b.state(i, ev.STATE_Z), err_msg=f"step {t} node {i}")
        dya = a.outputs()[0]["dy"].cpu().numpy()
        if t % 3 == 0:
            # internal sets are empty after a refresh; the output increment is y(n) - y(n-1) at every
            # site (one fp32 subtraction), listed in full, so that Eq.2 holds across the refresh
            assert a.site_list(-1).size == 0 and a.site_list(3).size == 0
            np.testing.assert_array_equal(dya, ya - y_before, err_msg=f"step {t}: dy of a refresh step")
            np.testing.assert_array_equal(a.site_list(out), np.arange(ya[0].size, dtype=np.int32))
            ora.reset(a.state(-1, ev.STATE_X_PREV))
            ref = np.transpose(ora.y(out), (2, 0, 1))
            assert np.abs(ya - ref).max() <= TOL * np.abs(ref).max()
        else:
            np.testing.assert_array_equal(ya, y_before + dya, err_msg=f"step {t}: Eq.2")
        y_before = ya
    with pytest.raises(ev.EvConvError):
        a.set_refresh_period(-1)
    a.destroy()
    b.destroy()


# --------------------------------------------------------------------------- fp32 through bf16 high/low parts

def test_split_bf16_conv_shapes_meet_the_fp32_bar():
    """EVCONV_F32_SPLIT: fp32 weights and increments contracted as three bf16 products.  Every
    kernel variant on ragged sizes, against the fp64 oracle with the unrounded fp32 weights, at
    the fp32 tolerance."""
    _say("split-bf16 matrix-core conv variants at the fp32 tolerance")
    worst = 0.0
    for k, s, ci, co in [(3, 1, 32, 32), (3, 2, 16, 64), (5, 1, 64, 32), (5, 2, 48, 96), (7, 2, 16, 32), (1, 1, 32, 64),
                         (3, 1, 128, 64), (3, 1, 68, 32), (5, 2, 20, 32),
                         (3, 1, 69, 32), (5, 2, 21, 32), (3, 1, 18, 64), (5, 1, 35, 64),   # c_in % 4 != 0
                         (3, 1, 32, 16), (3, 1, 37, 28)]:                                   # c_out % 32 != 0
        b = wl._NetBuilder(f"conv{k}s{s}", ci, 21, 27, 100 + k * 10 + s, bias=True)
        b.conv(-1, co, k, s, act=wl.ACT_RELU, out=1)
        net = wl.with_weight_dtype(b.finish(), wl.WD_F32_SPLIT)
        rng = np.random.default_rng(k + s)
        x0 = rng.standard_normal((ci, 21, 27)).astype(np.float32)
        incs = []
        for t in range(4):
            m = rng.random((21, 27)) < (0.03 if t < 3 else 1.0)
            incs.append(rng.standard_normal(x0.shape).astype(np.float32) * m[None])
        g = ev.EvConvNet(net)
        assert g.kernel_name(0) == "conv_mfma_f32_split_bf16x3"
        g.destroy()
        rep = run_stream(net, x0, incs, "increment", label=f"split k{k}s{s}", max_flips=2)
        worst = max(worst, rep.max_rel_z, rep.max_rel_y)
    _say(f"split-bf16: worst relative error {worst:.2e} (bar {TOL:.0e})")


def test_split_bf16_unet_reduced():
    _say("UNet depth net, full width on 5x64x96, split-bf16 contraction, fp32 tolerance")
    net = wl.with_weight_dtype(wl.net_unet_depth(1003, h=64, w=96), wl.WD_F32_SPLIT)
    g = ev.EvConvNet(net)
    names = [g.kernel_name(i) for i in range(len(net.nodes))]
    g.destroy()
    assert names.count("conv_mfma_f32_split_bf16x3") == 10, names
    frames = list(wl.stream_voxel(1003, 64, 96, 20, 0.02, n_prim=6))
    rep = run_stream(net, frames[0], frames[1:], "frame", label="unet-split", max_flips=40)
    _say(f"split-bf16 UNet: max rel z err {rep.max_rel_z:.2e}, y err {rep.max_rel_y:.2e}")


@pytest.mark.timeout(900)
def test_workload3_unet_split_bf16_full_size_100_steps():
    """The bench configuration with the split-bf16 contraction: 100 frames, fp32 tolerance."""
    _say("workload 3, split-bf16 contraction: UNet depth net 5x256x352, 100 frames at 2 %")
    net = wl.with_weight_dtype(wl.net_unet_depth(), wl.WD_F32_SPLIT)
    gen = wl.stream_voxel(1003, 256, 352, 100, 0.02)
    x0 = next(gen)
    rep = run_stream(net, x0, gen, "frame", check_nodes_at={1, 2, 50, 100}, label="w3-split",
                     max_flips=600)   # (measured: 170 over the 100 steps)
    assert set(rep.flips_by_node) <= {"node 20 active"}, rep.flips_by_node
    _say(f"split-bf16 w3: max rel z err {rep.max_rel_z:.2e}, y err {rep.max_rel_y:.2e}")


# --------------------------------------------------------------------------- several streams per net

@pytest.mark.parametrize("which", ["unet", "mixed_ops", "sparsified", "recurrent"])
def test_streams_stepped_together_equal_single_stream_nets(which):
    """n_streams = 3: three independent event streams share the weights and are stepped by one
    call.  Every stream must equal a single-stream net fed the same frames, and stream 1 is also
    checked against the oracle."""
    _say(f"three streams in one net ({which}) against three single-stream nets")
    import torch
    if which == "unet":
        net = wl.net_unet_depth(1003, h=64, w=96)
        gens = [list(wl.stream_voxel(40 + s, 64, 96, 6, 0.01 * (s + 1), n_prim=5)) for s in range(3)]
    elif which == "recurrent":
        net = wl.net_convlstm(44, in_c=4, h=16, w=24, hidden=32, out_c=2)
        rng = np.random.default_rng(4)
        gens = []
        for s in range(3):
            x = rng.standard_normal((4, 16, 24)).astype(np.float32)
            fr = [x]
            for _ in range(6):
                x = (x + rng.standard_normal(x.shape).astype(np.float32) * (rng.random((1, 16, 24)) < 0.1)).astype(np.float32)
                fr.append(x)
            gens.append(fr)
    elif which == "mixed_ops":
        net = wl.net_random_small(7)
        rng = np.random.default_rng(3)
        gens = []
        for s in range(3):
            x = rng.standard_normal((3, 13, 11)).astype(np.float32)
            fr = [x]
            for _ in range(6):
                x = (x + rng.standard_normal(x.shape).astype(np.float32) * (rng.random((1, 13, 11)) < 0.2)).astype(np.float32)
                fr.append(x)
            gens.append(fr)
    else:
        net = wl.net_conv_stack(1002, h=40, w=56, sparsify=True)
        net.sparsify_tp = 0.2
        gens = [list(wl.stream_voxel(50 + s, 40, 56, 6, 0.03, n_prim=4)) for s in range(3)]
    multi = ev.EvConvNet(net, n_streams=3)
    singles = [ev.EvConvNet(net) for _ in range(3)]
    assert multi.n_streams == 3 and multi.stream_stride % 256 == 0
    ora = Oracle(net)
    keeps = [i for i in range(len(net.nodes)) if not multi.kernel_name(i).startswith("fused_into_")]
    for t in range(7):
        batch = _dev(np.stack([gens[s][t] for s in range(3)]))
        if t == 0:
            multi.reset(batch)
            ora.reset(gens[1][0])
        else:
            multi.step_frame(batch)
            ora.step_frame(gens[1][t])
        for s in range(3):
            (singles[s].reset if t == 0 else singles[s].step_frame)(_dev(gens[s][t]))
        torch.cuda.synchronize()
        # The matrix-core convolutions pick their launch shape (and with it the order of the partial
        # sums) from the number of workgroups, which grows with the number of streams: those nets
        # agree to rounding, the net without matrix-core layers bit for bit.  With sparsification
        # layers a last-bit difference can flip a rounding decision, which moves an element by one
        # rounding step k (and the sets behind it): those outputs are compared at a bar that a
        # stream mix-up would still miss by two orders of magnitude.
        exact = which == "mixed_ops"
        loose = which == "sparsified"
        for s in range(3):
            for a, b in zip(multi.outputs(s), singles[s].outputs()):
                if exact:
                    assert torch.equal(a["y"], b["y"]) and torch.equal(a["dy"], b["dy"]), f"step {t} stream {s}"
                    assert int(a["count"]) == int(b["count"])
                else:
                    scale = float(b["y"].abs().max())
                    assert float((a["y"] - b["y"]).abs().max()) <= (2e-2 if loose else 1e-5) * scale, f"step {t} stream {s}"
            for i in keeps[:: max(1, len(keeps) // 6)]:
                if exact:
                    np.testing.assert_array_equal(multi.state(i, ev.STATE_OCC, s), singles[s].state(i, ev.STATE_OCC))
                    np.testing.assert_array_equal(multi.site_list(i, s), singles[s].site_list(i))
                    np.testing.assert_array_equal(multi.state(i, ev.STATE_DY, s), singles[s].state(i, ev.STATE_DY))
                elif not loose:
                    np.testing.assert_array_equal(multi.state(i, ev.STATE_OCC_TOUCHED, s),
                                                  singles[s].state(i, ev.STATE_OCC_TOUCHED))
            np.testing.assert_array_equal(multi.state(-1, ev.STATE_X_PREV, s), gens[s][t])
        if which != "sparsified":
            out = ora.outputs[0]
            y1 = multi.outputs(1)[[o["node"] for o in multi.outputs(1)].index(out)]["y"].cpu().numpy()
            ref = np.transpose(ora.y(out), (2, 0, 1))
            assert np.abs(y1 - ref).max() <= TOL * max(np.abs(ref).max(), 1e-30)
    with pytest.raises(ev.EvConvError):
        multi.state(0, ev.STATE_DY, stream=3)
    multi.destroy()
    for g in singles:
        g.destroy()


# --------------------------------------------------------------------------- HIP graph replay

@pytest.mark.parametrize("which", ["unet", "recurrent"])
def test_step_captured_in_a_hip_graph_replays_bit_identically(which):
    """A step is a fixed sequence of kernel launches on the caller's stream (no allocation, no
    synchronisation, no memset), so the caller may capture it once and replay it.  Every replay,
    with eager work and synchronisations in between, must equal the eager net bit for bit."""
    _say("one step captured in a HIP graph, replayed 8 times against an eager net")
    import torch
    if which == "unet":
        net = wl.net_unet_depth(1003, h=64, w=96)
        frames = list(wl.stream_voxel(77, 64, 96, 9, 0.03, n_prim=5))
        watch = (0, 5, 12, 18)
    else:
        # a net with DELAY nodes is captured after an incremental step, as the header asks: the
        # kernels take "the previous pass was a regular one" as an argument
        net = wl.net_convlstm(45, in_c=5, h=32, w=48, hidden=32, out_c=1)
        frames = list(wl.stream_voxel(78, 32, 48, 9, 0.03, n_prim=5))
        watch = (0, 1, 7, 11)
    side = torch.cuda.Stream()
    eager = ev.EvConvNet(net)
    with torch.cuda.stream(side):
        captured = ev.EvConvNet(net, stream=side)
        static_in = torch.empty_like(_dev(frames[0]))
        static_in.copy_(_dev(frames[0]))
        captured.reset(static_in)
        static_in.copy_(_dev(frames[1]))
        captured.step_frame(static_in)          # one eager step first (warm-up outside the capture)
    side.synchronize()
    eager.reset(_dev(frames[0]))
    eager.step_frame(_dev(frames[1]))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        captured.step_frame(static_in)
    # capture does not execute: the state is still that of frame 1
    for t in range(2, 10):
        eager.step_frame(_dev(frames[t]))
        with torch.cuda.stream(side):
            static_in.copy_(_dev(frames[t]))
        side.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        a, b = eager.outputs()[0], captured.outputs()[0]
        assert torch.equal(a["y"], b["y"]) and torch.equal(a["dy"], b["dy"]), f"replay {t - 1}"
        assert int(a["count"]) == int(b["count"])
        for i in watch:
            np.testing.assert_array_equal(eager.state(i, ev.STATE_Z), captured.state(i, ev.STATE_Z))
    del graph
    eager.destroy()
    captured.destroy()


# --------------------------------------------------------------------------- random graphs

@pytest.mark.parametrize("seed", range(9))
def test_random_wide_graphs_all_contraction_modes(seed):
    """Random graphs over the matrix-core paths (ragged channel counts, fused epilogue adds, fused
    up-sampling gather, gates, heads), each in one of the three contraction modes, all nodes at
    every step against the oracle."""
    rng = np.random.default_rng(100 + seed)
    mode = ["f32", "split", "bf16"][seed % 3]
    net = wl.net_random_wide(seed)
    if mode == "bf16":
        net = wl.with_weight_dtype(dataclasses.replace(net, weights=wl.round_to_bf16(net.weights)), wl.WD_BF16)
    elif mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    _say(f"random wide graph {seed}: {len(net.nodes)} nodes, {mode}")
    g = ev.EvConvNet(net)
    names = [g.kernel_name(i) for i in range(len(net.nodes))]
    g.destroy()
    want = {"f32": "conv_mfma_f32", "split": "conv_mfma_f32_split_bf16x3", "bf16": "conv_mfma_bf16"}[mode]
    # (the up-sampling is folded into the gather of 32-channel-chunk convs only: some seeds keep it apart)
    assert names.count(want) >= 4 and "fused_into_conv_epilogue" in names, names
    x = rng.standard_normal((net.in_c, net.in_h, net.in_w)).astype(np.float32)
    frames = [x]
    for t in range(6):
        m = rng.random((1, net.in_h, net.in_w)) < (0.04 if t != 3 else 0.6)
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    if mode == "bf16":
        run_stream(net, frames[0], frames[1:], "frame", tol=2e-2, label=f"wide{seed}", max_flips=40, frobenius=True)
    else:
        run_stream(net, frames[0], frames[1:], "frame", label=f"wide{seed}", max_flips=40)


@pytest.mark.parametrize("seed,h,w", [(0, 84, 108), (6, 84, 108), (7, 72, 136), (19, 100, 92), (2, 84, 108)])
def test_upsampling_folded_into_conv_weights(seed, h, w):
    """A 5 x 5 conv reading a x2 up-sampling at sizes where the stored tensor has tiles away from
    the border: those run per output phase with folded 4 x 4 weights, the border tiles through the
    interpolating gather (ragged tile rows and columns, one or two output-channel blocks, 32-96
    input channels, fp32 and split products; bf16-declared weights must not fold).  All nodes at
    every step against the oracle; then the same frames with folding switched off: identical
    touched sets, values apart by rounding only."""
    rng = np.random.default_rng(300 + seed)
    mode = ["f32", "split", "bf16"][seed % 3]
    net = wl.net_random_wide(seed, h, w)
    if mode == "bf16":
        net = wl.with_weight_dtype(dataclasses.replace(net, weights=wl.round_to_bf16(net.weights)), wl.WD_BF16)
    elif mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    _say(f"folded up-sampling, random wide graph {seed} at {h}x{w}: {len(net.nodes)} nodes, {mode}")
    up = [i for i, n in enumerate(net.nodes) if n.op == wl.OP_UPSAMPLE2X][0]
    g = ev.EvConvNet(net)
    assert g.kernel_name(up) == ("fused_into_conv_gather" if mode == "bf16" else "fused_into_conv_weights")
    g.destroy()
    x = rng.standard_normal((net.in_c, h, w)).astype(np.float32)
    frames = [x]
    for t in range(5):
        m = rng.random((1, h, w)) < (0.03 if t != 2 else 0.5)
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    if mode == "bf16":
        run_stream(net, frames[0], frames[1:], "frame", tol=2e-2, label=f"fold{seed}", max_flips=40, frobenius=True)
        return
    run_stream(net, frames[0], frames[1:], "frame", label=f"fold{seed}", max_flips=40)
    folded, recomputed = ev.EvConvNet(net), ev.EvConvNet(net)
    plain = ev.EvConvNet(net, flags=ev.FLAG_NO_FOLD)
    assert plain.kernel_name(up) == "fused_into_conv_gather"
    conv = [i for i, n in enumerate(net.nodes) if n.op == wl.OP_CONV2D and n.in0 == up][0]
    for t, f in enumerate(frames):
        for net_ in (folded, plain, recomputed):
            (net_.reset if t == 0 else net_.step_frame)(_dev(f))
        if t == 0:
            recomputed.set_mode(ev.MODE_DENSE_RECOMPUTE)
        np.testing.assert_array_equal(folded.state(conv, ev.STATE_OCC_TOUCHED), plain.state(conv, ev.STATE_OCC_TOUCHED))
        za, zb = folded.state(conv, ev.STATE_Z), plain.state(conv, ev.STATE_Z)
        assert np.abs(za - zb).max() <= 2e-5 * np.abs(zb).max(), (t, np.abs(za - zb).max(), np.abs(zb).max())
    # a regular forward pass through the folded kernels, as a reset and as a dense-recompute step: same bits
    folded.reset(_dev(frames[-1]))
    np.testing.assert_array_equal(folded.state(conv, ev.STATE_Z), recomputed.state(conv, ev.STATE_Z))
    for net_ in (folded, plain, recomputed):
        net_.destroy()


def test_folded_upsampling_ragged_channels_and_output_node():
    """Folded up-sampling conv with an input channel count that is not a multiple of the chunk
    (36: the last chunk is zero-padded in the patch and in the folded weight sets), three blocks
    of output channels, a bias, and the conv being a network output itself."""
    _say("folded up-sampling conv, 36 -> 96 channels on 40x56 -> 80x112, network output")
    b = wl._NetBuilder("fold_ragged", 4, 40, 56, 4242, bias=True)
    x = b.conv(-1, 36, 3)
    u = b.simple(wl.OP_UPSAMPLE2X, x)
    b.conv(u, 96, 5, act=wl.ACT_RELU, out=1)
    net = b.finish()
    g = ev.EvConvNet(net)
    assert [g.kernel_name(i) for i in range(3)] == ["conv_narrow_mfma_f32", "fused_into_conv_weights", "conv_mfma_f32"]
    g.destroy()
    rng = np.random.default_rng(4242)
    x = rng.standard_normal((4, 40, 56)).astype(np.float32)
    frames = [x]
    for t in range(5):
        m = rng.random((1, 40, 56)) < (0.02 if t != 3 else 0.7)
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    run_stream(net, frames[0], frames[1:], "frame", label="fold-ragged", max_flips=10)


@pytest.mark.parametrize("h,w,ci,co", [(18, 18, 32, 32), (17, 33, 32, 32), (26, 19, 96, 32), (48, 21, 32, 64)])
def test_folded_upsampling_smallest_interiors(h, w, ci, co):
    """Stored tensors that have just one tile away from the border (18 rows: sites 8-15 lie 2 or
    more from both edges), none (17 rows), or a single row / column of them."""
    _say(f"folded up-sampling conv, stored tensor {h}x{w}, {ci} -> {co} channels")
    b = wl._NetBuilder("fold_small", 4, h, w, 7 * h + w, bias=True)
    x = b.conv(-1, ci, 3)
    u = b.simple(wl.OP_UPSAMPLE2X, x)
    d = b.conv(u, co, 5)
    b.conv(d, 2, 1, 1, 0, wl.ACT_NONE, out=1)
    net = b.finish()
    g = ev.EvConvNet(net)
    assert g.kernel_name(u) == ("fused_into_conv_weights" if min(h, w) >= 18 else "fused_into_conv_gather")
    g.destroy()
    rng = np.random.default_rng(h * 100 + w)
    x = rng.standard_normal((4, h, w)).astype(np.float32)
    frames = [x]
    for t in range(4):
        m = rng.random((1, h, w)) < (0.03 if t != 2 else 0.6)
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    run_stream(net, frames[0], frames[1:], "frame", label=f"fold{h}x{w}", max_flips=10)


@pytest.mark.parametrize("h,w,ci,co,mode", [(18, 18, 32, 32, "f32"), (20, 45, 64, 40, "split"), (59, 68, 32, 64, "f32"), (60, 66, 96, 64, "split"),
                                            (64, 65, 32, 64, "f32"), (57, 72, 33, 64, "f32"), (66, 63, 40, 50, "split")])
def test_folded_upsampling_borders(h, w, ci, co, mode):
    """The folded kernel's border taps, in half tiles (the first two) and in whole ones: last tiles of one to
    eight rows and columns (one block of the upper rows or of eight rows of four columns where the image
    holds no more), ragged channels.  Against the oracle at every step; then infinite and NaN increments on
    the border: not a site further than the oracle's."""
    _say(f"folded up-sampling, borders: stored tensor {h}x{w}, {ci} -> {co} channels, {mode}")
    b = wl._NetBuilder("fold_border", ci, h, w, 11 * h + w, bias=True)
    u = b.simple(wl.OP_UPSAMPLE2X, -1)
    c = b.conv(u, co, 5, 1, act=wl.ACT_NONE, out=1)
    net = b.finish()
    if mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    gpu, ora = ev.EvConvNet(net), Oracle(net)
    assert gpu.kernel_name(u) == "fused_into_conv_weights"
    rng = np.random.default_rng(h)
    x0 = rng.standard_normal((ci, h, w)).astype(np.float32)
    edge = np.zeros((1, h, w), bool)
    edge[:, [0, 1, -2, -1]] = edge[:, :, [0, 1, -2, -1]] = True
    rep = cmp.Report()
    gpu.reset(_dev(x0))
    ora.reset(x0)
    # fp32 sums of at most 25 * 96 products (2^-24 each, random) and 16-bit parts (2^-16 a product)
    tol = 2e-6 if mode == "f32" else 4e-5
    for q in (1.0, 0.1, 0.02):
        d = (rng.standard_normal(x0.shape) * ((rng.random((1, h, w)) < q) & (edge | (q > 0.05)))).astype(np.float32)
        gpu.step(_dev(d))
        ora.step_increment(d)
        z, zr = gpu.state(c, ev.STATE_Z).astype(np.float64), ora.z(c)
        assert np.abs(z - zr).max() <= tol * np.abs(zr).max(), np.abs(z - zr).max() / np.abs(zr).max()
        cmp.compare_outputs(gpu, ora, rep)
        cmp.compare_node(gpu, ora, c, rep, tol=tol, act_scale=np.abs(zr).max())
    if mode == "f32":
        d = np.zeros_like(x0)
        d[0, 0, 3], d[1, h - 1, 0], d[2, h // 2, w - 1], d[3, h - 1, w - 2], d[4, 1, w // 2] = np.inf, -np.inf, np.inf, np.nan, -np.inf
        gpu.step(_dev(d))
        ora.step_increment(d)
        # (which of infinity and NaN depends on whether the taps of a source meet before or after its products)
        z, zr = gpu.state(c, ev.STATE_Z), ora.z(c)
        np.testing.assert_array_equal(np.isfinite(z), np.isfinite(zr))
        assert 0 < np.isfinite(zr).sum() < zr.size
    gpu.destroy()


class _Stream:
    """One stream of a net, for the comparisons with an oracle."""

    def __init__(self, gpu, stream):
        self._gpu, self._stream = gpu, stream

    def state(self, node, kind):
        return self._gpu.state(node, kind, self._stream)

    def site_list(self, node):
        return self._gpu.site_list(node, self._stream)

    def outputs(self):
        return self._gpu.outputs(self._stream)

    def __getattr__(self, name):
        return getattr(self._gpu, name)


@pytest.mark.parametrize("h,w,ci,co,streams,mode,kind", [
    (60, 66, 32, 64, 1, "f32", "add"), (62, 65, 32, 64, 1, "split", "add"), (64, 65, 32, 64, 1, "f32", "two adds"),
    (59, 68, 32, 64, 1, "split", "two adds"), (60, 67, 32, 64, 1, "f32", "sparsify"), (63, 66, 32, 64, 1, "split", "sparsify"),
    (57, 67, 32, 64, 1, "f32", "sigmoid"), (66, 60, 32, 64, 1, "split", "tanh"), (28, 35, 32, 96, 3, "f32", "add"),
    (34, 36, 32, 64, 3, "split", "sparsify"), (20, 27, 32, 32, 2, "f32", "two adds")])
def test_folded_upsampling_epilogue_stages(h, w, ci, co, streams, mode, kind):
    """What runs in the folded kernel's epilogue (ADDs whose other input is active beyond the conv's touched sites,
    a sparsification layer, activations other than ReLU) on the sites of whole tiles, with last tiles of
    one to eight columns and rows (eight rows of four columns where there are no more) and with streams whose
    number decides between whole and half tiles (the last case: half).  Exact arithmetic (dyadic weights and
    increments): sets, lists and sums equal the fp64 oracle's; with sigmoid and tanh to fp32 accuracy."""
    _say(f"folded up-sampling, epilogue: {kind}, stored tensor {h}x{w}, {ci} -> {co} channels, {mode}, {streams} streams")
    smooth = kind in ("sigmoid", "tanh")
    b = wl._NetBuilder("fold_stages", ci, h, w, 3, sparsify=kind == "sparsify", sparsify_k=0.5)
    u2 = b.simple(wl.OP_UPSAMPLE2X, -1)
    s = b.conv(u2, co, 7, act=wl.ACT_NONE, sparsify_input=False)
    u = b.simple(wl.OP_UPSAMPLE2X, -1)
    c = b.conv(u, co, 5, act=wl.ACT_SIGMOID if kind == "sigmoid" else wl.ACT_NONE, out=int(kind == "sigmoid"), sparsify_input=False)
    stages = []
    if kind != "sigmoid":
        stages.append(b.simple(wl.OP_ADD, s, c, act={"tanh": wl.ACT_TANH, "two adds": wl.ACT_NONE}.get(kind, wl.ACT_RELU), out=1))
    if kind == "two adds":
        stages.append(b.simple(wl.OP_ADD, stages[0], s, act=wl.ACT_RELU, out=1))
    if kind == "sparsify":
        b.conv(stages[0], 16, 1, 1, 0, act=wl.ACT_NONE, out=1)
        stages.append(stages[0] + 1)
    net = b.finish()
    rng = np.random.default_rng(h * w)
    wts = net.weights.copy()
    for nd in net.nodes:
        if nd.op == wl.OP_CONV2D:
            n = nd.c_out * nd.c_in * nd.k * nd.k
            wts[nd.w_off:nd.w_off + n] = rng.integers(-1, 2, n) * (rng.random(n) < 2.0 / (nd.k * nd.k)) / 8.0
    net.weights = wts
    if mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    gpu = ev.EvConvNet(net, n_streams=streams)
    assert gpu.kernel_name(u) == "fused_into_conv_weights" and [gpu.kernel_name(i) for i in stages] == ["fused_into_conv_epilogue"] * len(stages)
    oras = [Oracle(net) for _ in range(streams)]
    dev = lambda a: _dev(a if streams > 1 else a[0])
    value = lambda q: (rng.integers(-8, 9, (streams, ci, h, w)) / 4.0 * (rng.random((streams, 1, h, w)) < q)).astype(np.float32)
    x0, rep, tol = value(1.0), cmp.Report(), 1e-5 if smooth else 1e-7
    gpu.reset(dev(x0))
    for k, ora in enumerate(oras):
        ora.reset(x0[k])
    for q in (0.004, 1.0, 0.002, 0.05):
        d = value(q)
        gpu.step(dev(d))
        for k, ora in enumerate(oras):
            ora.step_increment(d[k])
            cmp.compare_outputs(_Stream(gpu, k), ora, rep, tol)
            for i in range(len(net.nodes)):
                cmp.compare_node(_Stream(gpu, k), ora, i, rep, tol=tol, exact_sets=not smooth)
    assert rep.flips <= (200 if smooth else 0), rep.flips_by_node
    gpu.destroy()


# --------------------------------------------------------------------------- recurrent state

def _running_sum_net(c, h, w):
    nodes = [
        wl.Node(wl.OP_DELAY, wl.ACT_NONE, 1, -1, c, c, 1, 1, 0, -1, -1, 0),
        wl.Node(wl.OP_ADD, wl.ACT_NONE, -1, 0, c, c, 1, 1, 0, -1, -1, 1),
    ]
    return wl.Net("running_sum", c, h, w, nodes, np.zeros(0, np.float32))


def test_delay_running_sum_bit_exact_against_fp32_oracle():
    """s(n) = x(n) + s(n-1) through a DELAY node: every operation is a single fp32 add or
    subtraction, so the GPU must agree bit for bit with the oracle run in binary32, through
    incremental steps, refreshes (regular passes that keep the state) and the steps after them."""
    _say("recurrent running sum, bit-exact, with refreshes")
    c, h, w = 3, 9, 19
    net = _running_sum_net(c, h, w)
    rng = np.random.default_rng(11)
    x = rng.standard_normal((c, h, w)).astype(np.float32)
    gpu, ora = ev.EvConvNet(net), Oracle(net, fp32_state=True)
    gpu.set_refresh_period(4)
    gpu.reset(_dev(x))
    ora.reset(x)
    for t in range(1, 11):
        m = rng.random((1, h, w)) < 0.1
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        gpu.step_frame(_dev(x))
        (ora.refresh if t % 4 == 0 else ora.step_frame)(x)
        import torch
        torch.cuda.synchronize()
        for i in (0, 1):
            np.testing.assert_array_equal(gpu.state(i, ev.STATE_Z).view(np.uint32) if i == 0 else 0,
                                          ora.z(i).astype(np.float32).view(np.uint32) if i == 0 else 0,
                                          err_msg=f"step {t} node {i} accumulated value")
        y = gpu.outputs()[0]["y"].cpu().numpy()
        np.testing.assert_array_equal(y.view(np.uint32), np.transpose(ora.y(1), (2, 0, 1)).astype(np.float32).view(np.uint32),
                                      err_msg=f"step {t} output")
        if t % 4:
            for i in (0, 1):
                np.testing.assert_array_equal(cmp.words_to_mask(gpu.state(i, ev.STATE_OCC), h, w), ora.mask(i),
                                              err_msg=f"step {t} node {i} active set")
                on = ora.mask(i).astype(bool)
                np.testing.assert_array_equal(gpu.state(i, ev.STATE_DY)[on].view(np.uint32),
                                              ora.dy(i).astype(np.float32)[on].view(np.uint32), err_msg=f"step {t} node {i} increment")
    gpu.destroy()


@pytest.mark.parametrize("mode,in_c", [("f32", 4), ("split", 4), ("f32", 5), ("split", 5)])
def test_convlstm_cell_against_oracle(mode, in_c):
    """A ConvLSTM cell (gates on the matrix cores, products, tanh, two recurrent states) and a
    1 x 1 head: all nodes at every step.  With 5 input channels the gate convs read 37 channels
    (not a multiple of four)."""
    net = wl.net_convlstm(41, in_c=in_c, h=24, w=40, hidden=32, out_c=2)
    if mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    _say(f"ConvLSTM cell, {mode}, {in_c}x24x40, hidden 32")
    g = ev.EvConvNet(net)
    names = [g.kernel_name(i) for i in range(len(net.nodes))]
    g.destroy()
    assert names[0] == names[1] == "delay", names
    assert names.count("conv_mfma_f32" if mode == "f32" else "conv_mfma_f32_split_bf16x3") == 4, names
    rng = np.random.default_rng(12)
    x = rng.standard_normal((in_c, 24, 40)).astype(np.float32)
    frames = [x]
    for t in range(8):
        m = rng.random((1, 24, 40)) < 0.05
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    run_stream(net, frames[0], frames[1:], "frame", label=f"convlstm-{mode}", max_flips=40)


def test_convlstm_refresh_and_dense_recompute_keep_the_state():
    """Regular forward passes in mid-stream (refresh period; dense-recompute mode) keep the
    recurrent state: outputs follow the oracle's refresh()."""
    _say("ConvLSTM cell with refresh period 3, and in dense-recompute mode")
    net = wl.net_convlstm(42, in_c=4, h=16, w=24, hidden=32, out_c=2)
    rng = np.random.default_rng(13)
    x = rng.standard_normal((4, 16, 24)).astype(np.float32)
    frames = [x]
    for t in range(7):
        m = rng.random((1, 16, 24)) < 0.1
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    import torch
    for which in ("refresh", "dense"):
        gpu, ora = ev.EvConvNet(net), Oracle(net)
        if which == "refresh":
            gpu.set_refresh_period(3)
        else:
            gpu.set_mode(ev.MODE_DENSE_RECOMPUTE)
        gpu.reset(_dev(frames[0]))
        ora.reset(frames[0])
        out = ora.outputs[0]
        for t in range(1, 8):
            gpu.step_frame(_dev(frames[t]))
            regular = which == "dense" or t % 3 == 0
            (ora.refresh if regular else ora.step_frame)(frames[t])
            torch.cuda.synchronize()
            y = gpu.outputs()[0]["y"].cpu().numpy()
            ref = np.transpose(ora.y(out), (2, 0, 1))
            assert np.abs(y - ref).max() <= TOL * np.abs(ref).max(), f"{which} step {t}: {np.abs(y - ref).max():.3e}"
            for d in (0, 1):
                z, zr = gpu.state(d, ev.STATE_Z).astype(np.float64), ora.z(d)
                assert np.abs(z - zr).max() <= TOL * max(np.abs(zr).max(), 1e-30), f"{which} step {t} state {d}"
        gpu.destroy()


def test_convgru_cell_against_oracle():
    """A ConvGRU cell: two sigmoid gates, r * h', a tanh candidate on [x, r * h'], 1 - z, two
    products and an add, one recurrent state; all nodes at every step."""
    net = wl.net_convgru(43, in_c=4, h=24, w=40, hidden=32, out_c=2)
    _say("ConvGRU cell, 4x24x40, hidden 32")
    rng = np.random.default_rng(14)
    x = rng.standard_normal((4, 24, 40)).astype(np.float32)
    frames = [x]
    for t in range(8):
        m = rng.random((1, 24, 40)) < 0.05
        x = (x + rng.standard_normal(x.shape).astype(np.float32) * m).astype(np.float32)
        frames.append(x)
    run_stream(net, frames[0], frames[1:], "frame", label="convgru", max_flips=40)


def test_large_frame_720p():
    """A 720p sensor (5 x 720 x 1280, 14400 tiles; widths 16..128): launch shapes and offsets far
    from the benchmark's size, two steps against the oracle."""
    _say("UNet depth net on a 5x720x1280 frame, width 16, reset + 2 steps")
    net = wl.net_unet_depth(1003, h=720, w=1280, width=16)
    frames = list(wl.stream_voxel(1010, 720, 1280, 2, 0.01, n_prim=12))
    rep = run_stream(net, frames[0], frames[1:], "frame", check_nodes_at={2}, label="720p", max_flips=400)
    _say(f"720p: max rel z err {rep.max_rel_z:.2e}, y err {rep.max_rel_y:.2e}, flips {rep.flips}")


@pytest.mark.gpu
@pytest.mark.parametrize("c_in,c_out,h,w,wd,streams,one_launch", [
    (64, 128, 56, 56, wl.WD_F32, 1, True),        # neither conv splits its channels
    (128, 256, 28, 28, wl.WD_F32, 1, True),       # the first one does
    (256, 512, 14, 14, wl.WD_F32_SPLIT, 1, True),
    (64, 64, 27, 31, wl.WD_BF16, 1, True),
    (128, 48, 21, 9, wl.WD_F32_SPLIT, 3, True),   # c_out that is not whole blocks, several streams
    (1024, 64, 17, 15, wl.WD_F32, 1, False),      # both would split their channels
    (96, 128, 28, 28, wl.WD_F32, 1, False),       # channels that are not whole chunks
    (64, 128, 130, 120, wl.WD_F32, 1, False),     # too many workgroups for the common variant
])
def test_shortcut_conv_in_the_first_convs_launch(c_in, c_out, h, w, wd, streams, one_launch):
    """A stride-2 block whose 1 x 1 shortcut runs in the launch of its first conv: every sum, set and
    result bit for bit as with separate launches, and fp32 sums against the oracle, through a reset,
    sparse steps, a dense step and a step without a change."""
    b = wl._NetBuilder("block", c_in, h, w, c_in + c_out, bias=True, bf16=wd == wl.WD_BF16)
    first = b.conv(-1, c_out, 3, 2)
    second = b.conv(first, c_out, 3, 1, act=wl.ACT_NONE)
    short = b.conv(-1, c_out, 1, 2, 0, act=wl.ACT_NONE)
    b.simple(wl.OP_ADD, second, short, act=wl.ACT_RELU, out=1)
    net = wl.with_weight_dtype(b.finish(), wd)
    one, apart = ev.EvConvNet(net, n_streams=streams), ev.EvConvNet(net, n_streams=streams, flags=ev.FLAG_NO_FUSION)
    oras = [Oracle(net) for _ in range(streams)]
    rng = np.random.default_rng(c_in)
    x0 = rng.standard_normal((streams, c_in, h, w)).astype(np.float32)
    for g in (one, apart):
        g.profile_begin(100)
        g.reset(_dev(x0 if streams > 1 else x0[0]))
        g.profile_end()
    assert (one.node_time(short)[1] == 0) == one_launch and apart.node_time(short)[1] == 1
    for q, o in enumerate(oras):
        o.reset(x0[q])
    for share in (None, 0.02, 0.3, 1.0, 0.0, 0.01):
        if share is not None:
            d = (rng.standard_normal(x0.shape) * (rng.random((streams, 1, h, w)) < share)).astype(np.float32)
            for g in (one, apart):
                g.step(_dev(d if streams > 1 else d[0]))
            for q, o in enumerate(oras):
                o.step_increment(d[q])
        for q, o in enumerate(oras):
            for i in range(len(net.nodes)):
                for kind in (ev.STATE_Z, ev.STATE_OCC, ev.STATE_OCC_TOUCHED, ev.STATE_COUNT):
                    np.testing.assert_array_equal(one.state(i, kind, q), apart.state(i, kind, q), err_msg=f"share {share} node {i} state {kind}")
                if wd == wl.WD_F32:
                    z, zr = one.state(i, ev.STATE_Z, q).astype(np.float64), o.z(i)
                    assert np.abs(z - zr).max() <= 2e-6 * np.abs(zr).max(), f"share {share} node {i} z"
            for key in ("y", "dy"):
                np.testing.assert_array_equal(one.outputs(q)[0][key].cpu().numpy(), apart.outputs(q)[0][key].cpu().numpy())
    one.destroy()
    apart.destroy()


def _merged_net(kind):
    """(net, {conv: launches of its own}, {node: how it is run}) for launches that hold several convs."""
    if kind == "lstm":             # gates of a real cell
        net = wl.net_convlstm(1008, h=96, w=88, hidden=64)
        gates = [i for i, n in enumerate(net.nodes) if n.op == wl.OP_CONV2D][:4]
        return net, dict(zip(gates, (1, 0, 0, 0))), {}
    pair = kind.startswith("pair")
    c, h, w = (64, 56, 50) if pair else (32, 136, 124)
    b = wl._NetBuilder(kind, c, h, w, 11, bias=True, sparsify="sparsify" in kind, sparsify_k=0.05)
    if kind == "delay":            # a delay of the second conv between the two: it must see the previous step's
        x = b.conv(-1, c, 3)
        prev = b.delay(c, like=x)
        y = b.conv(-1, c, 3, act=wl.ACT_TANH)
        b.close_delay(prev, y)
        b.simple(wl.OP_ADD, b.simple(wl.OP_MUL, x, prev), y, act=wl.ACT_RELU, out=1)
        return b.finish(), {x: 1, y: 1}, {}
    if kind == "mixed":            # kernels of different size, and two of each: a launch per size
        ids = [b.conv(-1, c, k, act=wl.ACT_RELU, out=1) for k in (3, 1, 5, 7, 5, 1, 3, 7)]
        return b.finish(), dict(zip(ids, (1, 1, 1, 1, 0, 0, 0, 0))), {}
    early = b.simple(wl.OP_MAXPOOL, -1, k=3, stride=2, pad=1) if pair else b.simple(wl.OP_ACT, -1, act=wl.ACT_TANH)
    x = b.conv(-1, c, 3, 2 if pair else 1, act=wl.ACT_RELU)
    y = b.conv(-1, c, 1 if pair else 3, 2 if pair else 1, act=wl.ACT_NONE)
    if "add" in kind:              # both convs host an ADD with an earlier tensor, the second one two
        sx, sy = b.simple(wl.OP_ADD, x, early, act=wl.ACT_RELU, out=1), b.simple(wl.OP_ADD, early, y)
        sy2 = b.simple(wl.OP_ADD, sy, early, act=wl.ACT_TANH, out=1)
        fused = (sx, sy, sy2)
    else:                          # both host a sparsification layer, the second one behind an ADD
        sy = b.simple(wl.OP_ADD, y, early, act=wl.ACT_RELU)
        b.conv(x, 16, 1, 1, 0, out=1)
        b.conv(sy, 16, 1, 1, 0, out=1)
        fused = [sy] + [i for i, n in enumerate(b.nodes) if n.op == wl.OP_SPARSIFY]
        assert len(fused) == 3
    return b.finish(), {x: 1, y: 0}, {i: "fused_into_conv_epilogue" for i in fused}


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["lstm", "delay", "mixed", "batch_add", "batch_sparsify", "pair_add", "pair_sparsify"])
def test_merged_convs_with_epilogues_and_delays(kind):
    """Convs in one launch that host ADDs and sparsification layers, of each kernel's variant, beside DELAY nodes:
    every sum, set and result bit for bit as with a launch per node, through sparse and dense steps, a dense
    recompute and a refresh."""
    net, launches, names = _merged_net(kind)
    one, apart = ev.EvConvNet(net), ev.EvConvNet(net, flags=ev.FLAG_NO_FUSION)
    rng = np.random.default_rng(len(kind))
    shape = (net.in_c, net.in_h, net.in_w)
    x0 = _dev(rng.standard_normal(shape))
    for g in (one, apart):
        g.profile_begin(200)
        g.reset(x0)
        g.profile_end()
    assert {i: one.node_time(i)[1] for i in launches} == launches
    assert {i: one.kernel_name(i) for i in names} == names
    for step, (share, mode) in enumerate(((0.01, ev.MODE_INCREMENTAL), (0.4, ev.MODE_INCREMENTAL), (0.1, ev.MODE_DENSE_RECOMPUTE),
                                          (0.02, ev.MODE_INCREMENTAL), (0.0, ev.MODE_INCREMENTAL), (1.0, ev.MODE_INCREMENTAL),
                                          (0.02, ev.MODE_INCREMENTAL))):
        d = _dev(rng.standard_normal(shape) * (rng.random((1,) + shape[1:]) < share))
        for g in (one, apart):
            g.set_refresh_period(1 if step == 3 else 0)
            g.set_mode(mode)
            g.step(d)
        for i, n in enumerate(net.nodes):
            kinds = [ev.STATE_DY, ev.STATE_OCC, ev.STATE_OCC_TOUCHED, ev.STATE_COUNT]
            if n.op in (wl.OP_CONV2D, wl.OP_MUL, wl.OP_SPARSIFY, wl.OP_DELAY) or n.act != wl.ACT_NONE:
                kinds.append(ev.STATE_Z)
            for k in kinds:
                u, v = one.state(i, k), apart.state(i, k)
                if k == ev.STATE_DY and share < 1.0 and mode == ev.MODE_INCREMENTAL and step != 3:
                    touched = one.site_list(i)   # (an increment is defined at the active sites only)
                    u, v = u.reshape(-1, u.shape[-1])[touched], v.reshape(-1, v.shape[-1])[touched]
                np.testing.assert_array_equal(u, v, err_msg=f"step {step} node {i} state {k}")
        for o, r in zip(one.outputs(), apart.outputs()):
            for key in ("y", "dy"):
                np.testing.assert_array_equal(o[key].cpu().numpy(), r[key].cpu().numpy(), err_msg=f"step {step} node {o['node']} {key}")
    one.destroy()
    apart.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("c_in,c_out,h,w,k2,stride,between", [
    (64, 128, 40, 40, 1, 2, "act"),      # a block's shortcut; its ADD's other input is an activation of the first conv
    (36, 64, 120, 112, 3, 1, "mul"),     # two gate convs, the other input a product of the first one
    (36, 64, 120, 112, 3, 1, "concat"),  # the other input a narrow conv's
    (36, 64, 120, 112, 3, 1, "sum"),     # ADD of both
])
def test_a_conv_that_hosts_an_add_is_not_moved_away_from_it(c_in, c_out, h, w, k2, stride, between):
    """A conv that could run in an earlier conv's launch, but whose epilogue computes an ADD with an input that
    exists only after that launch, keeps its own: the ADD is no launch of its own, results are those of
    separate launches."""
    b = wl._NetBuilder("host", c_in, h, w, c_in + k2, bias=True)
    first = b.conv(-1, c_out, 3, stride)
    if between == "act":
        other = b.simple(wl.OP_ACT, first, act=wl.ACT_TANH)
    elif between == "mul":
        other = b.simple(wl.OP_MUL, first, first)
    elif between == "concat":
        other = b.simple(wl.OP_CONCAT, b.conv(first, c_out - 8, 1, 1, 0), b.conv(first, 8, 1, 1, 0))
    else:
        other = first
    late = b.conv(-1, c_out, k2, stride, act=wl.ACT_NONE)
    total = b.simple(wl.OP_ADD, other, late, act=wl.ACT_RELU, out=1)
    net = b.finish()
    one, apart = ev.EvConvNet(net), ev.EvConvNet(net, flags=ev.FLAG_NO_FUSION)
    assert one.kernel_name(total) == "fused_into_conv_epilogue"
    rng = np.random.default_rng(c_in)
    x0 = rng.standard_normal((c_in, h, w)).astype(np.float32)
    for g in (one, apart):
        g.profile_begin(100)
        g.reset(_dev(x0))
        g.profile_end()
    assert one.node_time(late)[1] == 1 and one.node_time(total)[1] == 0
    for share in (0.02, 1.0, 0.0, 0.3):
        d = _dev(rng.standard_normal(x0.shape) * (rng.random((1, h, w)) < share))
        for g in (one, apart):
            g.step(d)
        for i in range(len(net.nodes)):
            for kind in (ev.STATE_Z, ev.STATE_OCC, ev.STATE_OCC_TOUCHED, ev.STATE_COUNT):
                if kind != ev.STATE_Z or net.nodes[i].op not in (wl.OP_CONCAT,):
                    np.testing.assert_array_equal(one.state(i, kind), apart.state(i, kind), err_msg=f"share {share} node {i} state {kind}")
        for key in ("y", "dy"):
            np.testing.assert_array_equal(one.outputs()[0][key].cpu().numpy(), apart.outputs()[0][key].cpu().numpy())
    one.destroy()
    apart.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("heads,launches,streams", [
    ([2, 2], [0, 1], 1),
    ([2, 2, 2, 2, 2], [0, 0, 0, 1, 1], 1),   # more than a batch holds
    ([1, 3, 1, 4, 8], [0, 0, 1, 1, 1], 2),   # 3 and 4 channels share a variant, 8 stands alone
])
def test_prediction_heads_in_one_launch(heads, launches, streams):
    """Heads that nothing reads run in the launch of the last of their variant: results, sets and public
    outputs bit for bit as from launches of their own, in regular passes, steps and dense recompute.
    (A head that another node reads keeps its own launch: the last one of the net here.)"""
    b = wl._NetBuilder("heads", 4, 43, 29, sum(heads), bias=True)
    x, at = -1, []
    for i, c in enumerate(heads):
        x = b.conv(x, 12 + 8 * i, 3, 2 if i in (1, 3) else 1)
        at.append(b.conv(x, c, 1, 1, 0, act=(wl.ACT_NONE, wl.ACT_SIGMOID)[i % 2], out=1))
    own = b.conv(x, 2, 1, 1, 0, act=wl.ACT_NONE, out=1)
    b.simple(wl.OP_ACT, own, act=wl.ACT_RELU, out=1)
    net = b.finish()
    one, apart = ev.EvConvNet(net, n_streams=streams), ev.EvConvNet(net, n_streams=streams, flags=ev.FLAG_NO_FUSION)
    rng = np.random.default_rng(len(heads))
    shape = (4, 43, 29) if streams == 1 else (streams, 4, 43, 29)
    x0 = _dev(rng.standard_normal(shape))
    for g in (one, apart):
        g.profile_begin(100)
        g.reset(x0)
        g.profile_end()
    assert [int(one.node_time(i)[1]) for i in at + [own]] == launches + [1]
    assert all(apart.node_time(i)[1] == 1 for i in at + [own])
    for share, mode in ((None, 0), (0.02, ev.MODE_INCREMENTAL), (1.0, ev.MODE_INCREMENTAL), (0.0, ev.MODE_INCREMENTAL),
                        (0.1, ev.MODE_DENSE_RECOMPUTE), (0.05, ev.MODE_INCREMENTAL)):
        if share is not None:
            d = _dev(rng.standard_normal(shape) * (rng.random(shape[:-3] + (1, 43, 29)) < share))
            for g in (one, apart):
                g.set_mode(mode)
                g.step(d)
        for q in range(streams):
            for i in range(len(net.nodes)):
                for kind in (ev.STATE_Z, ev.STATE_OCC, ev.STATE_OCC_TOUCHED, ev.STATE_COUNT):
                    np.testing.assert_array_equal(one.state(i, kind, q), apart.state(i, kind, q), err_msg=f"share {share} node {i} state {kind}")
            for o, r in zip(one.outputs(q), apart.outputs(q)):
                for key in ("y", "dy"):
                    np.testing.assert_array_equal(o[key].cpu().numpy(), r[key].cpu().numpy(), err_msg=f"share {share} node {o['node']} {key}")
    one.destroy()
    apart.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("c_in,c_out,h,w,wd,streams,n,launches", [
    (69, 64, 96, 88, wl.WD_F32, 1, 4, [1, 0, 0, 0]),          # a ConvLSTM cell's gates: ragged channels
    (32, 40, 61, 75, wl.WD_F32, 2, 5, [1, 0, 0, 0, 1]),       # one more than a batch, ragged blocks and tiles
    (32, 64, 160, 176, wl.WD_F32_SPLIT, 2, 2, [1, 0]),
    (36, 64, 160, 176, wl.WD_BF16, 2, 3, [1, 0, 0]),
    (36, 64, 96, 96, wl.WD_BF16, 1, 2, [1, 0]),               # 576 workgroups per conv
    (36, 64, 320, 328, wl.WD_BF16, 1, 2, [1, 0]),             # 6560
    (32, 32, 24, 24, wl.WD_F32, 1, 2, [1, 1]),                # too few workgroups: another variant
])
def test_convs_of_one_tensor_in_one_launch(c_in, c_out, h, w, wd, streams, n, launches):
    """Gate convs that read the same tensor run in one launch: every sum, set and result bit for bit as
    with separate launches, through a reset and steps; an ADD of two of them keeps its place in the
    later one's epilogue (and these two their own launches)."""
    b = wl._NetBuilder("gates", c_in, h, w, c_in + c_out, bias=True, bf16=wd == wl.WD_BF16)
    acts = (wl.ACT_SIGMOID, wl.ACT_TANH, wl.ACT_RELU, wl.ACT_SIGMOID, wl.ACT_NONE)
    gates = [b.conv(-1, c_out, 3, 1, act=acts[i]) for i in range(n)]
    prod = b.simple(wl.OP_MUL, gates[0], gates[1])
    b.simple(wl.OP_ADD, prod, gates[-1], act=wl.ACT_RELU, out=1)
    net = wl.with_weight_dtype(b.finish(), wd)
    one, apart = ev.EvConvNet(net, n_streams=streams), ev.EvConvNet(net, n_streams=streams, flags=ev.FLAG_NO_FUSION)
    rng = np.random.default_rng(c_in + n)
    shape = (c_in, h, w) if streams == 1 else (streams, c_in, h, w)
    x0 = _dev(rng.standard_normal(shape))
    for g in (one, apart):
        g.profile_begin(100)
        g.reset(x0)
        g.profile_end()
    assert [int(one.node_time(i)[1]) for i in gates] == launches
    assert all(apart.node_time(i)[1] == 1 for i in gates)
    for share in (None, 0.01, 0.4, 1.0, 0.0):
        if share is not None:
            d = _dev(rng.standard_normal(shape) * (rng.random(shape[:-3] + (1, h, w)) < share))
            for g in (one, apart):
                g.step(d)
        for q in range(streams):
            for i in range(len(net.nodes)):
                kinds = (ev.STATE_Z, ev.STATE_OCC, ev.STATE_OCC_TOUCHED, ev.STATE_COUNT)
                for kind in kinds:
                    np.testing.assert_array_equal(one.state(i, kind, q), apart.state(i, kind, q), err_msg=f"share {share} node {i} state {kind}")
            for key in ("y", "dy"):
                np.testing.assert_array_equal(one.outputs(q)[0][key].cpu().numpy(), apart.outputs(q)[0][key].cpu().numpy())
    one.destroy()
    apart.destroy()
    # an ADD of two of the convs
    b = wl._NetBuilder("sum", c_in, h, w, 3)
    x, y = b.conv(-1, c_out, 3, 1, act=wl.ACT_NONE), b.conv(-1, c_out, 3, 1, act=wl.ACT_NONE)
    total = b.simple(wl.OP_ADD, x, y, act=wl.ACT_RELU, out=1)
    assert ev.EvConvNet(b.finish()).kernel_name(total) == "fused_into_conv_epilogue"


@pytest.mark.gpu
@pytest.mark.parametrize("make", [lambda: wl.net_flow(5, h=48, w=64), lambda: wl.net_resnet18(6, h=64, w=64)], ids=["flow", "resnet18"])
def test_in1_of_one_input_operators_is_ignored(monkeypatch, make):
    """The description's in1 belongs to operators with two inputs: whatever the others hold there (an index
    far beyond the nodes, one of a real node), the plan and the results are the same."""
    net = make()
    marshal, rng = ev.marshal_desc, np.random.default_rng(2)
    shape = (net.in_c, net.in_h, net.in_w)
    x0 = _dev(rng.standard_normal(shape))
    d = _dev(rng.standard_normal(shape) * (rng.random((1,) + shape[1:]) < 0.05))
    seen = []
    for other in (-1, 1 << 20, -(1 << 30), 0):
        def with_in1(*a, **kw):
            desc, nodes = marshal(*a, **kw)
            for n in nodes:
                if n.op not in (wl.OP_ADD, wl.OP_CONCAT, wl.OP_MUL, wl.OP_DELAY):
                    n.in1 = other
            return desc, nodes
        monkeypatch.setattr(ev, "marshal_desc", with_in1)
        g = ev.EvConvNet(net)
        g.profile_begin(2 * len(net.nodes) + 8)
        g.reset(x0)
        g.step(d)
        g.profile_end()
        seen.append(([g.node_time(i)[1] for i in range(len(net.nodes))],
                     [(o["y"].cpu().numpy(), o["dy"].cpu().numpy()) for o in g.outputs()]))
        g.destroy()
    for launches, outs in seen[1:]:
        assert launches == seen[0][0]
        for (y, dy), (y0, dy0) in zip(outs, seen[0][1]):
            np.testing.assert_array_equal(y, y0)
            np.testing.assert_array_equal(dy, dy0)


@pytest.mark.gpu
@pytest.mark.parametrize("c,h,w", [
    (4, 5, 9),     # one vector per thread (as on all maps of few tiles: the channels are split over workgroups)
    (3, 9, 13),    # channels that are not whole vectors
    (20, 8, 8),
    (64, 7, 11),
    (76, 3, 5),    # several workgroups per tile, the last one narrower
    (32, 71, 87),  # 396 tiles of the up-sampled map: two vectors per thread
    (44, 71, 87),  # four, or twice two; the last ones beyond the tile's sites for some threads
    (72, 71, 87),  # as many, and a second, narrower workgroup per tile
    (18, 71, 87),  # 16 single channels, and two
])
def test_elementwise_operators_by_channel_count(c, h, w):
    """Up-sampling stored and inside a concatenation, concatenation, sum, product and activation over the
    numbers of vectors per thread and channel counts that are not whole vectors, on odd sizes."""
    b = wl._NetBuilder("ew", c, h, w, 7 + c)
    up = b.simple(wl.OP_UPSAMPLE2X, -1, out=1)
    two = b.conv(up, 2, 1, 1, 0, act=wl.ACT_NONE)
    fused = b.simple(wl.OP_UPSAMPLE2X, -1)
    cat_up = b.simple(wl.OP_CONCAT, fused, two, out=1)
    cat = b.simple(wl.OP_CONCAT, two, up, out=1)
    act = b.simple(wl.OP_ACT, up, act=wl.ACT_TANH, out=1)
    total = b.simple(wl.OP_ADD, up, act, act=wl.ACT_RELU, out=1)
    b.simple(wl.OP_MUL, up, total, out=1)
    net = b.finish()
    assert ev.EvConvNet(net).kernel_name(fused) == "fused_into_concat_gather" and cat_up < cat
    rng = np.random.default_rng(c)
    x0 = rng.standard_normal((c, h, w)).astype(np.float32)
    incs = [(rng.standard_normal((c, h, w)) * (rng.random((1, h, w)) < p)).astype(np.float32) for p in (0.05, 0.0, 1.0, 0.2)]
    # (a value-pruned set may differ where an increment is rounded to nothing on one side only)
    run_stream(net, x0, incs, "increment", tol=1e-5, label=f"elementwise {c} x {h} x {w}", max_flips=4)


@pytest.mark.gpu
@pytest.mark.parametrize("c", [3, 20, 68])
def test_pooling_windows_on_many_tiles(c):
    """Windows of 2, 3 and 5 sites where a thread has several elements (more than 384 tiles), whole vectors and
    single channels, at the ragged borders of the map."""
    h, w = 141, 179
    b = wl._NetBuilder("pools", c, h, w, c)
    for k, pad in ((2, 1), (3, 1), (5, 2)):
        b.simple(wl.OP_MAXPOOL, -1, k=k, stride=1, pad=pad, out=1)
    net = b.finish()
    rng = np.random.default_rng(c)
    x0 = rng.standard_normal((c, h, w)).astype(np.float32)
    incs = [(rng.standard_normal((c, h, w)) * (rng.random((1, h, w)) < p)).astype(np.float32) for p in (0.01, 0.0, 1.0)]
    run_stream(net, x0, incs, "increment", tol=1e-6, label=f"pools {c}", max_flips=0)


@pytest.mark.parametrize("ci,co,k,s,hw,streams", [
    (128, 64, 3, 1, (8, 8), 1), (192, 40, 3, 1, (17, 9), 1), (448, 32, 3, 1, (9, 7), 1),    # 2, 3, 7 chunks of 64
    (256, 96, 1, 1, (5, 20), 1), (128, 32, 3, 2, (15, 30), 1), (192, 64, 1, 2, (11, 9), 1),  # 1 x 1, stride 2
    (64, 32, 5, 2, (20, 9), 1), (96, 48, 5, 2, (33, 16), 1), (1024, 128, 3, 1, (16, 24), 1),  # chunks of 32; several chunks each
    (256, 32, 3, 1, (11, 13), 3)])
def test_channels_split_over_workgroups(ci, co, k, s, hw, streams):
    """Convs on maps of a few tiles split their input channels over several workgroups, the last of
    which to arrive runs the epilogue (residual ADD, ReLU, a second conv behind it).  Sparse steps
    with untouched tiles, tiles that only the ADD's other input touches, a dense step, a refresh;
    every net twice in the same state (run-to-run identical whatever the order of arrival)."""
    import torch
    h, w = hw
    _say(f"channels split over workgroups: {ci} -> {co}, {k} x {k} stride {s}, {h} x {w}, {streams} streams")
    b = wl._NetBuilder("ksplit", ci, h, w, ci + k, bias=True)
    a = b.conv(-1, co, 1, s, 0, act=wl.ACT_RELU)
    c = b.conv(-1, co, k, s, act=wl.ACT_NONE)
    b.simple(wl.OP_ADD, c, a, act=wl.ACT_RELU, out=1)
    net = b.finish()
    rng = np.random.default_rng(ci + k)
    nets = [ev.EvConvNet(net, n_streams=streams) for _ in range(2)]
    assert nets[0].kernel_name(c) == "conv_mfma_f32"
    oras = [Oracle(net) for _ in range(streams)]
    rep = cmp.Report()
    x0 = rng.standard_normal((streams, ci, h, w)).astype(np.float32)
    for g in nets:
        g.reset(_dev(x0 if streams > 1 else x0[0]))
    for q, o in enumerate(oras):
        o.reset(x0[q])
    for t in range(5):
        m = rng.random((streams, 1, h, w)) < (1.0 if t == 2 else 0.02)
        d = (rng.standard_normal(x0.shape) * m).astype(np.float32)
        for g in nets:
            g.step(_dev(d if streams > 1 else d[0]))
        torch.cuda.synchronize()
        for q, o in enumerate(oras):
            o.step_increment(d[q])
            for i in range(len(net.nodes)):
                z, zr = nets[0].state(i, ev.STATE_Z, q).astype(np.float64), o.z(i)
                assert np.abs(z - zr).max() <= 2e-6 * np.abs(zr).max(), f"step {t} node {i} z"
                np.testing.assert_array_equal(nets[0].state(i, ev.STATE_OCC_TOUCHED, q), nets[1].state(i, ev.STATE_OCC_TOUCHED, q))
                np.testing.assert_array_equal(z, nets[1].state(i, ev.STATE_Z, q).astype(np.float64))
        if streams == 1:
            for i in range(len(net.nodes)):
                cmp.compare_node(nets[0], oras[0], i, rep)
    assert rep.flips <= 2
    for g in nets:
        g.destroy()


@pytest.mark.parametrize("k,s,ci,co", [(3, 1, 64, 32), (5, 2, 16, 64), (5, 1, 20, 32), (1, 1, 96, 32)])
def test_fp32_contraction_keeps_24_bits_and_ieee_specials(k, s, ci, co):
    """The fp32 matrix-core conv writes every operand as three bf16 parts.  Against 64 bits the sums
    are within 2^-21 of the sum of the absolute products (three dropped partial products of 2^-25
    each at most, and fp32 accumulation); finite values that a bf16 would round to infinity stay
    finite; infinities and NaN come out where IEEE products put them, zero weights included."""
    _say(f"fp32 contraction: {k} x {k} stride {s}, {ci} -> {co}")
    h, w = 18, 21
    b = wl._NetBuilder("bits24", ci, h, w, 5 + k)
    b.conv(-1, co, k, s, act=wl.ACT_NONE, out=1)
    net = b.finish()
    rng = np.random.default_rng(9)
    wt = net.weights
    wt *= np.exp2(rng.integers(-6, 7, wt.shape)).astype(np.float32)     # mixed magnitudes
    wt[rng.random(wt.shape) < 0.1] = 0.0
    wt[rng.random(wt.shape) < 0.1] = 1.0                                # one part only
    x = (rng.standard_normal((ci, h, w)) * np.exp2(rng.integers(-20, 8, (ci, h, w)))).astype(np.float32)
    gpu, ora, absolute = ev.EvConvNet(net), Oracle(net), Oracle(dataclasses.replace(net, weights=np.abs(wt)))
    assert gpu.kernel_name(0) == "conv_mfma_f32"
    gpu.reset(_dev(x))
    ora.reset(x)
    absolute.reset(np.abs(x))
    err = np.abs(gpu.state(0, ev.STATE_Z).astype(np.float64) - ora.z(0))
    assert (err <= 2.0 ** -21 * absolute.z(0)).all(), float((err / absolute.z(0)).max())
    # 3.4e38 is above the largest value that a bf16 rounds to a finite one
    wt[:] = np.where(np.abs(wt) > 0, np.sign(wt) * 1e-3, 0).astype(np.float32)
    gpu.destroy()
    gpu, ora = ev.EvConvNet(net), Oracle(net)
    x0 = np.zeros((ci, h, w), np.float32)
    d = np.zeros_like(x0)
    d[0, 2, 3], d[ci - 1, 2, 12], d[1, 9, 4], d[2, 15, 15] = 3.4e38, -np.finfo(np.float32).max, np.inf, np.nan
    d[3, 9, 12] = -np.inf
    gpu.reset(_dev(x0))
    ora.reset(x0)
    gpu.step(_dev(d))
    ora.step_increment(d)
    z, zr = gpu.state(0, ev.STATE_Z).astype(np.float64), ora.z(0)
    np.testing.assert_array_equal(np.isnan(z), np.isnan(zr))
    np.testing.assert_array_equal(z[np.isinf(zr)], zr[np.isinf(zr)])
    fin = np.isfinite(zr)
    assert np.isfinite(z[fin]).all() and np.abs(z[fin] - zr[fin]).max() <= 2.0 ** -21 * np.abs(zr[fin]).max()
    assert np.abs(zr[fin]).max() > 1e35
    gpu.destroy()


@pytest.mark.parametrize("c,co,hw", [(8, 4, (9, 65)), (9, 5, (8, 8)), (64, 16, (17, 23)), (65, 17, (7, 9)), (200, 101, (9, 5))])
def test_wide_inputs_and_wide_outputs(c, co, hw):
    """The increment builder's two forms (up to 8 channels: strips of 64 columns; more: tiles x 64
    channels whose words meet through a scratch word) and the output integration's two (up to 4
    channels, more): cached frame, increment, words and lists bit-exact through frames, supplied
    increments, a refresh and dense recompute."""
    h, w = hw
    _say(f"wide inputs and outputs: {c} -> {co}, {h} x {w}")
    b = wl._NetBuilder("wide", c, h, w, c + co, bias=True)
    b.conv(-1, co, 1, 1, 0, act=wl.ACT_RELU, out=1)
    net = b.finish()
    rng = np.random.default_rng(c)
    gpu, ora, rep = ev.EvConvNet(net), Oracle(net), cmp.Report()
    x = rng.standard_normal((c, h, w)).astype(np.float32)
    gpu.reset(_dev(x))
    ora.reset(x)
    cmp.compare_outputs(gpu, ora, rep)
    for t in range(6):
        d = np.zeros_like(x)
        for _ in range(3):   # single elements: a site's bit comes from one channel group only
            d[rng.integers(c), rng.integers(h), rng.integers(w)] = rng.standard_normal()
        if t == 3:
            d = (rng.standard_normal(x.shape) * (rng.random((1, h, w)) < 0.5)).astype(np.float32)
        if t % 2:
            gpu.step(_dev(d))
            ora.step_increment(d)
            x = x + d
        else:
            x = x + d
            gpu.step_frame(_dev(x))
            ora.step_frame(x)
        cmp.compare_input_stage(gpu, ora, rep)
        cmp.compare_outputs(gpu, ora, rep)
        cmp.compare_node(gpu, ora, 0, rep)
    y_inc = gpu.outputs()[0]["y"].clone()
    gpu.set_mode(ev.MODE_DENSE_RECOMPUTE)
    gpu.step(_dev(np.zeros_like(x)))       # a regular pass of the cached frame
    y_dense = gpu.outputs()[0]["y"]
    assert float((y_dense - y_inc).abs().max()) <= 1e-5 * max(1.0, float(y_dense.abs().max()))
    gpu.destroy()


@pytest.mark.parametrize("ci,co,k,hw", [(32, 48, 5, (31, 45)), (64, 80, 3, (33, 50)), (64, 32, 1, (9, 7)), (96, 128, 3, (141, 150)),
                                        (32, 128, 5, (140, 153)), (160, 256, 5, (60, 66))])
def test_stride2_convs_in_larger_channel_chunks(ci, co, k, hw):
    """Stride-2 layers of few workgroups take chunks of 64 (3 x 3, 1 x 1) or 32 channels; with eight
    waves per workgroup and, from 512 workgroups on, four.  Ragged sizes, sparse and dense steps."""
    h, w = hw
    b = wl._NetBuilder("s2", ci, h, w, ci + k, bias=True)
    b.conv(-1, co, k, 2, act=wl.ACT_RELU, out=1)
    net = b.finish()
    rng = np.random.default_rng(ci + h)
    x0 = rng.standard_normal((ci, h, w)).astype(np.float32)
    incs = [(rng.standard_normal(x0.shape) * (rng.random((1, h, w)) < d)).astype(np.float32) for d in (0.01, 1.0, 0.02)]
    run_stream(net, x0, incs, "increment", label=f"stride 2, {ci} -> {co}, {k} x {k}", max_flips=3, tol=1e-5)


@pytest.mark.parametrize("mode", ["f32", "split", "bf16"])
@pytest.mark.parametrize("ci,k", [(33, 3), (47, 5), (69, 3), (96, 1), (37, 7)])
def test_last_channel_chunk_of_one_group(mode, ci, k):
    """Input channels that leave the last chunk of 32 with 1..16 channels: its units are the taps
    alone (in fp32 mode the signs of its stored weights follow).  The same conv behind an
    up-sampling that is not folded keeps both groups."""
    _say(f"last chunk of one group: {ci} channels, {k} x {k}, {mode}")
    h, w = 26, 35
    b = wl._NetBuilder("tail", ci, h, w, ci, bf16=mode == "bf16", bias=True)
    c = b.conv(-1, 40, k, 1, act=wl.ACT_RELU)
    u = b.simple(wl.OP_UPSAMPLE2X, -1)
    d = b.conv(u, 32, k, 1, act=wl.ACT_NONE)
    b.simple(wl.OP_ACT, c, act=wl.ACT_NONE, out=1)
    b.simple(wl.OP_ACT, d, act=wl.ACT_RELU, out=1)
    net = b.finish()
    if mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    rng = np.random.default_rng(ci)
    x0 = rng.standard_normal((ci, h, w)).astype(np.float32)
    dx = [(rng.standard_normal(x0.shape) * (rng.random((1, h, w)) < q)).astype(np.float32) for q in (0.02, 1.0)]
    for flags in (0, ev.FLAG_NO_FUSION):
        gpu, ora = ev.EvConvNet(net, flags=flags), Oracle(net)
        gpu.reset(_dev(x0))
        ora.reset(x0)
        for inc in dx:
            gpu.step(_dev(inc))
            ora.step_increment(inc)
            for i in (c, d):
                z, zr = gpu.state(i, ev.STATE_Z).astype(np.float64), ora.z(i)
                lim = {"f32": 2e-6, "split": 1e-4, "bf16": 2e-2}[mode]
                assert np.linalg.norm(z - zr) <= lim * np.linalg.norm(zr), (flags, i)
        gpu.destroy()


@pytest.mark.parametrize("ci,co", [(256, 1), (20, 2), (19, 3), (64, 4), (48, 5), (33, 7), (16, 8)])
def test_pointwise_heads_of_one_to_eight_channels(ci, co):
    """Prediction heads: output channels rounded up to 1, 2, 4 or 8 inside the kernel, input channels
    that do and do not fill the unrolled pieces."""
    _say(f"pointwise head: {ci} -> {co}")
    b = wl._NetBuilder("head", ci, 11, 18, ci + co, bias=True)
    b.conv(-1, co, 1, 1, 0, act=wl.ACT_SIGMOID if co % 2 else wl.ACT_NONE, out=1)
    net = b.finish()
    rng = np.random.default_rng(ci)
    x0 = rng.standard_normal((ci, 11, 18)).astype(np.float32)
    incs = [(rng.standard_normal(x0.shape) * (rng.random((1, 11, 18)) < q)).astype(np.float32) for q in (0.05, 1.0, 0.1)]
    run_stream(net, x0, incs, "increment", label=f"head {ci} -> {co}", max_flips=6, tol=1e-5)


@pytest.mark.parametrize("mode", ["split", "bf16"])
@pytest.mark.parametrize("ci,co,k,hw", [(32, 32, 5, (256, 250)), (64, 40, 3, (190, 185)), (96, 32, 1, (250, 256))])
def test_stride2_sums_do_not_depend_on_the_channel_chunk(mode, ci, co, k, hw):
    """bf16 and split modes: a stride-2 layer of 512 to 1024 half-tile workgroups takes chunks of 32
    channels, with more streams (more workgroups) chunks of 16; the sums come out bit for bit the
    same, sparse and dense."""
    import torch
    h, w = hw
    _say(f"stride-2 chunks: {ci} -> {co}, {k} x {k}, {mode}")
    b = wl._NetBuilder("s2order", ci, h, w, ci + k, bf16=mode == "bf16")
    b.conv(-1, co, k, 2, act=wl.ACT_NONE, out=1)
    net = wl.with_weight_dtype(b.finish(), wl.WD_F32_SPLIT if mode == "split" else wl.WD_BF16)
    c, oh, ow = ev.EvConvNet(net).shape(0)
    per_stream = -(-oh // 8) * -(-ow // 8) * -(-co // 32) * 2
    streams = 1024 // per_stream + 1
    assert 512 <= per_stream <= 1024
    rng = np.random.default_rng(ci)
    x0 = rng.standard_normal((ci, h, w)).astype(np.float32)
    d = (rng.standard_normal(x0.shape) * (rng.random((1, h, w)) < 0.05)).astype(np.float32)
    one, many = ev.EvConvNet(net), ev.EvConvNet(net, n_streams=streams)
    one.reset(_dev(x0))
    many.reset(_dev(np.stack([x0] * streams)))
    np.testing.assert_array_equal(one.state(0, ev.STATE_Z), many.state(0, ev.STATE_Z, streams - 1))
    one.step(_dev(d))
    many.step(_dev(np.stack([d] * streams)))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(one.state(0, ev.STATE_Z), many.state(0, ev.STATE_Z, streams - 1))
    one.destroy()
    many.destroy()


def _conv64(net, x, co, ci, k, s):
    import torch
    w = torch.from_numpy(net.weights[:co * ci * k * k].reshape(co, ci, k, k)).double()
    run = lambda a, b: torch.nn.functional.conv2d(torch.from_numpy(a).double()[None], b, None, s, k // 2)[0].numpy()
    return run(x, w), run(np.abs(x), w.abs())


@pytest.mark.parametrize("k,s,ci,co", [(3, 1, 64, 32), (5, 2, 32, 48), (1, 1, 40, 32)])
@pytest.mark.parametrize("exp", [-100, -112, -120, -133, -141])
def test_fp32_contraction_of_tiny_weights(k, s, ci, co, exp):
    """fp32 matrix-core conv, weights around 2^exp, where a bf16 (no bits below 2^-133) runs out of
    them: in every channel, and in one channel beside ordinary weights.  Sums within 2^-21 of the sum
    of the absolute products as for other weights (and two steps of the subnormal range for results
    in it); an infinite increment times a nonzero weight is infinite."""
    _say(f"tiny weights: {k} x {k} stride {s}, {ci} -> {co}, 2^{exp}")
    h, w = 18, 21
    b = wl._NetBuilder("tinyw", ci, h, w, 5 + k)
    b.conv(-1, co, k, s, act=wl.ACT_NONE, out=1)
    net = b.finish()
    base = net.weights.copy().reshape(co, ci, k, k)
    rng = np.random.default_rng(3)
    x = (rng.standard_normal((ci, h, w)) * 2.0 ** 12).astype(np.float32)
    mixed = base.copy()
    mixed[:, 2] = (base[:, 2].astype(np.float64) * 2.0 ** exp).astype(np.float32)
    mixed[:, 2] = np.where(mixed[:, 2] == 0, np.float32(1.4e-45), mixed[:, 2])
    only2 = np.zeros_like(x)
    only2[2] = x[2]
    for wt, xx in (((base.astype(np.float64) * 2.0 ** exp).astype(np.float32), x), (mixed, only2), (mixed, x)):
        net.weights[:] = wt.ravel()
        ref, absolute = _conv64(net, xx, co, ci, k, s)
        gpu = ev.EvConvNet(net)
        assert gpu.kernel_name(0) == "conv_mfma_f32"
        gpu.reset(_dev(xx))
        z = gpu.state(0, ev.STATE_Z).astype(np.float64).transpose(2, 0, 1)
        assert (np.abs(z - ref) <= 2.0 ** -21 * absolute + 2.0 ** -148).all(), float(np.abs(z - ref).max())
        gpu.destroy()
    gpu = ev.EvConvNet(net)
    x0 = np.zeros_like(x)
    d = x0.copy()
    d[2, 8, 8] = np.inf
    gpu.reset(_dev(x0))
    gpu.step(_dev(d))
    z = gpu.state(0, ev.STATE_Z)[8 // s, 8 // s]
    np.testing.assert_array_equal(z, np.copysign(np.inf, mixed[:, 2, k // 2, k // 2]))
    gpu.destroy()


@pytest.mark.parametrize("exp", [-60, -109, -118, -127, -140])
def test_fp32_contraction_of_tiny_increments(exp):
    """Increments around 2^exp: exact down to 2^-110, below it each is rounded to a multiple of 2^-133
    (an error of at most 2^-134 times the weight), the bound that the header states."""
    _say(f"tiny increments: 2^{exp}")
    ci, co, k, h, w = 48, 32, 3, 18, 21
    b = wl._NetBuilder("tinyx", ci, h, w, 8)
    b.conv(-1, co, k, 1, act=wl.ACT_NONE, out=1)
    net = b.finish()
    net.weights[:] *= np.float32(4096)
    x = (np.random.default_rng(4).standard_normal((ci, h, w)) * 2.0 ** exp).astype(np.float32)
    ref, absolute = _conv64(net, x, co, ci, k, 1)
    step = _conv64(net, (x != 0).astype(np.float32), co, ci, k, 1)[1] * 2.0 ** -134
    gpu = ev.EvConvNet(net)
    gpu.reset(_dev(x))
    err = np.abs(gpu.state(0, ev.STATE_Z).astype(np.float64).transpose(2, 0, 1) - ref)
    assert (err <= 2.0 ** -21 * absolute + (step if exp < -104 else 0.0)).all(), float((err / absolute).max())
    gpu.destroy()


def test_fp32_weights_too_far_apart_take_the_vector_path():
    """Weights with bits below 2^-133 beside weights of 2^112: no power of two holds both in three bf16
    parts; the conv runs on the vector kernel, as with an infinite weight."""
    ci, co, h, w = 32, 32, 9, 11
    b = wl._NetBuilder("apart", ci, h, w, 8)
    b.conv(-1, co, 3, 1, act=wl.ACT_NONE, out=1)
    net = b.finish()
    wt = net.weights.reshape(co, ci, 3, 3)
    wt[:, 0], wt[:, 1] = 1e-41, 2.0 ** 113
    x = np.zeros((ci, h, w), np.float32)
    x[0, 4, 4], x[1, 2, 8] = 2.0 ** 120, 2.0 ** -100
    ref, absolute = _conv64(net, x, co, ci, 3, 1)
    gpu = ev.EvConvNet(net)
    assert gpu.kernel_name(0) == "conv_valu_f32"
    gpu.reset(_dev(x))
    err = np.abs(gpu.state(0, ev.STATE_Z).astype(np.float64).transpose(2, 0, 1) - ref)
    assert (err <= 2.0 ** -21 * absolute + 2.0 ** -148).all()
    gpu.destroy()


def test_fp32_products_just_below_the_largest_value():
    """A product whose operands' high parts multiply to more than the largest fp32 value while the
    product itself does not: finite, and within 2^-21 of the exact one."""
    rng = np.random.default_rng(6)
    top = float(np.finfo(np.float32).max)
    for t in range(40):
        b = wl._NetBuilder("top", 16, 4, 4, t)
        b.conv(-1, 32, 1, 1, 0, act=wl.ACT_NONE, out=1)
        net = b.finish()
        a = np.float32(min(2.0 ** rng.uniform(-0.01, 127.9), top))
        net.weights[:] = 0
        wt = np.float32((0.99, 0.996, 0.998, 0.9999)[t % 4] * top / float(a))
        net.weights.reshape(32, 16)[:, 3] = wt
        x = np.zeros((16, 4, 4), np.float32)
        x[3, 1, 2] = -a
        gpu = ev.EvConvNet(net)
        gpu.reset(_dev(x))
        z = gpu.state(0, ev.STATE_Z)[1, 2].astype(np.float64)
        want = -float(a) * float(wt)
        assert (np.abs(z - want) <= 2.0 ** -21 * abs(want)).all(), (t, float(a), float(wt), z[0])
        gpu.destroy()


@pytest.mark.parametrize("mode", ["f32", "split"])
def test_folded_weights_that_would_overflow_are_not_folded(mode):
    """A 5x5 conv behind an up-sampling whose finite weights add up to more than the largest fp32 value
    when the up-sampling is folded into them: the results are those of the unfolded form, finite."""
    _say(f"fold overflow, {mode}")
    b = wl._NetBuilder("foldmax", 32, 40, 35, 3)
    u = b.simple(wl.OP_UPSAMPLE2X, -1)
    c = b.conv(u, 32, 5, 1, act=wl.ACT_NONE, out=1)
    net = b.finish()
    if mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    net.weights.reshape(32, 32, 5, 5)[:, 7] = 3e38
    rng = np.random.default_rng(1)
    x0 = np.zeros((32, 40, 35), np.float32)
    d = (rng.standard_normal(x0.shape) * 1e-3).astype(np.float32)
    gpu, ora = ev.EvConvNet(net), Oracle(net)
    gpu.reset(_dev(x0))
    ora.reset(x0)
    gpu.step(_dev(d))
    ora.step_increment(d)
    z, zr = gpu.state(c, ev.STATE_Z).astype(np.float64), ora.z(c)
    assert np.abs(z - zr).max() <= (3e-6 if mode == "f32" else 1e-4) * np.abs(zr).max()
    gpu.destroy()


@pytest.mark.parametrize("ci,co,k,s,hw,streams", [(16, 32, 1, 1, 96, 1), (48, 32, 1, 1, 96, 1), (80, 32, 1, 1, 96, 1),
                                                  (64, 128, 1, 2, 56, 16), (96, 32, 1, 1, 96, 1), (48, 32, 3, 1, 96, 1)])
def test_fp32_sums_have_no_error_of_one_sign(ci, co, k, s, hw, streams):
    """The matrix instruction's sums come out low; units whose weights are stored negated cancel that,
    and where a chunk is a single unit a second wave with negated weights.  Inputs as behind a
    ReLU; the mean signed error against 64 bits, over the mean magnitude, is below 5e-9 (with one sign throughout these layers are off by 1e-8 and more; the mean over 3e5 sums of
    random errors of 1.3e-7 varies by 2e-10)."""
    _say(f"signed error: {ci} -> {co}, {k} x {k} stride {s}, {streams} streams")
    rng = np.random.default_rng(ci)
    mean = []
    for seed in range(3):
        b = wl._NetBuilder("bias", ci, hw, hw, seed)
        b.conv(-1, co, k, s, act=wl.ACT_NONE, out=1)
        net = b.finish()
        x = np.abs(rng.standard_normal((streams, ci, hw, hw))).astype(np.float32)
        gpu = ev.EvConvNet(net, n_streams=streams)
        assert gpu.kernel_name(0) == "conv_mfma_f32"
        gpu.reset(_dev(x if streams > 1 else x[0]))
        for q in range(0, streams, 5):
            ref = _conv64(net, x[q], co, ci, k, s)[0]
            err = gpu.state(0, ev.STATE_Z, q).astype(np.float64).transpose(2, 0, 1) - ref
            mean.append((err.mean((1, 2)) / np.abs(ref).mean((1, 2))).mean())
        gpu.destroy()
    assert abs(np.mean(mean)) < 5e-9, np.mean(mean)


@pytest.mark.parametrize("ci,co,k,hw,streams", [(64, 32, 5, (9, 7), 1), (96, 40, 5, (17, 9), 1), (288, 96, 5, (20, 20), 1),
                                                (160, 32, 7, (8, 21), 1), (96, 32, 7, (5, 6), 3)])
def test_channels_of_large_kernels_split_over_workgroups(ci, co, k, hw, streams):
    """fp32 convs of 5 x 5 and more taps on few tiles split their channels in chunks of 32: against the
    oracle through sparse and dense steps, twice in the same state (run-to-run identical)."""
    import torch
    h, w = hw
    _say(f"channels of large kernels: {ci} -> {co}, {k} x {k}, {h} x {w}, {streams} streams")
    b = wl._NetBuilder("ksplit5", ci, h, w, ci + k, bias=True)
    b.conv(-1, co, k, 1, act=wl.ACT_RELU, out=1)
    net = b.finish()
    rng = np.random.default_rng(ci + k)
    nets = [ev.EvConvNet(net, n_streams=streams) for _ in range(2)]
    oras = [Oracle(net) for _ in range(streams)]
    x0 = rng.standard_normal((streams, ci, h, w)).astype(np.float32)
    for g in nets:
        g.reset(_dev(x0 if streams > 1 else x0[0]))
    for q, o in enumerate(oras):
        o.reset(x0[q])
    for t in range(4):
        m = rng.random((streams, 1, h, w)) < (1.0 if t == 2 else 0.03)
        d = (rng.standard_normal(x0.shape) * m).astype(np.float32)
        for g in nets:
            g.step(_dev(d if streams > 1 else d[0]))
        torch.cuda.synchronize()
        for q, o in enumerate(oras):
            o.step_increment(d[q])
            z, zr = nets[0].state(0, ev.STATE_Z, q).astype(np.float64), o.z(0)
            assert np.abs(z - zr).max() <= 2e-6 * np.abs(zr).max(), f"step {t}"
            np.testing.assert_array_equal(z, nets[1].state(0, ev.STATE_Z, q).astype(np.float64))
    for g in nets:
        g.destroy()


@pytest.mark.parametrize("mode", ["f32", "split", "bf16"])
@pytest.mark.parametrize("ci,co,hw,streams", [(64, 128, (181, 190), 1), (96, 32, (63, 70), 21), (32, 16, (360, 355), 1)])
def test_large_stride2_1x1_convs(mode, ci, co, hw, streams):
    """1 x 1 convs at stride 2 of more than 1024 half-tile workgroups, one or many streams: chunks of 32
    channels.  Against 64 bits (bf16 weights and increments: products are exact in fp32)."""
    _say(f"large 1 x 1 stride 2: {ci} -> {co}, {hw}, {streams} streams, {mode}")
    h, w = hw
    b = wl._NetBuilder("k1s2", ci, h, w, ci, bf16=mode == "bf16")
    b.conv(-1, co, 1, 2, act=wl.ACT_NONE, out=1)
    net = b.finish()
    if mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    x = np.random.default_rng(ci).standard_normal((streams, ci, h, w)).astype(np.float32)
    if mode == "bf16":
        x = wl.round_to_bf16(x)
    gpu = ev.EvConvNet(net, n_streams=streams)
    gpu.reset(_dev(x if streams > 1 else x[0]))
    for q in (0, streams - 1):
        ref, absolute = _conv64(net, x[q], co, ci, 1, 2)
        err = np.abs(gpu.state(0, ev.STATE_Z, q).astype(np.float64).transpose(2, 0, 1) - ref)
        # split: 2^-17 per operand and the dropped low x low product; the others: fp32 sums
        assert (err <= (2.0 ** -15 if mode == "split" else 2.0 ** -20) * absolute).all(), float((err / absolute).max())
    gpu.destroy()


@pytest.mark.parametrize("mode,ci,co,k,hw", [("bf16", 96, 96, 5, (100, 109)), ("bf16", 33, 64, 3, (136, 139)),
                                             ("split", 64, 128, 3, (95, 90)), ("split", 128, 96, 1, (159, 160))])
def test_launches_of_five_workgroups_per_cu(mode, ci, co, k, hw):
    """Four-wave half tiles whose launch takes one round less with five workgroups per CU: bit for bit
    what launches of another number of rounds (more streams) give, and within rounding of 64 bits."""
    _say(f"five workgroups per CU: {ci} -> {co}, {k} x {k}, {hw}, {mode}")
    h, w = hw
    n = -(-h // 8) * -(-w // 8) * -(-co // 32) * 2
    assert 1024 < n <= 1280 or 2048 < n <= 2560
    streams = next(q for q in range(2, 9) if not (1024 < q * n <= 1280 or 2048 < q * n <= 2560))
    b = wl._NetBuilder("five", ci, h, w, ci, bf16=mode == "bf16")
    b.conv(-1, co, k, 1, act=wl.ACT_RELU, out=1)
    net = b.finish()
    if mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    rng = np.random.default_rng(ci)
    x = wl.round_to_bf16(rng.standard_normal((ci, h, w)).astype(np.float32))
    d = (rng.standard_normal(x.shape) * (rng.random((1, h, w)) < 0.05)).astype(np.float32)
    one, many = ev.EvConvNet(net), ev.EvConvNet(net, n_streams=streams)
    one.reset(_dev(x))
    many.reset(_dev(np.stack([x] * streams)))
    ref, absolute = _conv64(net, x, co, ci, k, 1)
    err = np.abs(one.state(0, ev.STATE_Z).astype(np.float64).transpose(2, 0, 1) - ref)
    assert (err <= (2.0 ** -15 if mode == "split" else 2.0 ** -20) * absolute).all(), float((err / absolute).max())
    for _ in range(2):
        np.testing.assert_array_equal(one.state(0, ev.STATE_Z), many.state(0, ev.STATE_Z, streams - 1))
        np.testing.assert_array_equal(one.state(0, ev.STATE_OCC), many.state(0, ev.STATE_OCC, streams - 1))
        one.step(_dev(d))
        many.step(_dev(np.stack([d] * streams)))
    one.destroy()
    many.destroy()


def _sums_against_64_bits(mode, ci, co, k, s, h, w):
    b = wl._NetBuilder("small", ci, h, w, ci + k, bf16=mode == "bf16")
    b.conv(-1, co, k, s, act=wl.ACT_NONE, out=1)
    net = b.finish()
    if mode == "split":
        net = wl.with_weight_dtype(net, wl.WD_F32_SPLIT)
    rng = np.random.default_rng(ci + 10 * k + s)
    x = wl.round_to_bf16(rng.standard_normal((ci, h, w)).astype(np.float32))
    d = wl.round_to_bf16((rng.standard_normal(x.shape) * (rng.random((1, h, w)) < 0.05)).astype(np.float32))
    gpu = ev.EvConvNet(net)
    assert gpu.kernel_name(0).startswith("conv_mfma")
    gpu.reset(_dev(x))
    ref, absolute = _conv64(net, x, co, ci, k, s)
    bound = 2.0 ** -15 if mode == "split" else 2.0 ** -20   # of the sum of the absolute products
    err = np.abs(gpu.state(0, ev.STATE_Z).astype(np.float64).transpose(2, 0, 1) - ref)
    assert (err <= bound * absolute).all(), (h, w, float((err / absolute).max()))
    gpu.step(_dev(d))
    ref_d, absolute_d = _conv64(net, d, co, ci, k, s)
    err = np.abs(gpu.state(0, ev.STATE_Z).astype(np.float64).transpose(2, 0, 1) - ref - ref_d)
    assert (err <= bound * (absolute + absolute_d)).all(), (h, w, float((err / absolute).max()))
    gpu.destroy()


@pytest.mark.parametrize("k,s", [(1, 1), (2, 1), (3, 1), (1, 2), (2, 2), (3, 2)])
@pytest.mark.parametrize("mode,ci", [("f32", 24), ("f32", 48), ("f32", 69), ("f32", 96), ("f32", 128),
                                     ("split", 69), ("split", 128), ("bf16", 48), ("bf16", 96)])
def test_variants_for_small_kernels(mode, ci, k, s):
    """Kernels of one to three sites have variants that hold no more of a patch than they need: chunks of 16, 32
    (full and ragged), 64 and 128 channels, eight and four waves, channels split over workgroups; every
    site of odd maps against 64 bits, in a regular pass and a sparse step."""
    for h, w in ((13, 21), (201, 197)):
        _sums_against_64_bits(mode, ci, 40, k, s, h, w)


@pytest.mark.parametrize("mode,ci,co,k,hw", [("f32", 1632, 512, 1, (64, 30)), ("split", 1616, 512, 1, (61, 32)), ("f32", 224, 256, 3, (64, 61)),
                                             ("bf16", 208, 256, 3, (59, 64)), ("split", 1600, 512, 1, (64, 32))])
def test_variants_for_small_kernels_on_whole_tiles(mode, ci, co, k, hw):
    """... and long contractions of many blocks, which take whole tiles."""
    _sums_against_64_bits(mode, ci, co, k, 1, *hw)


@pytest.mark.parametrize("ci,co", [(20, 5), (19, 6), (64, 7), (36, 8), (20, 4), (20, 3), (40, 3), (64, 4), (33, 5)])
def test_pointwise_heads_on_many_tiles(ci, co):
    """Prediction heads of more than 1024 tiles: the variants of exactly three to eight channels, with the old
    values requested before and after dot products of fewer and more than 32 channels."""
    _say(f"pointwise head on many tiles: {ci} -> {co}")
    h, w = 257, 259
    b = wl._NetBuilder("heads", ci, h, w, ci + co, bias=True)
    b.conv(-1, co, 1, 1, 0, act=wl.ACT_SIGMOID if co % 2 else wl.ACT_NONE, out=1)
    net = b.finish()
    rng = np.random.default_rng(ci)
    x0 = rng.standard_normal((ci, h, w)).astype(np.float32)
    incs = [(rng.standard_normal(x0.shape) * (rng.random((1, h, w)) < q)).astype(np.float32) for q in (0.05, 1.0)]
    run_stream(net, x0, incs, "increment", label=f"head {ci} -> {co}", max_flips=12, tol=1e-5)


@pytest.mark.parametrize("c,hw", [(128, (50, 61)), (20, (9, 17)), (33, (56, 56)), (256, (64, 65))])
def test_elementwise_maps_split_over_the_channels(c, hw):
    """Elementwise nodes on maps of few tiles in workgroups of 16, 8 and 4 channel vectors (4-wide and
    single channels): activations, product and max-pool against the oracle, sparse and dense."""
    _say(f"elementwise channel split: {c} channels, {hw}")
    h, w = hw
    b = wl._NetBuilder("ewsplit", c, h, w, c)
    a = b.simple(wl.OP_ACT, -1, act=wl.ACT_RELU)
    m = b.simple(wl.OP_MUL, a, -1)
    b.simple(wl.OP_ADD, m, a, act=wl.ACT_TANH, out=1)
    b.simple(wl.OP_MAXPOOL, a, k=3, stride=2, pad=1, out=1)
    net = b.finish()
    rng = np.random.default_rng(c)
    x0 = rng.standard_normal((c, h, w)).astype(np.float32)
    incs = [(rng.standard_normal(x0.shape) * (rng.random((1, h, w)) < q)).astype(np.float32) for q in (0.03, 1.0, 0.02)]
    run_stream(net, x0, incs, "increment", label=f"elementwise {c}", max_flips=6, tol=1e-5)


@pytest.mark.parametrize("c,hw", [(9, (70, 1030)), (10, (131, 261)), (11, (4700, 7)), (12, (1030, 65)), (16, (130, 513)), (33, (500, 130)), (2, (40, 70)), (4, (33, 129))])
def test_wide_inputs_in_strips(c, hw):
    """Inputs of 9 to 12 channels on maps of 32768 sites and more (and of up to 8 on any) go through the strip form
    of the increment builder, all channels in flight; 16 and 33 channels on such maps in rows: cached frame,
    increment, words and lists bit-exact through frames and supplied increments, elements in single channels."""
    h, w = hw
    _say(f"wide inputs in strips: {c} channels, {h} x {w}")
    b = wl._NetBuilder("strips", c, h, w, c)
    b.conv(-1, 2, 1, 1, 0, act=wl.ACT_RELU, out=1)
    net = b.finish()
    rng = np.random.default_rng(c)
    gpu, ora, rep = ev.EvConvNet(net), Oracle(net), cmp.Report()
    x = rng.standard_normal((c, h, w)).astype(np.float32)
    gpu.reset(_dev(x))
    ora.reset(x)
    for t in range(4):
        d = np.zeros_like(x)
        for _ in range(40):
            d[rng.integers(c), rng.integers(h), rng.integers(w)] = rng.standard_normal()
        x = x + d
        if t % 2:
            gpu.step(_dev(d))
            ora.step_increment(d)
        else:
            gpu.step_frame(_dev(x))
            ora.step_frame(x)
        cmp.compare_input_stage(gpu, ora, rep)
        cmp.compare_outputs(gpu, ora, rep)
    gpu.destroy()


@pytest.mark.parametrize("c,hw,streams", [(9, (9, 63), 1), (16, (8, 64), 1), (17, (23, 65), 1), (20, (1, 130), 2), (32, (7, 7), 1),
                                          (36, (17, 96), 1), (66, (10, 97), 2), (1028, (3, 129), 1), (1063, (9, 10), 1),
                                          (9, (37, 5), 2), (68, (21, 8), 1), (33, (21, 9), 1), (20, (6, 16), 2), (40, (9, 17), 1), (13, (19, 32), 1),
                                          (16, (130, 33), 1)])
def test_wide_inputs_in_rows(c, hw, streams):
    """The increment builder for more than 8 channels (64 sites of a row, or of two to eight rows of a narrow
    image, x 16 or 32 channels, blocks of channels that meet in a scratch word, several blocks to a workgroup beyond 1024
    channels): cached frame, increment and words are those of the same subtraction and comparison in numpy, bit for bit."""
    h, w = hw
    _say(f"wide inputs in rows: {c} channels, {h} x {w}, {streams} streams")
    b = wl._NetBuilder("rows", c, h, w, c)
    b.conv(-1, 2, 1, 1, 0, act=wl.ACT_RELU, out=1)
    rng = np.random.default_rng(c)
    gpu = ev.EvConvNet(b.finish(), n_streams=streams)
    dev = lambda a: _dev(a if streams > 1 else a[0])
    x = rng.standard_normal((streams, c, h, w)).astype(np.float32)
    gpu.reset(dev(x))
    for t in range(5):
        d = np.zeros_like(x)
        for s in range(streams):
            for _ in range(2 + 20 * (t == 3)):  # single elements: a site's bit comes from one block only
                d[s, rng.integers(c), rng.integers(h), rng.integers(w)] = rng.standard_normal()
        if t % 2:
            gpu.step(dev(d))
            x, inc = x + d, d
        else:
            inc = (x + d) - x
            x = x + d
            gpu.step_frame(dev(x))
        for s in range(streams):
            mask = cmp.words_to_mask(gpu.state(-1, ev.STATE_OCC, s), h, w) != 0
            np.testing.assert_array_equal(mask, (inc[s] != 0).any(0))
            np.testing.assert_array_equal(gpu.state(-1, ev.STATE_DY, s), inc[s].transpose(1, 2, 0))
            np.testing.assert_array_equal(gpu.state(-1, ev.STATE_X_PREV, s), x[s])
            np.testing.assert_array_equal(gpu.site_list(-1, s), np.flatnonzero(mask))
    gpu.reset(dev(x))
    assert not any(gpu.state(-1, ev.STATE_OCC, s).any() for s in range(streams))
    gpu.destroy()


@pytest.mark.parametrize("mode", ["step", "dense"])
def test_large_wide_outputs_read_active_sites_only(mode):
    """An output of more than 12 Mi values (97 channels on 352 x 370, ragged in both): y and dy bit for bit
    those of the increments and words that the conv left, through sparse steps and regular passes."""
    import torch
    c, h, w = 97, 352, 370
    assert c * h * w > 12 << 20
    b = wl._NetBuilder("largeout", 9, h, w, 3)
    n = b.conv(-1, c, 3, 1, act=wl.ACT_RELU, out=1)
    net = b.finish()
    rng = np.random.default_rng(5)
    gpu = ev.EvConvNet(net)
    gpu.reset(_dev(rng.standard_normal((9, h, w)).astype(np.float32)))
    if mode == "dense":
        gpu.set_mode(ev.MODE_DENSE_RECOMPUTE)
    for q in (0.002, 0.3):
        d = (rng.standard_normal((9, h, w)) * (rng.random((1, h, w)) < q)).astype(np.float32)
        before = gpu.outputs()[0]["y"].clone()
        gpu.step(_dev(d))
        torch.cuda.synchronize()
        out = gpu.outputs()[0]
        inc = np.ascontiguousarray(gpu.state(n, ev.STATE_DY).transpose(2, 0, 1))
        if mode == "dense":
            np.testing.assert_array_equal(out["y"].cpu().numpy(), inc)
            np.testing.assert_array_equal(out["dy"].cpu().numpy(), inc - before.cpu().numpy())
            continue
        mask = cmp.words_to_mask(gpu.state(n, ev.STATE_OCC), h, w) != 0
        want = np.where(mask, inc, np.float32(0))
        np.testing.assert_array_equal(out["dy"].cpu().numpy(), want)
        np.testing.assert_array_equal(out["y"].cpu().numpy(), before.cpu().numpy() + want)
        assert 0 < mask.sum() < h * w
    gpu.destroy()


@pytest.mark.parametrize("ca,cb,hw", [(5, 64, (17, 20)), (1, 1, (9, 7)), (6, 3, (8, 33)), (4, 7, (25, 12)), (130, 9, (16, 24)), (67, 66, (72, 80)),
                                      (5, 64, (153, 207)), (130, 9, (97, 160)), (1, 6, (547, 551)), (34, 67, (145, 145))])
def test_concat_of_ragged_channel_counts(ca, cb, hw):
    """Concatenations whose operands are not whole vectors of four channels, single floats below 2 Mi values and
    pieces of four from there on (the last four), one to three channels of a site left over, several
    workgroups to a tile where a site has more than 32 pieces: copies of the operands'
    increments where these are active and zeros elsewhere, the OR of their sets, bit for bit."""
    h, w = hw
    _say(f"concat {ca} + {cb} channels on {h} x {w}")
    b = wl._NetBuilder("cat", ca, h, w, ca + cb)
    x = b.conv(-1, cb, 1, 1, 0, act=wl.ACT_RELU)
    y = b.simple(wl.OP_CONCAT, -1, x)
    b.conv(y, 2, 1, 1, 0, act=wl.ACT_NONE, out=1)
    gpu = ev.EvConvNet(b.finish(), flags=ev.FLAG_NO_FUSION)
    rng = np.random.default_rng(ca)
    gpu.reset(_dev(rng.standard_normal((ca, h, w)).astype(np.float32)))
    for q in (0.02, 1.0, 0.3):
        gpu.step(_dev((rng.standard_normal((ca, h, w)) * (rng.random((1, h, w)) < q)).astype(np.float32)))
        sets = [cmp.words_to_mask(gpu.state(n, ev.STATE_OCC), h, w) != 0 for n in (-1, x)]
        want = np.concatenate([np.where(s[..., None], gpu.state(n, ev.STATE_DY), np.float32(0)) for n, s in zip((-1, x), sets)], axis=2)
        both = sets[0] | sets[1]
        np.testing.assert_array_equal(cmp.words_to_mask(gpu.state(y, ev.STATE_OCC), h, w) != 0, both)
        np.testing.assert_array_equal(cmp.words_to_mask(gpu.state(y, ev.STATE_OCC_TOUCHED), h, w) != 0, both)
        np.testing.assert_array_equal(gpu.state(y, ev.STATE_DY)[both], want[both])
    x1 = rng.standard_normal((ca, h, w)).astype(np.float32)
    gpu.reset(_dev(x1))   # a regular pass: the values at every site
    np.testing.assert_array_equal(gpu.state(y, ev.STATE_DY)[..., :ca], x1.transpose(1, 2, 0))
    np.testing.assert_array_equal(gpu.state(y, ev.STATE_DY)[..., ca:], gpu.state(x, ev.STATE_DY))
    gpu.destroy()


@pytest.mark.parametrize("flags", [0, ev.FLAG_NO_FUSION])
@pytest.mark.parametrize("act", [wl.ACT_RELU, wl.ACT_SIGMOID, wl.ACT_TANH, wl.ACT_ONE_MINUS])
@pytest.mark.parametrize("kind,ca,cb", [("concat", 8, 24), ("concat", 5, 7), ("concat", 68, 33), ("concat", 2, 2), ("up", 8, 0), ("up", 36, 0),
                                        ("up", 7, 0), ("up_concat", 8, 16), ("up_concat", 3, 6)])
def test_concatenations_and_up_samplings_with_an_activation(kind, ca, cb, act, flags):
    """CONCAT and UPSAMPLE_BILINEAR2X with an activation, whole vectors of channels and ragged ones: accumulated
    tensor, increments and value-pruned sets are the oracle's, through steps, a regular pass in mid-stream
    and a reset (in exact arithmetic where the activation has it: no flip of a set then)."""
    h, w = 21, 19
    _say(f"{kind} {ca} + {cb} channels, activation {act}, flags {flags}")
    b = wl._NetBuilder("cat_act", ca, h, w, ca + cb)
    if kind == "concat":
        x = b.conv(-1, cb, 1, 1, 0, act=wl.ACT_NONE)
        y = b.simple(wl.OP_CONCAT, -1, x, act=act)
    elif kind == "up":
        y = b.simple(wl.OP_UPSAMPLE2X, -1, act=act)
    else:
        u = b.simple(wl.OP_UPSAMPLE2X, -1)
        v = b.simple(wl.OP_UPSAMPLE2X, -1)
        x = b.conv(v, cb, 1, 1, 0, act=wl.ACT_NONE)
        y = b.simple(wl.OP_CONCAT, u, x, act=act)
    b.simple(wl.OP_ACT, y, act=wl.ACT_NONE, out=1)
    b.conv(y, 2, 1, 1, 0, act=wl.ACT_NONE, out=1)
    net = b.finish()
    exact = act in (wl.ACT_RELU, wl.ACT_ONE_MINUS)
    rng = np.random.default_rng(ca)
    wts = net.weights.copy()
    wts[:] = rng.integers(-2, 3, wts.size) / 4.0
    net.weights = wts
    value = lambda q: (rng.integers(-8, 9, (ca, h, w)) / 4.0 * (rng.random((1, h, w)) < q)).astype(np.float32)
    gpu, ora, rep = ev.EvConvNet(net, flags=flags), Oracle(net), cmp.Report()
    tol = 1e-7 if exact else 1e-5
    for x0 in (value(1.0), value(1.0)):
        gpu.reset(_dev(x0))
        ora.reset(x0)
        cmp.compare_outputs(gpu, ora, rep, tol)
        for q in (0.05, 1.0, 0.3, 0.02):
            d = value(q)
            gpu.step(_dev(d))
            ora.step_increment(d)
            cmp.compare_outputs(gpu, ora, rep, tol)
            for i in range(len(net.nodes)):
                cmp.compare_node(gpu, ora, i, rep, tol=tol)
            assert ora.z(y).size and gpu.state(y, ev.STATE_Z).size == ora.z(y).size
    assert rep.flips <= (0 if exact else 60), rep.flips_by_node
    gpu.destroy()


@pytest.mark.parametrize("h,w,streams", [(20, 28, 1), (9, 4200, 1), (33, 60, 2)])
def test_reset_leaves_every_set_empty(h, w, streams):
    """After a reset in mid-stream every node's S and T words, count and bitmap are zero (a row of more than 512
    tiles, two streams), and the next step starts from there."""
    _say(f"reset empties the sets: {h} x {w}, {streams} streams")
    b = wl._NetBuilder("empty", 3, h, w, 5)
    x = b.conv(-1, 16, 3, act=wl.ACT_RELU)
    y = b.conv(x, 32, 3, act=wl.ACT_NONE)
    z = b.simple(wl.OP_ADD, y, y, act=wl.ACT_RELU)
    b.conv(z, 5, 1, 1, 0, act=wl.ACT_RELU, out=1)
    net = b.finish()
    rng = np.random.default_rng(w)
    gpu, fresh = ev.EvConvNet(net, n_streams=streams), ev.EvConvNet(net, n_streams=streams)
    dev = lambda a: _dev(a if streams > 1 else a[0])
    x0, x1, x2 = rng.standard_normal((3, streams, 3, h, w)).astype(np.float32)
    gpu.reset(dev(x0))
    gpu.step_frame(dev(x1))
    assert gpu.state(z, ev.STATE_OCC).any()
    gpu.reset(dev(x2))
    fresh.reset(dev(x2))
    for s in range(streams):
        for n in range(-1, len(net.nodes)):
            for kind in (ev.STATE_OCC, ev.STATE_COUNT, ev.STATE_BITMAP) + ((ev.STATE_OCC_TOUCHED,) if n >= 0 else ()):
                assert not gpu.state(n, kind, s).any(), (n, kind, s)
    for g in (gpu, fresh):
        g.step_frame(dev(x1))
    for s in range(streams):
        np.testing.assert_array_equal(gpu.state(z, ev.STATE_Z, s), fresh.state(z, ev.STATE_Z, s))
        np.testing.assert_array_equal(gpu.site_list(z, s), fresh.site_list(z, s))
    gpu.destroy()
    fresh.destroy()


def test_outputs_keep_the_workspace():
    """Outputs that outlive their net: its workspace is not given to the next allocation under them."""
    import gc
    import torch
    net = wl.net_single_conv(3, 16, 40, 48)
    rng = np.random.default_rng(3)
    gpu = ev.EvConvNet(net)
    gpu.reset(_dev(rng.standard_normal((16, 40, 48)).astype(np.float32)))
    out, size = gpu.outputs()[0], gpu.workspace.numel()
    want = out["y"].clone()
    del gpu
    gc.collect()
    for _ in range(4):
        torch.full((size,), 255, dtype=torch.uint8, device="cuda")
    assert torch.equal(out["y"], want)


def test_reset_clears_arrival_counters():
    """Counters that a pass cut short leaves behind (here: written by hand, those of the channel split behind the
    last node's occupancy words, the increment builder's scratch words behind the last output) are cleared by a
    reset, those of the channel split by every pass: the results are those of a fresh net."""
    import torch
    c, h, w = 256, 11, 20
    b = wl._NetBuilder("counters", c, h, w, 3)
    n = b.conv(-1, 32, 3, 1, act=wl.ACT_RELU, out=1)
    net = b.finish()
    rng = np.random.default_rng(5)
    x0 = rng.standard_normal((c, h, w)).astype(np.float32)
    incs = [(rng.standard_normal(x0.shape) * (rng.random((1, h, w)) < q)).astype(np.float32) for q in (0.2, 0.1, 0.3)]
    tiles = -(-h // 8) * -(-w // 8)
    gpu, clean = ev.EvConvNet(net), ev.EvConvNet(net)
    for g in (gpu, clean):
        g.reset(_dev(x0))
        g.step(_dev(incs[0]))
    torch.cuda.synchronize()
    words = gpu.state(n, ev.STATE_OCC).tobytes() + gpu.state(n, ev.STATE_OCC_TOUCHED).tobytes()
    counters = gpu.workspace.cpu().numpy().tobytes().index(words) + len(words)
    align = lambda p: (p + 255) // 256 * 256
    dy = gpu.outputs()[0]["dy"]
    at = align(dy.data_ptr() + dy.numel() * 4) - gpu.workspace.data_ptr()
    groups = -(-h // 8) * 8 // 2   # of two rows (17 to 32 columns), rows below the image among them: two words each
    split = gpu.workspace[counters:counters + 8 * tiles].view(torch.int32)      # one per half tile and block of 32 channels
    builder = gpu.workspace[at:at + 16 * groups].view(torch.int64)
    assert not int(split.abs().sum()) and not int(builder.abs().sum())
    split.fill_(1)
    builder.fill_(-1)              # every site and every arrival bit
    for g in (gpu, clean):
        g.reset(_dev(x0))
    torch.cuda.synchronize()
    assert not int(builder.abs().sum())
    np.testing.assert_array_equal(gpu.state(n, ev.STATE_Z), clean.state(n, ev.STATE_Z))
    for k, d in enumerate(incs):
        split.fill_(1 + k)
        for g in (gpu, clean):
            g.step(_dev(d))
        torch.cuda.synchronize()
        for kind in (ev.STATE_Z, ev.STATE_OCC, ev.STATE_OCC_TOUCHED):
            np.testing.assert_array_equal(gpu.state(n, kind), clean.state(n, kind))
        np.testing.assert_array_equal(gpu.state(-1, ev.STATE_OCC), clean.state(-1, ev.STATE_OCC))
        assert torch.equal(gpu.outputs()[0]["y"], clean.outputs()[0]["y"])
        assert not int(builder.abs().sum())
    gpu.destroy()
    clean.destroy()


def test_channel_split_with_sparsification_layers_exact_arithmetic():
    """Convs whose channels are split over workgroups, with sparsification layers and an ADD folded into
    their epilogues: exact arithmetic (dyadic weights and inputs, k = 0.5), so the GPU equals the fp64
    oracle on every tensor and every list."""
    _say("channel split with folded sparsification layers, exact arithmetic")
    b = wl._NetBuilder("sp_ks", 128, 13, 19, 5, sparsify=True, sparsify_k=0.5)
    c1 = b.conv(-1, 128, 3)                      # 2 x 3 tiles x 4 blocks: 48 half-tile workgroups
    c2 = b.conv(c1, 128, 5)
    c3 = b.conv(c2, 128, 3, act=wl.ACT_NONE)
    a = b.simple(wl.OP_ADD, c1, c3, act=wl.ACT_RELU)
    b.conv(a, 32, 3, out=1)
    net = b.finish()
    rng = np.random.default_rng(8)
    wts = net.weights.copy()
    for nd in net.nodes:
        if nd.op == wl.OP_CONV2D:
            n = nd.c_out * nd.c_in * nd.k * nd.k
            wts[nd.w_off:nd.w_off + n] = rng.integers(-1, 2, n) * (rng.random(n) < 0.03) / 8.0
    net.weights = wts
    x0 = (rng.integers(-8, 9, (128, 13, 19)) / 4.0).astype(np.float32)
    incs = [((rng.integers(-4, 5, x0.shape) / 4.0) * (rng.random((1, 13, 19)) < q)).astype(np.float32) for q in (0.05, 0.05, 1.0, 0.1)]
    gpu, ora, rep = ev.EvConvNet(net), Oracle(net), cmp.Report()
    names = [gpu.kernel_name(i) for i in range(len(net.nodes))]
    assert [names[i] for i, nd in enumerate(net.nodes) if nd.op == wl.OP_SPARSIFY] == ["fused_into_conv_epilogue"] * 3, names
    gpu.reset(_dev(x0))
    ora.reset(x0)
    for d in incs:
        gpu.step(_dev(d))
        ora.step_increment(d)
        cmp.compare_outputs(gpu, ora, rep, 1e-7)
        for i in range(len(net.nodes)):
            cmp.compare_node(gpu, ora, i, rep, tol=1e-7, exact_sets=True)
    assert rep.flips == 0
    gpu.destroy()


@pytest.mark.parametrize("act", [wl.ACT_SIGMOID, wl.ACT_TANH, wl.ACT_ONE_MINUS])
def test_channel_split_with_other_activations(act):
    """The general epilogue (activations other than ReLU) behind a channel split, with a folded ADD."""
    b = wl._NetBuilder("ks_act", 192, 9, 20, 5, bias=True)
    a = b.conv(-1, 40, 1, act=wl.ACT_NONE)
    c = b.conv(-1, 40, 3, act=act)
    b.simple(wl.OP_ADD, c, a, act=wl.ACT_TANH, out=1)
    net = b.finish()
    rng = np.random.default_rng(act)
    x0 = (rng.standard_normal((192, 9, 20)) * 0.5).astype(np.float32)
    incs = [(rng.standard_normal(x0.shape) * 0.3 * (rng.random((1, 9, 20)) < q)).astype(np.float32) for q in (0.05, 1.0, 0.1)]
    run_stream(net, x0, incs, "increment", label=f"channel split, activation {act}", max_flips=4, tol=1e-5)


@pytest.mark.parametrize("where", ["split", "gather"])
def test_infinities_through_the_channel_split_and_the_up_sampling_gather(where):
    """Infinite and NaN increments through a conv whose channels are split over workgroups, and through
    the interpolating gather of a conv behind an up-sampling: infinities and NaN where the oracle's
    IEEE products put them, every other site as without them."""
    _say(f"infinities: {where}")
    if where == "split":
        ci, h, w, flags = 256, 12, 21, 0
        b = wl._NetBuilder("inf_ks", ci, h, w, 5)
        c = b.conv(-1, 32, 3, act=wl.ACT_NONE, out=1)
    else:
        ci, h, w, flags = 32, 12, 21, ev.FLAG_NO_FOLD
        b = wl._NetBuilder("inf_ups", ci, h, w, 5)
        c = b.conv(b.simple(wl.OP_UPSAMPLE2X, -1), 32, 5, act=wl.ACT_NONE, out=1)
    net = b.finish()
    net.weights[::7] = 0.0
    gpu, ora = ev.EvConvNet(net, flags=flags), Oracle(net)
    rng = np.random.default_rng(2)
    x0 = np.zeros((ci, h, w), np.float32)
    d = (rng.standard_normal(x0.shape) * (rng.random((1, h, w)) < 0.2)).astype(np.float32)
    d[ci - 1, 2, 3], d[1, 9, 4], d[ci // 2, 6, 17] = np.inf, np.nan, -np.inf
    gpu.reset(_dev(x0))
    ora.reset(x0)
    gpu.step(_dev(d))
    ora.step_increment(d)
    z, zr = gpu.state(c, ev.STATE_Z).astype(np.float64), ora.z(c)
    np.testing.assert_array_equal(np.isnan(z), np.isnan(zr))
    np.testing.assert_array_equal(z[np.isinf(zr)], zr[np.isinf(zr)])
    fin = np.isfinite(zr)
    assert fin.any() and (~fin).any()
    assert np.isfinite(z[fin]).all() and np.abs(z[fin] - zr[fin]).max() <= 2e-6 * np.abs(zr[fin]).max()
    gpu.destroy()
