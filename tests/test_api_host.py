"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, sizes workspaces, and rejects bad descriptions before any GPU work."""
import ctypes
import dataclasses
import os
import re

import numpy as np
import pytest

from paper_2303_04670_amd import evconv as ev
from paper_2303_04670_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    text = open(os.path.join(ROOT, "include", "evconv.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(evconv_[a-z_]+)\s*\(", text))
    assert declared == set(ev.EXPORTS)
    L = ev.lib()
    for name in sorted(declared):
        assert hasattr(L, name), name


@pytest.mark.parametrize("make", [wl.net_single_conv, wl.net_conv_stack, wl.net_unet_depth, wl.net_resnet18,
                                  wl.net_flow, wl.net_convlstm], ids=lambda f: f.__name__)
def test_query_workspace_all_workloads(make):
    net = make()
    desc, keep = ev.marshal_desc(net)
    n = ev.evconv_query_workspace(desc)
    shapes = net.node_shapes()
    lower = sum(c * h * w * 4 for c, h, w in shapes)   # at least one increment buffer per node
    assert lower < n < 40 * lower + (64 << 20)


def _status(desc):
    n = ctypes.c_size_t(0)
    return ev.lib().evconv_query_workspace(ctypes.byref(desc), ctypes.byref(n))


def test_bad_descriptions_are_rejected():
    net = wl.net_conv_stack(1, h=16, w=16)
    desc, nodes = ev.marshal_desc(net)
    assert _status(desc) == ev.OK
    desc.abi_version = 99
    assert _status(desc) == ev.ERR_BAD_DESC
    desc.abi_version = ev.ABI_VERSION
    nodes[1].in0 = 3                       # forward reference
    assert _status(desc) == ev.ERR_BAD_DESC
    nodes[1].in0 = 0
    nodes[1].c_in = 7                      # channel mismatch
    assert _status(desc) == ev.ERR_SHAPE
    nodes[1].c_in = 32
    nodes[2].kh = 9
    assert _status(desc) == ev.ERR_UNSUPPORTED
    nodes[2].kh = 3
    nodes[0].op = 42
    assert _status(desc) == ev.ERR_INVALID_ARG
    nodes[0].op = wl.OP_CONV2D
    nodes[0].act = 5                       # one past the last activation
    assert _status(desc) == ev.ERR_INVALID_ARG
    nodes[0].act = wl.ACT_TANH
    assert _status(desc) == ev.OK
    nodes[0].act = wl.ACT_RELU
    nodes[3].op, nodes[3].in1 = wl.OP_MUL, 1       # 64 x 4 x 4 times 32 x 8 x 8
    assert _status(desc) == ev.ERR_SHAPE
    nodes[3].op, nodes[3].in1 = wl.OP_CONV2D, -2
    desc.sparsify_tp = -0.1
    assert _status(desc) == ev.ERR_INVALID_ARG
    desc.sparsify_tp = 0.0
    desc.flags = 8                         # not a planner switch
    assert _status(desc) == ev.ERR_INVALID_ARG
    desc.flags = ev.FLAG_NO_FUSION | ev.FLAG_NO_FOLD | ev.FLAG_FORCE_VALU
    assert _status(desc) == ev.OK
    desc.abi_version = 1                   # a description laid out for the previous ABI is refused
    assert _status(desc) == ev.ERR_BAD_DESC
    desc.abi_version = ev.ABI_VERSION
    assert ev.lib().evconv_query_workspace(None, None) == ev.ERR_INVALID_ARG
    assert b"" != ev.lib().evconv_last_error(None)


def test_recurrent_descriptions():
    """DELAY: in0 must name a later node of the same shape, in1 an earlier node of its size."""
    net = wl.net_convlstm(h=16, w=16, hidden=8)
    desc, nodes = ev.marshal_desc(net)
    assert _status(desc) == ev.OK
    src = nodes[0].in0
    nodes[0].in0 = 0                       # itself
    assert _status(desc) == ev.ERR_BAD_DESC
    nodes[0].in0 = len(net.nodes)          # past the end
    assert _status(desc) == ev.ERR_BAD_DESC
    nodes[0].in0 = len(net.nodes) - 1      # the 2-channel head: shape differs
    assert _status(desc) == ev.ERR_SHAPE
    nodes[0].in0 = src
    nodes[0].act = wl.ACT_RELU
    assert _status(desc) == ev.ERR_UNSUPPORTED
    nodes[0].act = wl.ACT_NONE
    nodes[1].in1 = 5                       # the size reference must be an earlier node
    assert _status(desc) == ev.ERR_BAD_DESC
    nodes[1].in1 = -1
    assert _status(desc) == ev.OK


def test_null_handles():
    L = ev.lib()
    assert L.evconv_destroy(None) == ev.OK
    assert L.evconv_num_outputs(None) == 0
    assert L.evconv_reset(None, None, None) == ev.ERR_INVALID_ARG
    assert L.evconv_step(None, None, None) == ev.ERR_INVALID_ARG
    assert L.evconv_set_mode(None, 0) == ev.ERR_INVALID_ARG
    assert L.evconv_current_mode(None) == -1


class _HostTorch:
    """What EvConvNet.outputs needs of torch, on the CPU: every tensor is one that `make` returns."""

    def __init__(self, make):
        self.as_tensor = lambda span, device: make(span)

    @staticmethod
    def is_inference_mode_enabled():
        return False


def _net_without_a_gpu(make):
    net = object.__new__(ev.EvConvNet)
    net.torch, net.device, net._outs, net._out_spans, net.stream_stride, net._h = _HostTorch(make), "cuda:0", (ev.Out * 1)(), {}, 4096, None
    return net


@pytest.mark.parametrize("stream", [0, 3])
def test_outputs_before_the_first_reset_are_refused(stream):
    """The output pointers are null until then: no tensor may be made of them."""
    made = []
    net = _net_without_a_gpu(made.append)
    with pytest.raises(ev.EvConvError) as e:
        net.outputs(stream)
    assert e.value.status == ev.ERR_STATE and not made


class _HostTensor:
    def __init__(self, ptr, value):
        self.ptr, self.data = ptr, value

    def data_ptr(self):
        return self.ptr


@pytest.mark.parametrize("copies", [False, True])
def test_outputs_keeps_tensors_over_the_net_s_memory_only(copies):
    """Where torch makes a copy of the outputs (a net on another device than the current one) every call
    makes a new one; tensors over the memory itself are made once."""
    made = []

    def make(span):
        a = span.__cuda_array_interface__
        made.append((a["data"][0], a["typestr"], a["shape"]))
        return _HostTensor(a["data"][0] + (64 if copies else 0), len(made))
    net = _net_without_a_gpu(make)
    o = net._outs[0]
    o.node, o.c, o.h, o.w, o.y, o.dy, o.dy_idx, o.dy_count = 2, 3, 5, 7, 1 << 20, 1 << 21, 1 << 22, 1 << 23
    first, again, other = net.outputs(1), net.outputs(1), net.outputs(0)
    assert made[:4] == [((1 << 20) + 4096, "<f4", (3, 5, 7)), ((1 << 21) + 4096, "<f4", (3, 5, 7)),
                        ((1 << 22) + 4096, "<i4", (35,)), ((1 << 23) + 4096, "<i4", (1,))]
    assert first[0] == dict(node=2, y=1, dy=2, idx=3, count=4)
    assert (again == first) == (not copies) and other != first and len(made) == (12 if copies else 8)


def test_measurement_aids_reject_bad_arguments_before_any_gpu_work():
    L = ev.lib()
    out = (ctypes.c_float * ev.CHIP_PROBE_VALUES)()
    INVALID, UNSUPPORTED = ev.STATUS_NAMES.index("ERR_INVALID_ARG"), ev.STATUS_NAMES.index("ERR_UNSUPPORTED")
    assert L.evconv_debug_chip_probes(None, ev.CHIP_PROBE_SCRATCH_BYTES, None, out, ev.CHIP_PROBE_VALUES) == INVALID
    dummy = ctypes.c_void_p(4096)  # (never dereferenced: the size check comes first)
    assert L.evconv_debug_chip_probes(dummy, ev.CHIP_PROBE_SCRATCH_BYTES - 1, None, out, ev.CHIP_PROBE_VALUES) == INVALID
    assert L.evconv_debug_chip_probes(dummy, ev.CHIP_PROBE_SCRATCH_BYTES, None, out, ev.CHIP_PROBE_VALUES - 1) == INVALID
    # phase stamps exist only in the measurement build; the product library says so
    n = ctypes.c_int32(-5)
    for mode in (0, 1, 2):
        assert L.evconv_debug_phase_stamps(mode, None, 0, 0, ctypes.byref(n)) == UNSUPPORTED
    assert L.evconv_debug_phase_stamps(3, None, 0, 0, ctypes.byref(n)) == INVALID
    assert L.evconv_debug_phase_stamps(0, None, 0, 0, None) == INVALID
    assert L.evconv_debug_phase_stamps(0, None, 8, 0, ctypes.byref(n)) == INVALID
    assert n.value == -5


def test_product_package_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2303_04670_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith(".py"):
                src = open(os.path.join(dirpath, f)).read()
                assert not re.search(r"^\s*(from|import)\s+oracle", src, flags=re.M), f
                assert "libevconv_oracle" not in src, f


def test_static_workspace_holds_what_four_bytes_per_weight_and_32_mib_held():
    """fp32 matrix-core weights take six bytes in the workspace; the static array is large enough for every
    description that fits 32 MiB with four (which split-mode weights take), also when it is almost
    all weights and its convs need scratch for the channel split."""
    conv = lambda i, co: wl.Node(wl.OP_CONV2D, wl.ACT_RELU, i - 1, -2, 512, co, 3, 1, 1, 0, -1, int(i == 3))
    nodes = [conv(0, 512), conv(1, 512), conv(2, 512), conv(3, 256)]
    split = [dataclasses.replace(nd, wdtype=wl.WD_F32_SPLIT) for nd in nodes]
    net = lambda nds: wl.Net("weights", 512, 3, 3, nds, np.zeros(0, np.float32))
    query = lambda nds: ev.evconv_query_workspace(ev.marshal_desc(net(nds))[0])
    scratch = 32 * 8 * 32 * 32 * 4   # 32 half-tile workgroups x 8 shares of 32 x 32 sums
    assert (31 << 20) < query(split) - scratch < (32 << 20)
    assert query(nodes) <= ev.STATIC_WORKSPACE_BYTES


def _decoder(h, w, wdtype, up_act=wl.ACT_NONE, up_out=0, reader=False):
    nodes = [wl.Node(wl.OP_UPSAMPLE2X, up_act, -1, -2, 64, 64, is_output=up_out),
             wl.Node(wl.OP_CONV2D, wl.ACT_RELU, 0, -2, 64, 32, 5, 1, 2, 0, -1, 1, wdtype=wdtype)]
    if reader:
        nodes.append(wl.Node(wl.OP_ACT, wl.ACT_TANH, 0, -2, 64, 64, is_output=1))
    return wl.Net("decoder", 64, h, w, nodes, np.zeros(0, np.float32))


def test_folded_weights_take_room_only_where_they_are_used():
    """A conv whose up-sampling is folded into its weights: four phases of 6 x 6 taps, two bytes a part.  No room for
    them with bf16-declared weights, on small maps, under the flags that forbid it, or where the
    up-sampled tensor is needed itself."""
    query = lambda *a, flags=0, **k: ev.evconv_query_workspace(ev.marshal_desc(_decoder(*a, **k), flags=flags)[0])
    extra = lambda *a, flags=0, **k: query(*a, flags=flags, **k) - query(*a, flags=flags | ev.FLAG_NO_FOLD, **k)
    sets = 4 * 36 * 64 * 32 * 2
    for wdtype, parts in ((wl.WD_F32, 3), (wl.WD_F32_SPLIT, 2)):
        assert sets * parts <= extra(40, 56, wdtype) <= sets * parts + 1024
    assert extra(40, 56, wl.WD_BF16) == 0
    assert extra(17, 56, wl.WD_F32) == 0
    assert extra(40, 56, wl.WD_F32, flags=ev.FLAG_NO_FUSION) == 0 and extra(40, 56, wl.WD_F32, flags=ev.FLAG_FORCE_VALU) == 0
    assert extra(40, 56, wl.WD_F32, up_act=wl.ACT_RELU) == 0 and extra(40, 56, wl.WD_F32, up_out=1) == 0
    assert extra(40, 56, wl.WD_F32, reader=True) == 0


def test_streams_share_their_weights():
    """Every further stream of a net takes the same room, and none for the weights (8 conv layers of 128 channels on
    a map of 4 x 4: nearly all weights)."""
    nodes = [wl.Node(wl.OP_CONV2D, wl.ACT_RELU, i - 1, -2, 128, 128, 3, 1, 1, 0, -1, int(i == 7)) for i in range(8)]
    net = wl.Net("weights", 128, 4, 4, nodes, np.zeros(0, np.float32))
    query = lambda n: ev.evconv_query_workspace(ev.marshal_desc(net, n_streams=n)[0])
    weights = 8 * 9 * 128 * 128 * 6
    assert query(1) >= weights
    assert query(3) - query(2) == query(2) - query(1) < weights // 4


def test_no_kernel_uses_scratch_memory():
    """Registers spilled to scratch would make the runtime allocate device memory at a kernel's first
    launch, which the library promises not to: the metadata of every kernel in the built library
    states a private segment of 0 bytes (a small msgpack integer behind its key)."""
    blob = open(ev.LIB_PATH, "rb").read()
    sizes = [blob[m.end()] for m in re.finditer(rb"\.private_segment_fixed_size", blob)]
    assert len(sizes) > 50 and set(sizes) == {0}, sizes
