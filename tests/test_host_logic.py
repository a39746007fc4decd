"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every
declared symbol, plans networks, reports shapes / parameter layout and rejects
bad arguments with error codes."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_1312_6186_amd import binding as B
from paper_1312_6186_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "asgd.h")).read()
    declared = set(re.findall(r"\b(asgd_[a-z_]+)\s*\(", header))
    declared -= {"asgd_net"}
    assert declared == set(B.EXPORTS)
    L = B.lib()
    for name in declared:
        assert getattr(L, name) is not None


@pytest.mark.parametrize("cfg", [wl.TINY, wl.SMALL, wl.ALEXNET])
def test_plan_matches_the_workload_description(cfg):
    for dt in (B.F32, B.BF16):
        net = B.asgd_net_create(cfg["layers"], cfg["batch"], cfg["in_shape"], dt)
        try:
            assert B.asgd_param_count(net) == wl.param_count(cfg["layers"], cfg["in_shape"])
            layout = B.asgd_param_layout(net)
            ref = wl.param_shapes(cfg["layers"], cfg["in_shape"])
            assert len(layout) == len(ref)
            off = 0
            for t, (li, wshape, blen, _) in zip(layout, ref):
                assert t["layer"] == li and t["w_offset"] == off and t["w_count"] == int(np.prod(wshape))
                assert t["w_shape"][:len(wshape)] == tuple(wshape)
                off += t["w_count"]
                assert t["b_offset"] == off and t["b_count"] == blen
                off += blen
            assert B.asgd_workspace_bytes(net) > 0
        finally:
            B.asgd_net_destroy(net)


def test_full_cited_architecture_has_the_published_parameter_count():
    cfg = wl.ALEXNET_FULL
    net = B.asgd_net_create(cfg["layers"], 2, cfg["in_shape"], B.BF16)
    try:
        assert B.asgd_param_count(net) == 60965224 == wl.param_count(cfg["layers"], cfg["in_shape"])
        lay = {t["layer"]: t for t in B.asgd_param_layout(net)}
        assert lay[4]["w_shape"] == (256, 48, 5, 5) and lay[10]["w_shape"] == (384, 192, 3, 3) and lay[12]["w_shape"] == (256, 192, 3, 3)
    finally:
        B.asgd_net_destroy(net)


def test_alexnet_shapes():
    net = B.asgd_net_create(wl.ALEXNET["layers"], 128, (3, 224, 224), B.BF16)
    shapes = [B.asgd_layer_shape(net, i) for i in range(len(wl.ALEXNET["layers"]))]
    assert shapes[0] == (96, 55, 55) and shapes[2] == (96, 27, 27) and shapes[5] == (256, 13, 13)
    assert shapes[12] == (256, 6, 6) and shapes[13] == (4096, 1, 1) and shapes[-1] == (1000, 1, 1)
    B.asgd_net_destroy(net)


def _rc(layers, batch=4, in_shape=(3, 16, 16), dt=B.F32):
    arr = B.layer_descs(layers)
    h = ctypes.c_void_p(0)
    rc = B.lib().asgd_net_create(arr, len(arr), batch, in_shape[0], in_shape[1], in_shape[2], dt, ctypes.byref(h))
    if rc == 0:
        B.asgd_net_destroy(h)
    return rc


def test_bad_descriptors_are_rejected_with_codes():
    ok = [("conv", 8, 3, 1, 1), ("relu",), ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)]
    assert _rc(ok) == B.OK
    assert _rc(ok[:-1]) == B.ESHAPE                                   # no loss layer
    assert _rc([("relu",)] + ok) == B.ESHAPE                          # ReLU with nothing to fuse into
    assert _rc([("conv", 8, 32, 1, 0), ("fc", 10), ("softmax_ce",)]) == B.ESHAPE  # filter larger than image
    assert _rc([("conv", 8, 3, 1, 1), ("maxpool", 20, 2), ("fc", 10), ("softmax_ce",)]) == B.ESHAPE
    assert _rc([("conv", 3, 3, 1, 0), ("fc", 10), ("softmax_ce",)], in_shape=(3, 5, 5)) == B.ESHAPE  # fan-in 27
    assert _rc([("fc", 16), ("dropout", 0.5), ("fc", 10), ("softmax_ce",)]) == B.ESHAPE       # dropout needs FC+ReLU
    assert _rc([("fc", 16), ("relu",), ("dropout", 1.0), ("fc", 10), ("softmax_ce",)]) == B.ESHAPE
    lrn = [("conv", 8, 3, 1, 1), ("relu",), ("lrn", 5, 1e-4, 0.75, 2.0), ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)]
    assert _rc(lrn) == B.OK
    assert _rc([lrn[0]] + lrn[2:]) == B.ESHAPE                        # LRN needs CONV + RELU right before it
    assert _rc(lrn[:2] + [lrn[3], lrn[2]] + lrn[4:]) == B.ESHAPE      # not after a pool
    assert _rc(lrn[:2] + [("lrn", 4, 1e-4, 0.75, 2.0)] + lrn[3:]) == B.ESHAPE    # even window
    assert _rc(lrn[:2] + [("lrn", 11, 1e-4, 0.75, 2.0)] + lrn[3:]) == B.ESHAPE   # window above 9
    assert _rc(lrn[:2] + [("lrn", 5, 1e-4, 0.75, 0.0)] + lrn[3:]) == B.ESHAPE    # bias must be positive
    grp = [("conv", 16, 3, 1, 1), ("relu",), ("conv", 32, 3, 1, 1, 2), ("relu",), ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)]
    assert _rc(grp) == B.OK
    assert _rc(grp[:2] + [("conv", 32, 3, 1, 1, 4)] + grp[3:]) == B.ESHAPE      # 4 input channels per group: not a multiple of 8
    assert _rc(grp[:2] + [("conv", 24, 3, 1, 1, 2)] + grp[3:]) == B.ESHAPE      # 12 output channels per group
    assert _rc(grp[:2] + [("conv", 32, 3, 1, 1, 3)] + grp[3:]) == B.ESHAPE      # 16 does not divide by 3
    assert _rc(ok, batch=0) == B.ESHAPE
    assert _rc(ok, dt=7) == B.EINVAL
    assert "dtype" in B.asgd_last_error()
    h = ctypes.c_void_p(0)
    assert B.lib().asgd_net_create(None, 3, 1, 1, 1, 1, 0, ctypes.byref(h)) == B.EINVAL
    bad = (B.LayerDesc * 1)(B.LayerDesc(99, 0, 0, 0, 0, 0.0, 0.0))
    assert B.lib().asgd_net_create(bad, 1, 1, 1, 8, 8, 0, ctypes.byref(h)) == B.EINVAL


def test_null_and_misaligned_pointers_are_rejected_before_any_gpu_work():
    L = B.lib()
    net = B.asgd_net_create(wl.TINY["layers"], 8, (1, 28, 28), B.F32)
    vp = ctypes.c_void_p
    assert L.asgd_fwd_bwd(net, vp(0), vp(16), vp(16), 0, 0, 0, vp(16), vp(16), vp(0)) == B.EINVAL
    assert L.asgd_fwd_bwd(net, vp(4), vp(16), vp(16), 0, 0, 0, vp(16), vp(16), vp(0)) == B.EALIGN
    assert L.asgd_apply_update(vp(0), vp(16), vp(16), 10, 0.1, 0.9, 0.0, vp(0)) == B.EINVAL
    assert L.asgd_apply_update(vp(0), vp(0), vp(0), 0, 0.1, 0.9, 0.0, vp(0)) == B.OK          # nothing to do
    assert L.asgd_apply_update(vp(2), vp(16), vp(16), 10, 0.1, 0.9, 0.0, vp(0)) == B.EALIGN
    assert L.asgd_snapshot(vp(16), vp(16), 10, 5, vp(0)) == B.EINVAL
    assert L.asgd_snapshot(vp(0), vp(16), 10, B.BF16, vp(0)) == B.EINVAL
    assert L.asgd_debug_get(net, 0, 1, vp(16), 1 << 20, vp(0)) == B.EINVAL                     # nothing has run yet
    assert L.asgd_layer_shape(net, 99, (ctypes.c_int32 * 3)()) == B.EINVAL
    assert B.asgd_param_count(vp(0)) == 0
    B.asgd_net_destroy(net)
    assert L.asgd_net_destroy(vp(0)) == B.OK


def test_schedule_generator_agrees_with_definition_and_rejects_bad_arguments():
    MASK = (1 << 64) - 1

    def mix(z):
        z ^= z >> 30; z = (z * 0xBF58476D1CE4E5B9) & MASK
        z ^= z >> 27; z = (z * 0x94D049BB133111EB) & MASK
        return z ^ (z >> 31)

    worker, rv = B.asgd_schedule_generate(64, 4005, 4, 3)
    for a in range(64):
        assert worker[a] == a % 4 and rv[a] == a - min(a, (mix((mix(4005) + a) & MASK) >> 32) % 4)
    i32p = ctypes.POINTER(ctypes.c_int32)
    w = np.zeros(4, np.int32)
    assert B.lib().asgd_schedule_generate(w.ctypes.data_as(i32p), w.ctypes.data_as(i32p), 4, 1, 4, 4) == B.EINVAL
    assert B.lib().asgd_schedule_generate(None, None, 4, 1, 4, 3) == B.EINVAL


def test_replay_rejects_impossible_schedules_without_a_gpu():
    L = B.lib()
    vp = ctypes.c_void_p
    nets = [B.asgd_net_create(wl.TINY["layers"], 8, (1, 28, 28), B.F32) for _ in range(2)]
    net_arr = (vp * 2)(*[n.value for n in nets])
    bufs = (vp * 2)(16, 32)
    i32p = ctypes.POINTER(ctypes.c_int32)

    def run(worker, rv):
        w = np.array(worker, np.int32); r = np.array(rv, np.int32)
        return L.asgd_replay_run(net_arr, 2, vp(16), vp(16), bufs, bufs, vp(16), vp(16), w.ctypes.data_as(i32p),
                                 r.ctypes.data_as(i32p), len(worker), 0.1, 0.9, 0.0, 0, vp(16), vp(16), vp(0))

    assert run([0, 1, 0], [0, 0, 3]) == B.EINVAL      # reads a version that does not exist yet
    assert run([0, 1, 0], [0, 0, 0]) == B.EINVAL      # worker 0 reads before its own push 0 was applied
    assert run([0, 5], [0, 0]) == B.EINVAL            # no such worker
    for n in nets:
        B.asgd_net_destroy(n)


# ---- planning of the stride-1 convolution kernel (internal functions, by their mangled names)
class _Gather(ctypes.Structure):
    _fields_ = ([("x", ctypes.c_void_p)] + [(n, ctypes.c_int) for n in ("N", "H", "W", "C", "Ho", "Wo", "kh", "kw", "sm", "ds", "pad")]
                + [(n, ctypes.c_size_t) for n in ("bytes", "rowb", "pix")])


class _DirectPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("ks", "nchunks", "tile", "npl")] + [(n, ctypes.c_size_t) for n in ("nblk_elems", "pack_elems")]


def _plan_direct(dtype, batch, h, w, cin, cout, k, groups=1):
    """cin and cout of one group, as the gather of a layer's first group describes it"""
    es = 2 if dtype == B.BF16 else 4
    f = B.lib()["_ZN4asgd11plan_directEiRKNS_6GatherEii"]
    f.argtypes, f.restype = [ctypes.c_int, ctypes.POINTER(_Gather), ctypes.c_int, ctypes.c_int], _DirectPlan
    pix = cin * groups * es if groups > 1 else 0
    return f(dtype, ctypes.byref(_Gather(None, batch, h, w, cin, h, w, k, k, 1, 1, k // 2, batch * h * w * cin * groups * es, w * pix, pix)), cout, groups)


def _pieces_stored(ks, npos):
    """The loads of the next chunk's patch that are in LDS at the barrier that ends a chunk, in the order in which
    conv_direct_kernel loads and stores them: load j is issued in the first K step of window position j."""
    stored, on_its_way = set(), None
    for pos in range(npos):
        for step in range(ks):
            if pos == npos - 1 and step == ks - 1:
                return stored | {on_its_way}          # the last K step stores what has been loaded, then the barrier
            if step == 0:
                stored, on_its_way = stored | {on_its_way}, pos


@pytest.mark.parametrize("groups", [1, 2, 4])
@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_stride1_convolution_plans_copy_every_piece_of_a_patch(dtype, groups):
    wide = chunked = 0
    for k in (3, 5):
        for cin in list(range(8, 200, 8)) + [256, 384, 400, 512]:
            for cout in (8, 48, 64, 96, 128, 256):
                for w in list(range(5, 64, 9)) + list(range(64, 560, 5)) + [111, 112, 191, 192, 223, 224, 225, 240, 255, 256, 447, 448, 479, 480, 511, 512]:
                    for h, batch in ((3, 1), (w, 4)):
                        p = _plan_direct(dtype, batch, h, w, cin, cout, k, groups)
                        if p.ks == 0:
                            continue
                        assert p.nchunks == -(-cin // (16 * p.ks)) and p.npl > 0
                        # a group's filters whole, and those of all groups within what an operand may hold
                        assert p.pack_elems == -(-cout // 32) * p.nblk_elems and p.nblk_elems == p.nchunks * k * k * p.ks * 512
                        assert p.pack_elems * groups * (2 if dtype == B.BF16 else 4) <= 1 << 30
                        if p.nchunks > 1:
                            chunked += 1
                            missing = set(range(p.npl)) - _pieces_stored(p.ks, k * k)
                            assert not missing, (dtype, k, cin, cout, h, w, p.ks, p.npl, missing)
                            wide += p.npl >= k * k - 1
    assert chunked > 1000 and wide > 10   # the sweep reaches plans at the limit


# Layers (channels in, out, window, height, width, images) with the us of the general engine and of the stride-1 kernel in its best
# tile shape: those that the engine runs faster belong to it, the others do not
ENGINE_FASTER = [(B.F32, (48, 32, 3, 128, 192, 5), 69, 165), (B.F32, (80, 24, 3, 16, 192, 8), 32, 64), (B.F32, (192, 32, 3, 64, 80, 66), 647, 1070),
                 (B.F32, (48, 384, 5, 32, 128, 19), 622, 652), (B.BF16, (96, 16, 3, 32, 255, 26), 47, 110), (B.BF16, (64, 128, 3, 64, 480, 6), 44, 102),
                 (B.BF16, (256, 24, 5, 16, 112, 36), 64, 137), (B.BF16, (96, 384, 3, 128, 224, 1), 33, 52), (B.BF16, (80, 192, 5, 8, 8, 2591), 187, 223),
                 (B.BF16, (80, 64, 5, 64, 224, 3), 28, 60)]
DIRECT_FASTER = [(B.F32, (32, 32, 5, 16, 16, 128)), (B.F32, (256, 384, 3, 13, 13, 128)), (B.F32, (96, 256, 5, 27, 27, 16)), (B.F32, (256, 192, 5, 16, 16, 271)),
                 (B.BF16, (32, 32, 5, 16, 16, 93)), (B.BF16, (96, 256, 5, 27, 27, 128)), (B.BF16, (256, 384, 3, 13, 13, 32)), (B.BF16, (384, 256, 3, 13, 13, 256)),
                 (B.BF16, (48, 128, 5, 64, 64, 101)), (B.BF16, (192, 192, 3, 13, 13, 77))]

# The same of grouped layers: channels of one group, and groups; us of a pass with the engine's launches, one a group, and with the one launch
GROUPED_DIRECT_FASTER = [(B.F32, (16, 96, 5, 8, 16, 10), 2, 178, 143), (B.F32, (96, 24, 3, 21, 20, 60), 2, 239, 204), (B.F32, (168, 56, 5, 25, 66, 2), 4, 1356, 541),
                         (B.F32, (16, 16, 5, 9, 99, 37), 8, 652, 465), (B.BF16, (8, 8, 5, 13, 7, 103), 2, 98, 87), (B.BF16, (48, 152, 5, 18, 9, 5), 2, 176, 127),
                         (B.BF16, (16, 8, 3, 49, 152, 186), 4, 1480, 1127), (B.BF16, (56, 48, 3, 6, 7, 4), 4, 147, 90), (B.BF16, (56, 96, 5, 56, 7, 27), 8, 464, 195)]


def test_stride1_layers_go_to_the_faster_of_the_two_kernels():
    for dtype, (cin, cout, k, h, w, batch), engine, direct in ENGINE_FASTER:
        assert engine < direct and _plan_direct(dtype, batch, h, w, cin, cout, k).ks == 0, (dtype, cin, cout, k, h, w, batch)
    for dtype, (cin, cout, k, h, w, batch) in DIRECT_FASTER:
        assert _plan_direct(dtype, batch, h, w, cin, cout, k).ks > 0, (dtype, cin, cout, k, h, w, batch)
    for dtype, (cin, cout, k, h, w, batch), groups, engine, direct in GROUPED_DIRECT_FASTER:
        assert direct < engine and _plan_direct(dtype, batch, h, w, cin, cout, k, groups).ks > 0, (dtype, cin, cout, k, h, w, batch, groups)


def test_side_stream_hides_long_sums_of_few_workgroups():
    """Filter gradients of small fully-connected layers over very many images leave the chip to the side stream's neighbours;
    those of minibatches and of large layers do not."""
    f = B.lib()["_ZN4asgd16lone_fc_wgrad_usEilll"]
    f.argtypes, f.restype = [ctypes.c_int] + [ctypes.c_long] * 3, ctypes.c_double
    for dtype, out, fin, batch, us in ((B.F32, 8, 64, 16417, 1025), (B.F32, 8, 576, 8792, 552), (B.F32, 8, 256, 10372, 650), (B.F32, 8, 256, 4435, 286)):
        assert 200 <= f(dtype, out, fin, batch) and abs(f(dtype, out, fin, batch) / us - 1) < 0.1
    assert abs(f(B.BF16, 8, 512, 11591) / 105 - 1) < 0.1
    for dtype, out, fin, batch in ((B.F32, 10, 1024, 512), (B.BF16, 10, 1024, 512), (B.F32, 8, 3456, 2904)):
        assert f(dtype, out, fin, batch) < 200
    assert f(B.F32, 4096, 4096, 16384) == 0


# Updates (arrays of parameters and state, bytes a parameter of the copy, parameters) with the us by ordinary and by non-temporal loads, each the
# mean over vectors that were swept just before and vectors that were not.
UPDATES = [(2, 0, 16000000, 51.2, 54.2), (2, 0, 24000000, 72.8, 82.2), (2, 0, 36000000, 106.0, 121.5), (2, 0, 44000000, 142.1, 148.2), (2, 0, 62000000, 212.6, 208.9),
           (2, 2, 20000000, 69.0, 74.5), (2, 2, 28000000, 93.3, 101.1), (2, 2, 36000000, 122.0, 129.2), (2, 2, 44000000, 166.7, 156.3), (2, 2, 62378344, 242.3, 219.0),
           (2, 4, 16000000, 60.4, 62.2), (2, 4, 28000000, 102.0, 106.0), (2, 4, 36000000, 146.4, 134.4), (2, 4, 62000000, 267.3, 226.2),
           (3, 0, 20000000, 89.8, 99.2), (3, 0, 32000000, 142.6, 158.2), (3, 0, 44000000, 219.5, 213.8), (3, 0, 62000000, 316.9, 303.8)]


def test_updates_read_their_vectors_by_the_faster_loads():
    f = B.lib()["_ZN4asgd12beyond_cacheEmim"]
    f.argtypes, f.restype = [ctypes.c_size_t, ctypes.c_int, ctypes.c_size_t], ctypes.c_bool
    for arrays, copy_es, n, ordinary, nontemporal in UPDATES:
        assert f(n, arrays, copy_es) == (nontemporal < ordinary), (arrays, copy_es, n)


# Nets (parameters, operations of the convolutions' gradients, images, whether they stay on one stream, whether other replicas' passes run beside) with
# the us of a step or a replay by the general gradient kernel's pushes and by those that leave room beside them.
PUSHES = [(62378344, 4.4e9 * 16, 16, False, False, 660, 630), (62378344, 4.4e9 * 128, 128, False, False, 1280, 1228), (60965224, 2.4e9 * 32, 32, False, False, 697, 655),
          (16794000, 0.08e9 * 256, 256, False, False, 334, 298), (25200000, 0.08e9 * 128, 128, False, False, 291, 273), (33600000, 0.08e9 * 16, 16, False, False, 260, 255),
          (58800000, 1e6, 64, False, False, 440, 403), (33600000, 1e6, 128, False, False, 291, 278),
          (13100000, 1e6, 64, False, False, 183, 189), (18900000, 1e6, 64, False, False, 204, 215), (25700000, 1e6, 16, False, False, 217, 230),
          (62378344, 4.4e9 * 16, 16, False, True, 4759, 4895), (62378344, 4.4e9 * 32, 32, False, True, 5606, 5643), (62378344, 4.4e9 * 96, 96, False, True, 8427, 8388),
          (62378344, 4.4e9 * 128, 128, False, True, 9872, 9756), (18900000, 1e6, 16, False, True, 1212, 1328), (18900000, 1e6, 128, False, True, 1398, 1468),
          (62378344, 4.4e9 * 16, 16, False, False, 5632, 5594), (58800000, 1e6, 16, False, False, 3219, 2982), (2060000, 1e6, 64, True, False, 99.6, 94.9)]


def test_pushes_go_to_the_faster_of_the_two_kernels():
    f = B.lib()["_ZN4asgd12fc_push_paysEmdlbb"]
    f.argtypes, f.restype = [ctypes.c_size_t, ctypes.c_double, ctypes.c_long, ctypes.c_bool, ctypes.c_bool], ctypes.c_bool
    for params, conv_flops, batch, one_stream, others, general, beside in PUSHES:
        assert f(params, conv_flops, batch, one_stream, others) == (beside < general), (params, conv_flops, batch, one_stream, others)


# Passes of up to 64 images (MiB of 16-bit parameters, MiB of workspace, replicas beside each other) with the us by ordinary and by non-temporal loads
# of the fully-connected weights.
WEIGHT_LOADS = [(112, 4, 1, 366, 381), (112, 16, 1, 379, 403), (56, 12, 1, 262, 273), (119, 72, 1, 629, 639), (119, 106, 1, 664, 679), (119, 163, 1, 678, 672),
                (119, 221, 1, 803, 787), (119, 106, 2, 4768, 4722), (119, 106, 4, 4870, 4820), (119, 163, 2, 2200, 2190), (25, 8, 4, 1041, 1076), (36, 10, 2, 1145, 1187),
                (112, 13, 4, 3125, 3174)]


def test_fully_connected_weights_are_read_by_the_faster_loads():
    f = B.lib()["_ZN4asgd16fc_split_streamsEmmi"]
    f.argtypes, f.restype = [ctypes.c_size_t, ctypes.c_size_t, ctypes.c_int], ctypes.c_bool
    for weights, workspace, replicas, ordinary, nontemporal in WEIGHT_LOADS:
        assert f(weights << 20, workspace << 20, replicas) == (nontemporal < ordinary), (weights, workspace, replicas)
