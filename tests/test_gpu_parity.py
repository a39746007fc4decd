"""Parity of the HIP path (through the C ABI) against the CPU oracle.  GPU only."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from oracle import ops as oops, asgd as oasgd
from paper_1312_6186_amd import binding as B
from paper_1312_6186_amd import workloads as wl
from gpu_harness import (GpuNet, TOL, rel_l2, oracle_inputs, compare_grads, grad_errors, error_table, gpu_decisions,
                         decisions_line, progress)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# bf16 networks store their activations in bf16: the oracle rounds at the same points so that pooling
# positions and ReLU masks are decided in the same precision on both sides
ACT = {B.F32: "f64", B.BF16: "bf16"}

RAGGED = dict(name="ragged", in_shape=(3, 37, 29), classes=10,
              layers=[("conv", 12, 5, 2, 1), ("relu",), ("conv", 20, 3, 2, 1), ("relu",), ("conv", 12, 3, 1, 0), ("relu",),
                      ("maxpool", 3, 2), ("fc", 24), ("relu",), ("dropout", 0.3, 1.5), ("fc", 16), ("relu",), ("fc", 10),
                      ("softmax_ce",)])


# six input channels and 7x7 windows: the channel-padded first layer and the two-mask form of the window gather
# (more than 32 window positions), forward, data gradient and filter gradient; a 1x1 convolution; pool 3/1
WIDE = dict(name="wide", in_shape=(6, 21, 19), classes=10,
            layers=[("conv", 8, 7, 2, 3), ("relu",), ("conv", 12, 7, 1, 3), ("relu",), ("conv", 12, 1, 1, 0), ("relu",),
                    ("maxpool", 3, 1), ("fc", 24), ("relu",), ("fc", 10), ("softmax_ce",)])


# response normalisation after CONV + RELU: before a pool, and directly under the next convolution; windows 5 and 9;
# constants far larger than the cited ones so that the cross-channel terms weigh in
LRNNET = dict(name="lrn", in_shape=(3, 21, 19), classes=10,
              layers=[("conv", 16, 3, 1, 1), ("relu",), ("lrn", 5, 0.05, 0.75, 2.0), ("maxpool", 3, 2),
                      ("conv", 24, 3, 1, 1), ("relu",), ("lrn", 9, 0.02, 0.5, 1.0),
                      ("conv", 8, 3, 1, 1), ("relu",), ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)])


# grouped ("two-column") convolutions: 2 groups of 8 -> 16 channels, 2 groups with a stride (strided data gradient
# on channel slices), 3 groups under a pool; per-group channel counts are multiples of 8
GROUPED = dict(name="grouped", in_shape=(3, 23, 21), classes=10,
               layers=[("conv", 16, 3, 1, 1), ("relu",), ("conv", 32, 3, 1, 1, 2), ("relu",), ("maxpool", 3, 2),
                       ("conv", 48, 3, 2, 1, 2), ("relu",), ("conv", 24, 3, 1, 1, 3), ("relu",), ("maxpool", 2, 2),
                       ("fc", 10), ("softmax_ce",)])


# stride-1 convolutions with equal input and output grids, in chunks of channels over a patch of pixels in LDS: 120 channels
# (a partial last chunk of channels in both element types), 3x3 and 5x5 windows, 120 output columns (a ragged
# column tile), rows that are no multiple of the tile
PATCHNET = dict(name="patch", in_shape=(3, 15, 13), classes=10,
                layers=[("conv", 120, 3, 1, 1), ("relu",), ("conv", 120, 3, 1, 1), ("relu",), ("conv", 16, 5, 1, 2), ("relu",),
                        ("maxpool", 3, 2), ("fc", 10), ("softmax_ce",)])
# the same on rows of 27 pixels with a 5x5 window: a longer run of pixels per tile, 72 output columns
PATCHWIDE = dict(name="patchwide", in_shape=(3, 8, 27), classes=10,
                 layers=[("conv", 64, 3, 1, 1), ("relu",), ("conv", 72, 5, 1, 2), ("relu",), ("conv", 8, 5, 1, 2), ("relu",),
                         ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)])

# channel counts whose chunks are not of 64 channels (48 and 40: one of 48 in 16-bit data, three of 16 in 32-bit data; 96: of 32),
# 3x3 and 5x5 windows, forward and data gradient
HALFCHUNK = dict(name="halfchunk", in_shape=(3, 14, 13), classes=10,
                 layers=[("conv", 48, 3, 1, 1), ("relu",), ("conv", 96, 3, 1, 1), ("relu",), ("conv", 40, 5, 1, 2), ("relu",),
                         ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)])


# two and four input channels: the remaining pixel widths of the narrow-pixel form of the first layer
CH2 = dict(name="ch2", in_shape=(2, 14, 12), classes=10,
           layers=[("conv", 8, 3, 2, 1), ("relu",), ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)])
CH4 = dict(name="ch4", in_shape=(4, 14, 12), classes=10,
           layers=[("conv", 8, 5, 2, 2), ("relu",), ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)])


# first layers in the window-row form with 65..96 output channels: in bf16 these run the kernel that keeps the filter bank
# in LDS and reads its fragments from staged image rows (72 channels, 7x7 stride 4 over 3 input channels, two tiles per
# image of which the second holds 4 pixels; 80 channels, 5x5 stride 1 over 4 input channels, a run of 128 pixels
# touching 7 output rows, a last tile of 53)
ROWS3 = dict(name="rows3", in_shape=(3, 45, 41), classes=10,
             layers=[("conv", 72, 7, 4, 3), ("relu",), ("maxpool", 3, 2), ("fc", 10), ("softmax_ce",)])
ROWS4 = dict(name="rows4", in_shape=(4, 19, 23), classes=10,
             layers=[("conv", 80, 5, 1, 2), ("relu",), ("maxpool", 3, 2), ("fc", 10), ("softmax_ce",)])


# a pool over more than 256 channels: the bias-gradient band sums that the pooling backward kernel leaves behind
# take more than one round of the block's threads
WIDEPOOL = dict(name="widepool", in_shape=(3, 11, 13), classes=10,
                layers=[("conv", 272, 3, 1, 1), ("relu",), ("maxpool", 3, 2), ("fc", 10), ("softmax_ce",)])


# a pool on top of a pool: the ReLU mask of the convolution below is then applied by the lower pool's backward kernel
POOLPOOL = dict(name="poolpool", in_shape=(3, 17, 15), classes=10,
                layers=[("conv", 8, 3, 1, 1), ("relu",), ("maxpool", 3, 2), ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)])


# ---------------------------------------------------------------- update / snapshot
@pytest.mark.parametrize("n,offset", [(1, 0), (1023, 0), (4099, 0), (15898, 0), (100003, 1), (1 << 20, 4)])
def test_apply_update_matches_oracle(n, offset):
    rng = np.random.default_rng(n)
    w0, v0, g = (rng.standard_normal(n + offset).astype(np.float32) for _ in range(3))
    w, v, gd = (torch.from_numpy(a).to(DEV) for a in (w0, v0, g))
    lr, mu, wd = 0.01, 0.9, 5e-4
    for _ in range(3):
        B.asgd_apply_update(w[offset:], v[offset:], gd[offset:], lr, mu, wd)
    torch.cuda.synchronize()
    wr, vr = w0[offset:].astype(np.float64), v0[offset:].astype(np.float64)
    for _ in range(3):
        oops.apply_update(wr, vr, g[offset:], np.float32(lr), np.float32(mu), np.float32(wd))
    assert rel_l2(w.cpu().numpy()[offset:], wr) < 1e-6 and rel_l2(v.cpu().numpy()[offset:], vr) < 1e-6
    np.testing.assert_array_equal(w.cpu().numpy()[:offset], w0[:offset])      # nothing before the view is touched
    np.testing.assert_array_equal(gd.cpu().numpy(), g)


@pytest.mark.parametrize("n,offset", [(1, 0), (4099, 0), (100003, 1), (1 << 20, 4)])
def test_adagrad_and_adadelta_match_oracle(n, offset):
    rng = np.random.default_rng(n + 3)
    w0 = rng.standard_normal(n + offset).astype(np.float32)
    gs = [rng.standard_normal(n + offset).astype(np.float32) for _ in range(4)]
    # Adagrad
    w = torch.from_numpy(w0).to(DEV); h = torch.zeros_like(w)
    wr, hr = w0[offset:].astype(np.float64), np.zeros(n)
    for g in gs:
        B.asgd_apply_update_adagrad(w[offset:], h[offset:], torch.from_numpy(g).to(DEV)[offset:], 0.05, 1e-7, 1e-3)
        oops.apply_adagrad(wr, hr, g[offset:], np.float32(0.05), np.float32(1e-7), np.float32(1e-3))
    torch.cuda.synchronize()
    assert rel_l2(w.cpu().numpy()[offset:], wr) < 1e-6 and rel_l2(h.cpu().numpy()[offset:], hr) < 1e-6
    np.testing.assert_array_equal(w.cpu().numpy()[:offset], w0[:offset])
    # Adadelta
    w = torch.from_numpy(w0).to(DEV); a = torch.zeros_like(w); b = torch.zeros_like(w)
    wr, ar, br = w0[offset:].astype(np.float64), np.zeros(n), np.zeros(n)
    for g in gs:
        B.asgd_apply_update_adadelta(w[offset:], a[offset:], b[offset:], torch.from_numpy(g).to(DEV)[offset:], 0.9, 1e-6, 1e-3)
        oops.apply_adadelta(wr, ar, br, g[offset:], np.float32(0.9), np.float32(1e-6), np.float32(1e-3))
    torch.cuda.synchronize()
    assert rel_l2(w.cpu().numpy()[offset:], wr) < 1e-6 and rel_l2(a.cpu().numpy()[offset:], ar) < 1e-6
    assert rel_l2(b.cpu().numpy()[offset:], br) < 1e-5       # squares of steps of order sqrt(eps): a few more ulps
    np.testing.assert_array_equal(w.cpu().numpy()[:offset], w0[:offset])


@pytest.mark.parametrize("n,offset", [(1, 0), (7, 0), (4099, 0), (100003, 3), (1 << 20, 0)])
def test_snapshot_is_bit_exact(n, offset):
    rng = np.random.default_rng(n)
    a = (rng.standard_normal(n + offset) * 10.0 ** rng.integers(-20, 20, n + offset)).astype(np.float32)
    a[:: 97] = np.float32(1.0) + np.float32(2.0 ** -8)         # exact ties
    if n > 16:
        a[offset + 1], a[offset + 2], a[offset + 3], a[offset + 4] = np.inf, -0.0, 1e-45, -1e-40
    src = torch.from_numpy(a).to(DEV)
    dst = torch.zeros(n + offset + 8, dtype=torch.bfloat16, device=DEV)
    B.asgd_snapshot(src[offset:], dst[offset:offset + n], B.BF16)
    torch.cuda.synchronize()
    got = dst.view(torch.int16).cpu().numpy().view(np.uint16)
    np.testing.assert_array_equal(got[offset:offset + n], oops.snapshot_bf16(a[offset:]))
    assert (got[offset + n:] == 0).all() and (got[:offset] == 0).all()
    dst32 = torch.zeros(n + offset, dtype=torch.float32, device=DEV)
    B.asgd_snapshot(src[offset:], dst32[offset:], B.F32)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(dst32.cpu().numpy()[offset:].view(np.uint32), a[offset:].view(np.uint32))


@pytest.mark.parametrize("dst", [B.BF16, B.F32])
@pytest.mark.parametrize("n,offset", [(1, 0), (1023, 0), (4099, 0), (100003, 1), (100003, 4), (1 << 20, 8)])
def test_fused_update_snapshot_matches_oracle_and_the_two_calls(n, offset, dst):
    rng = np.random.default_rng(n + 7)
    w0, v0, g = (rng.standard_normal(n + offset).astype(np.float32) for _ in range(3))
    lr, mu, wd = 0.01, 0.9, 5e-4
    w, v, gd = (torch.from_numpy(a).to(DEV) for a in (w0, v0, g))
    tdt = torch.bfloat16 if dst == B.BF16 else torch.float32
    copy = torch.zeros(n + offset + 8, dtype=tdt, device=DEV)
    for _ in range(2):
        B.asgd_apply_update_snapshot(w[offset:], v[offset:], gd[offset:], lr, mu, wd, copy[offset:offset + n], dst)
    torch.cuda.synchronize()
    # against the oracle: update in fp64 twice, then the fetch
    wr, vr = w0[offset:].astype(np.float64), v0[offset:].astype(np.float64)
    for _ in range(2):
        oops.apply_update(wr, vr, g[offset:], np.float32(lr), np.float32(mu), np.float32(wd))
    assert rel_l2(w.cpu().numpy()[offset:], wr) < 1e-6 and rel_l2(v.cpu().numpy()[offset:], vr) < 1e-6
    got = copy.float().cpu().numpy()
    if dst == B.BF16:
        ref = oops.round_bf16(wr.astype(np.float32).astype(np.float64))
        # fp32 update arithmetic (operands of order 1, so errors of order 1e-7) may land on the other side of a
        # rounding boundary: one bf16 step at most, plus that absolute error where the result nearly cancels
        assert np.all(np.abs(got[offset:offset + n] - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-6)
    else:
        assert rel_l2(got[offset:offset + n], wr) < 1e-6
    assert (got[:offset] == 0).all() and (got[offset + n:] == 0).all()
    # consistency of the library with itself: the copy is what the separate fetch of the same parameters gives
    sep = torch.zeros(n, dtype=tdt, device=DEV)
    B.asgd_snapshot(w[offset:], sep, dst)
    torch.cuda.synchronize()
    assert torch.equal(sep.view(torch.int16 if dst == B.BF16 else torch.int32), copy[offset:offset + n].view(torch.int16 if dst == B.BF16 else torch.int32))


# ---------------------------------------------------------------- whole-network gradient
def _net_case(cfg, batch, dtype, seed=0, step=0, worker=0, bias_noise=0.05, capsys=None, plain=True):
    """One minibatch gradient on both sides.  The graded reference is the oracle's gradient for the HIP path's
    decisions where those differ from the oracle's own (each such difference validated and counted by
    gpu_decisions); the errors against the oracle's own decisions, and for bf16 networks against the oracle that
    does not round its activations (`plain`), are reported beside it."""
    layers, in_shape = cfg["layers"], cfg["in_shape"]
    params = wl.make_params(layers, in_shape, cfg.get("seeds", {}).get("init", 2000))
    if bias_noise:
        params = (params + bias_noise * np.random.default_rng(5).standard_normal(params.size).astype(np.float32)
                  * (params == 0)).astype(np.float32)             # non-zero biases
    images, labels = wl.make_batch(in_shape, batch, cfg["classes"], cfg.get("seeds", {}).get("data", 1000))
    g = GpuNet(layers, in_shape, batch, dtype)
    onet = oracle.OracleNet(layers, in_shape)
    p64, i64 = oracle_inputs(params, images, dtype)
    loss, grads = g.fwd_bwd(params, images, labels, seed, step, worker)
    own_loss, own_grads, trace = onet.fwd_bwd(p64, i64, labels, seed, step, worker, act_dtype=ACT[dtype])
    progress(capsys, "%s batch %d: oracle pass done" % (cfg["name"], batch))
    columns = []
    trace_plain = None
    if dtype == B.BF16 and plain:
        _, plain_grads, trace_plain = onet.fwd_bwd(p64, i64, labels, seed, step, worker, act_dtype="f64")
        progress(capsys, "%s batch %d: oracle pass without activation rounding done" % (cfg["name"], batch))
        columns.append(("vs unrounded oracle", grad_errors(onet, grads, plain_grads)))
    dec, report = gpu_decisions(g, layers, trace, dtype, trace_plain)
    columns.insert(0, ("vs oracle's decisions", grad_errors(onet, grads, own_grads)))
    ref_loss, ref_grads = own_loss, own_grads
    if report["flips"]:   # follow the gradient of the HIP path's equally valid decisions
        ref_loss, ref_grads, trace = onet.fwd_bwd(p64, i64, labels, seed, step, worker, act_dtype=ACT[dtype], decisions=dec)
        progress(capsys, "%s batch %d: oracle pass on the HIP path's decisions done" % (cfg["name"], batch))
    columns.insert(0, ("graded", grad_errors(onet, grads, ref_grads)))
    text = ("%s batch %d %s: %d differing ReLU / pooling decisions: %s\n" % (cfg["name"], batch, "bf16" if dtype == B.BF16 else "f32",
                                                                            report["flips"], decisions_line(report))
            + error_table("relative L2 of the parameter gradients", columns))
    print(text)
    if capsys is not None and batch >= 32:
        progress(capsys, text.replace("\n", "\n     "))
    return g, onet, (loss, grads), (ref_loss, ref_grads, trace), (params, images, labels)


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("cfg,batch", [(wl.TINY, 8), (wl.TINY, 1), (RAGGED, 5), (RAGGED, 131), (WIDE, 3), (LRNNET, 7), (GROUPED, 6), (PATCHNET, 5),
                                       (PATCHWIDE, 3), (HALFCHUNK, 5), (CH2, 4), (CH4, 4), (ROWS3, 5), (ROWS4, 3), (WIDEPOOL, 3), (POOLPOOL, 5),
                                       (wl.SMALL, 128)],
                         ids=["tiny", "tiny-batch1", "ragged5", "ragged131", "wide", "lrn", "grouped", "patch", "patchwide", "halfchunk", "ch2", "ch4",
                              "rows3", "rows4", "widepool", "poolpool", "small"])
def test_minibatch_gradient_matches_oracle(cfg, batch, dtype):
    g, onet, (loss, grads), (ref_loss, ref_grads, trace), _ = _net_case(cfg, batch, dtype, seed=3002, step=4, worker=1)
    try:
        tol = TOL[dtype]
        assert abs(loss - ref_loss) <= tol * abs(ref_loss), (loss, ref_loss)
        compare_grads(onet, grads, ref_grads, tol, cfg["name"])
        # layer outputs, masks and pooling positions
        for li, l in enumerate(cfg["layers"]):
            nxt = cfg["layers"][li + 1][0] if li + 1 < len(cfg["layers"]) else None
            group_end = (l[0] in ("maxpool", "lrn") or (l[0] == "relu" and nxt != "dropout") or l[0] == "dropout"
                         or (l[0] in ("conv", "fc") and nxt != "relu"))
            if group_end and l[0] != "softmax_ce":
                out = g.debug(B.DEBUG_OUTPUT, li)
                assert rel_l2(out, trace[li]["out"]) < tol, ("output of layer", li)
            if l[0] == "dropout":
                np.testing.assert_array_equal(g.debug(B.DEBUG_MASK, li).reshape(trace[li]["mask"].shape), trace[li]["mask"])
    finally:
        g.close()


# Stride-1 convolutions over equal grids: channel counts around the chunks (a chunk is 16, 32, 48 or 64 channels), output
# counts around the blocks of 32 columns, and enough pixels for every tile shape to be the cheapest one somewhere; then wide
# images whose patch takes as many loads as there are window positions to bring it (chunks of 16 channels: one less), and one
# pixel more (most of these wide ones run in the general engine, which is faster there).
DIRECT_SHAPES = [(8, 8, 3, 5, 7, 3), (16, 40, 5, 6, 9, 2), (48, 136, 3, 8, 8, 4), (72, 200, 3, 6, 5, 9), (120, 96, 3, 9, 9, 4), (136, 24, 5, 7, 11, 3),
                 (24, 128, 3, 33, 31, 64), (24, 128, 3, 31, 31, 50), (24, 96, 3, 31, 31, 80), (24, 96, 3, 31, 31, 53), (24, 192, 3, 31, 31, 26),
                 (24, 192, 3, 31, 31, 40), (32, 96, 5, 13, 13, 64),
                 (48, 64, 3, 3, 223, 1), (48, 48, 3, 4, 224, 1), (80, 64, 3, 2, 479, 1), (80, 64, 3, 2, 480, 1), (128, 64, 3, 3, 111, 1), (128, 64, 3, 3, 112, 1),
                 (96, 64, 3, 2, 255, 1), (144, 64, 3, 2, 111, 1), (40, 72, 3, 2, 194, 1), (16, 104, 3, 46, 46, 12), (24, 72, 3, 65, 65, 13), (24, 72, 3, 7, 7, 449),
                 (96, 8, 5, 182, 182, 1), (24, 72, 3, 257, 257, 1), (32, 136, 3, 163, 163, 1), (24, 136, 3, 199, 199, 1)]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", DIRECT_SHAPES, ids=lambda s: "%dto%d_k%d_%dx%dx%d" % s)
def test_stride1_convolution_shapes(shape, dtype):
    cin, cout, k, h, w, batch = shape
    layers = [("conv", cin, 1, 1, 0), ("relu",), ("conv", cout, k, 1, k // 2), ("relu",), ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "direct", "in_shape": (3, h, w), "classes": 10, "layers": layers}, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "direct")
    finally:
        g.close()


# Grouped ones, all groups in one launch: channels per group around the chunks, outputs per group around the blocks of 32 columns (data gradients:
# the other way round), two to four groups, fewer pixels than a tile and many tiles.
GROUPED_SHAPES = [(16, 16, 3, 5, 7, 1, 2), (72, 120, 3, 9, 11, 3, 3), (96, 256, 5, 27, 27, 2, 2), (64, 64, 5, 12, 9, 5, 4), (144, 400, 3, 13, 13, 4, 2), (384, 384, 3, 13, 13, 40, 2)]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", GROUPED_SHAPES, ids=lambda s: "%dto%d_k%d_%dx%dx%d_g%d" % s)
def test_grouped_stride1_convolution_shapes(shape, dtype):
    cin, cout, k, h, w, batch, groups = shape
    layers = [("conv", cin, 1, 1, 0), ("relu",), ("conv", cout, k, 1, k // 2, groups), ("relu",), ("maxpool", 2, 2), ("fc", 10), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "grouped", "in_shape": (3, h, w), "classes": 10, "layers": layers}, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "grouped")
    finally:
        g.close()


# Filter gradients of such layers in bf16: output channels around the tiles of 128, 192 and 256, input channels around the
# chunks of 32 and 64, two groups, images narrower and wider than a tile of 64 pixels, pixel counts below one tile and around
# an odd and an even number of tiles, and the largest count of splits.
WGRAD_SHAPES = [(64, 128, 3, 5, 7, 1, 1), (64, 128, 3, 8, 8, 2, 1), (56, 120, 3, 8, 8, 3, 1), (128, 192, 3, 13, 13, 5, 1), (136, 184, 3, 3, 70, 3, 1),
                (64, 256, 3, 9, 3, 11, 1), (72, 248, 3, 5, 64, 2, 1), (32, 256, 5, 9, 9, 4, 1), (96, 200, 5, 11, 27, 3, 1), (64, 128, 5, 5, 5, 6, 1),
                (96, 256, 5, 7, 65, 2, 2), (128, 256, 3, 13, 13, 9, 2), (64, 96, 3, 33, 31, 40, 1)]


@pytest.mark.parametrize("shape", WGRAD_SHAPES, ids=lambda s: "%dto%d_k%d_%dx%dx%d_g%d" % s)
def test_stride1_filter_gradient_shapes(shape):
    cin, cout, k, h, w, batch, groups = shape
    layers = [("conv", cin, 1, 1, 0), ("relu",), ("conv", cout, k, 1, k // 2) + ((groups,) if groups > 1 else ()), ("relu",), ("maxpool", 2, 2), ("fc", 10),
              ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "wgrad", "in_shape": (3, h, w), "classes": 10, "layers": layers}, batch, B.BF16, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[B.BF16] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[B.BF16], "wgrad")
    finally:
        g.close()


# Filter gradients of few output channels in tiles of 32 and 64 rows: output channels around the tiles, window columns around 128, strided and
# unstrided, first layers in window-row form, few and many pixels (one range, many ranges), grouped.
FEW_CHANNEL_SHAPES = [(1, 8, 5, 1, 9, 7, 1, 1), (3, 32, 5, 1, 32, 32, 40, 1), (3, 40, 3, 2, 21, 19, 3, 1), (16, 24, 3, 1, 12, 13, 2, 1), (8, 64, 4, 2, 18, 14, 5, 1),
                      (40, 56, 3, 1, 6, 5, 4, 1), (32, 72, 5, 1, 7, 7, 3, 1), (64, 64, 3, 2, 11, 11, 6, 2), (24, 32, 5, 1, 16, 15, 33, 1)]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", FEW_CHANNEL_SHAPES, ids=lambda s: "%dto%d_k%d_s%d_%dx%dx%d_g%d" % s)
def test_few_channel_filter_gradient_shapes(shape, dtype):
    cin, cout, k, stride, h, w, batch, groups = shape
    conv = ("conv", cout, k, stride, k // 2) + ((groups,) if groups > 1 else ())
    layers = ([] if cin <= 3 else [("conv", cin, 1, 1, 0), ("relu",)]) + [conv, ("relu",), ("maxpool", 2, 2), ("fc", 16), ("relu",), ("fc", 10), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "few", "in_shape": (min(cin, 3), h, w), "classes": 10, "layers": layers}, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "few")
    finally:
        g.close()


# Convolutions of up to 32 output columns in tiles of 128 x 32, forward and data gradient, and data gradients over few pixels in K
# splits (nets that stay on one stream): columns around the tile, pixels around one tile and half the CUs, strided and unstrided; data gradients
# of strided convolutions in bf16 by tiles of 128 columns, one or two to a CU, and past them.
NARROW_SHAPES = [(32, 64, 5, 1, 7, 7, 60), (24, 96, 3, 1, 5, 5, 5), (8, 136, 3, 1, 11, 12, 1), (40, 32, 3, 2, 13, 12, 7), (32, 40, 5, 1, 16, 16, 63), (32, 40, 5, 1, 16, 16, 65),
                 (16, 8, 7, 2, 20, 18, 9), (24, 64, 5, 2, 28, 27, 22), (8, 256, 3, 2, 41, 40, 23), (32, 64, 3, 2, 33, 32, 67)]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", NARROW_SHAPES, ids=lambda s: "%dto%d_k%d_s%d_%dx%dx%d" % s)
def test_narrow_convolution_shapes(shape, dtype):
    cin, cout, k, stride, h, w, batch = shape
    layers = [("conv", cin, 3, 1, 1), ("relu",), ("conv", cout, k, stride, k // 2), ("relu",), ("maxpool", 2, 2), ("fc", 16), ("relu",), ("fc", 10), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "narrow", "in_shape": (3, h, w), "classes": 10, "layers": layers}, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "narrow")
    finally:
        g.close()


# Weight gradients of fully-connected layers, batches around the K tiles (64 in bf16, 32 in fp32).  From 512 inputs into up to 264: the
# kernel for small products (up to 1024 tiles of 16 x 16), ragged outputs.  Larger ones in tiles of 128 x 128, ragged on both sides (648 inputs) or with
# 256 tiles and more (2048 inputs): the kernel for short sums up to its limits (two K tiles; 512 with 256 tiles and more), the general one past them.
@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("out,batch", [(136, 1), (200, 31), (128, 64), (72, 65), (264, 128), (40, 129), (536, 1), (528, 31), (520, 32), (552, 33), (520, 64), (552, 65), (536, 128),
                                       (520, 129), (2040, 33), (2056, 512), (2048, 513)])
def test_fc_weight_gradient_shapes(out, batch, dtype):
    shape = (8, 8, 8) if out < 500 else (8, 9, 9) if out < 1000 else (32, 8, 8)
    layers = [("fc", out), ("relu",), ("fc", 10), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "fc", "in_shape": shape, "classes": 10, "layers": layers}, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "fc")
    finally:
        g.close()


# A pool under the first fully-connected layer, flattened by the pool's own kernels: channels with padding and one group of 16 bytes to
# many, pooled grids of one pixel, around the 256 threads of a block, of several rounds of them (whole pixels of 8 channels, or where many
# blocks share the work) and past its LDS (2048 pixels) or its share of the work (the separate kernels), odd last rows and columns, with
# and without the ReLU.
FLAT_SHAPES = [(64, 34, 33, 3, 2, True), (8, 67, 66, 2, 1, True), (24, 43, 42, 2, 1, False), (24, 44, 42, 2, 1, True), (136, 90, 91, 2, 14, True), (64, 41, 42, 3, 16, False),
               (8, 2, 3, 2, 3, True), (12, 9, 10, 3, 2, True), (72, 13, 13, 3, 3, True), (72, 13, 12, 3, 2, False), (40, 33, 32, 2, 2, True), (24, 35, 33, 3, 1, True),
               (8, 92, 92, 2, 1, True), (264, 5, 4, 2, 5, False)]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", FLAT_SHAPES, ids=lambda s: "%d_%dx%d_k%dx%d_%d" % s)
def test_pool_under_fc_shapes(shape, dtype):
    c, h, w, k, batch, relu = shape
    layers = [("conv", c, 3, 1, 1)] + [("relu",)] * relu + [("maxpool", k, 2), ("fc", 24), ("relu",), ("fc", 10), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, trace), _ = _net_case({"name": "flat", "in_shape": (3, h, w), "classes": 10, "layers": layers}, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "flat")
        pool = 1 + relu
        assert rel_l2(g.debug(B.DEBUG_OUTPUT, pool), trace[pool]["out"]) < TOL[dtype]
    finally:
        g.close()


# Response normalisation with a pool of stride 2 on top, one kernel each way: channels around a wavefront's 64 groups of 16 bytes
# (512 channels in bf16, 256 in fp32; more run separate kernels) and with padding channels, rows around the width that fits
# the forward kernel's LDS (213 pixels for windows of 3), one pooled row, an odd last row and column, every window size; many pixels in
# turn for a workgroup, with too few of them (separate kernels) and with enough.
LRNPOOL_SHAPES = [(8, 3, 4, 3, 1, 3), (12, 9, 10, 2, 5, 3), (96, 23, 21, 3, 5, 3), (40, 13, 14, 2, 9, 2), (256, 9, 6, 2, 3, 3), (264, 5, 6, 1, 7, 2), (512, 6, 5, 1, 5, 3),
                  (520, 5, 5, 1, 5, 3), (8, 7, 213, 1, 5, 3), (8, 7, 216, 1, 5, 3), (16, 4, 320, 1, 5, 2),
                  (256, 5, 30, 1, 5, 3), (256, 22, 30, 8, 5, 3), (128, 16, 32, 10, 5, 2), (128, 16, 32, 9, 5, 2), (256, 14, 37, 3, 5, 3), (256, 14, 36, 3, 5, 3)]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("shape", LRNPOOL_SHAPES, ids=lambda s: "%d_%dx%dx%d_n%d_k%d" % s)
def test_normalised_pool_shapes(shape, dtype):
    c, h, w, batch, size, k = shape
    layers = [("conv", c, 3, 1, 1), ("relu",), ("lrn", size, 0.05, 0.75, 2.0), ("maxpool", k, 2), ("fc", 10), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "lrnpool", "in_shape": (3, h, w), "classes": 10, "layers": layers}, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "lrnpool")
    finally:
        g.close()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("relu,lrn", [(True, False), (True, True), (False, False)])
def test_pooling_of_infinities_and_nans(relu, lrn, dtype):
    """A window's result is its first maximum in row-major order; a NaN is one only where it comes first (no later value
    compares greater).  Infinite pixels make NaNs in the channels beside them and in their normalisation."""
    C, H, W, batch, k = 16, 13, 11, 3, 3
    layers = [("conv", C, 1, 1, 0)] + [("relu",)] * relu + [("lrn", 5, 1e-4, 0.75, 2.0)] * lrn + [("maxpool", k, 2), ("fc", 10), ("softmax_ce",)]
    rng = np.random.default_rng(11)
    onet = oracle.OracleNet(layers, (C, H, W))
    params = np.zeros(onet.param_count, dtype=np.float32)
    params[:C * C] = np.eye(C, dtype=np.float32).reshape(-1)
    images = (rng.integers(-3, 4, size=(batch, C, H, W)) * 0.25).astype(np.float32)
    images[rng.random(images.shape) < 0.01] = np.inf
    images[rng.random(images.shape) < 0.003] = -np.inf
    g = GpuNet(layers, (C, H, W), batch, dtype)
    try:
        g.fwd_bwd(params, images, rng.integers(0, 10, batch).astype(np.int32))
        below, at = 1 + relu + lrn - 1, 1 + relu + lrn
        x = g.debug(B.DEBUG_OUTPUT, below)
        y, idx = g.debug(B.DEBUG_OUTPUT, at), g.debug(B.DEBUG_ARGMAX, at)
        best, pos = x[:, :, 0:H - 2:2, 0:W - 2:2].copy(), np.zeros(y.shape, np.uint8)
        for p in range(1, k * k):
            v = x[:, :, p // k:H - 2 + p // k:2, p % k:W - 2 + p % k:2]
            up = v > best
            best[up], pos[up] = v[up], p
        np.testing.assert_array_equal(y, best)
        np.testing.assert_array_equal(idx, pos)
        assert np.isinf(x).any() or lrn
        assert np.isnan(x).any() or (relu and not lrn)
    finally:
        g.close()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("k,stride", [(2, 2), (3, 2), (3, 1)])
def test_pooling_positions_are_bit_exact(k, stride, dtype):
    """A 1x1 convolution with identity weights and zero bias passes the image through exactly in any
    precision, so the pooling kernel and the oracle see identical values: positions (first maximum in
    row-major order, many exact ties) and pooled values must agree bit for bit."""
    C, H, W, batch = 8, 13, 11, 9
    layers = [("conv", C, 1, 1, 0), ("relu",), ("maxpool", k, stride), ("fc", 10), ("softmax_ce",)]
    onet = oracle.OracleNet(layers, (C, H, W))
    rng = np.random.default_rng(k * 10 + stride)
    params = np.zeros(onet.param_count, dtype=np.float32)
    params[:C * C] = np.eye(C, dtype=np.float32).reshape(-1)
    fc_off = onet.param_slices[3][0]
    params[fc_off:] = wl.round_to_bf16(0.1 * rng.standard_normal(params.size - fc_off).astype(np.float32))
    images = (rng.integers(-3, 4, size=(batch, C, H, W)) * 0.25).astype(np.float32)    # few distinct values: ties everywhere
    labels = rng.integers(0, 10, batch).astype(np.int32)
    g = GpuNet(layers, (C, H, W), batch, dtype)
    try:
        g.fwd_bwd(params, images, labels)
        _, _, trace = onet.fwd_bwd(params.astype(np.float64), images.astype(np.float64), labels, act_dtype=ACT[dtype])
        np.testing.assert_array_equal(g.debug(B.DEBUG_OUTPUT, 1).astype(np.float64), trace[1]["out"])
        idx = g.debug(B.DEBUG_ARGMAX, 2)
        np.testing.assert_array_equal(idx, trace[2]["argmax"])
        np.testing.assert_array_equal(g.debug(B.DEBUG_OUTPUT, 2).astype(np.float64), trace[2]["out"])
        assert (trace[1]["out"] == 0).mean() > 0.3 and len(np.unique(idx)) == k * k
    finally:
        g.close()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_fwd_bwd_is_reproducible_bit_for_bit(dtype):
    cfg = wl.SMALL
    params = wl.make_params(cfg["layers"], cfg["in_shape"], 1)
    images, labels = wl.make_batch(cfg["in_shape"], 64, 10, 2)
    g = GpuNet(cfg["layers"], cfg["in_shape"], 64, dtype)
    try:
        l1, g1 = g.fwd_bwd(params, images, labels, 7, 1, 0)
        g.grads.fill_(float("nan"))
        l2, g2 = g.fwd_bwd(params, images, labels, 7, 1, 0)
        assert l1 == l2 and g1.tobytes() == g2.tobytes()          # also: grads are overwritten, not accumulated
        l3, g3 = g.fwd_bwd(params, images, labels, 7, 2, 0)       # another step -> another dropout mask
        assert g3.tobytes() != g1.tobytes()
    finally:
        g.close()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("cfg", [wl.ALEXNET, wl.ALEXNET_LRN, wl.ALEXNET_FULL], ids=["plain", "lrn", "lrn+groups"])
def test_alexnet_layers_small_batch(cfg, dtype):
    """Every layer shape of the AlexNet-style net (without and with the response normalisation of the cited
    architecture), at a batch the oracle finishes in seconds."""
    g, onet, (loss, grads), (ref_loss, ref_grads, trace), _ = _net_case(cfg, 4, dtype, seed=3003, step=0, worker=0,
                                                                       bias_noise=0.0)
    try:
        tol = TOL[dtype]
        assert abs(loss - ref_loss) <= tol * abs(ref_loss), (loss, ref_loss)
        errs = compare_grads(onet, grads, ref_grads, tol, "alexnet")
        print(errs)
    finally:
        g.close()


# ---------------------------------------------------------------- training steps (Small config, 20 steps)
def _checked_step(g, onet, params_f32, images, labels, dtype, seed, step, worker):
    """One minibatch gradient on both sides from the same parameters; returns (gpu loss, oracle loss, oracle grads)
    after the per-tensor comparison, the oracle following the HIP path's decisions where they are valid near-ties."""
    p64, i64 = oracle_inputs(params_f32, images, dtype)
    ref_loss, ref_grads, trace = onet.fwd_bwd(p64, i64, labels, seed, step, worker, act_dtype=ACT[dtype])
    loss, grads = g.fwd_bwd(params_f32, images, labels, seed, step, worker)
    dec, report = gpu_decisions(g, onet.layers, trace, dtype)
    if report["flips"]:
        ref_loss, ref_grads, _ = onet.fwd_bwd(p64, i64, labels, seed, step, worker, act_dtype=ACT[dtype], decisions=dec)
    assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
    compare_grads(onet, grads, ref_grads, TOL[dtype], "step %d" % step)
    return loss, ref_loss, ref_grads, report["flips"]


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_small_cnn_twenty_sgd_steps(dtype):
    """Twenty momentum-SGD steps on fresh minibatches.  Graded step by step from the oracle's parameters (a
    trajectory amplifies every near-tie decision, so the free-running HIP trajectory is reported and only
    loosely bounded)."""
    cfg = wl.SMALL
    layers, in_shape, batch, T = cfg["layers"], cfg["in_shape"], cfg["batch"], 20
    lr, mu, wd = cfg["lr"], cfg["mu"], cfg["wd"]
    params0 = wl.make_params(layers, in_shape, cfg["seeds"]["init"])
    onet = oracle.OracleNet(layers, in_shape)
    seed = cfg["seeds"]["dropout"]
    tol = TOL[dtype]

    def batch_fn(a):
        return wl.make_batch(in_shape, batch, cfg["classes"], cfg["seeds"]["data"] + a)

    g = GpuNet(layers, in_shape, batch, dtype)
    try:
        w_ref, v_ref = params0.astype(np.float64), np.zeros(params0.size)
        w_free = torch.from_numpy(params0).to(DEV); v_free = torch.zeros_like(w_free)
        losses_ref, losses_free, total_flips = [], [], 0
        for a in range(T):
            images, labels = batch_fn(a)
            # free-running HIP trajectory
            lf, _ = g.fwd_bwd(w_free, images, labels, seed, a, 0)
            B.asgd_apply_update(w_free, v_free, g.grads, lr, mu, wd)
            losses_free.append(lf)
            # graded step: both sides start from the oracle's parameters
            w_in, v_in = w_ref.astype(np.float32), v_ref.astype(np.float32)
            _, ref_loss, ref_grads, flips = _checked_step(g, onet, w_in, images, labels, dtype, seed, a, 0)
            total_flips += flips
            w_gpu, v_gpu = torch.from_numpy(w_in).to(DEV), torch.from_numpy(v_in).to(DEV)
            B.asgd_apply_update(w_gpu, v_gpu, g.grads, lr, mu, wd)
            w_ref, v_ref = w_in.astype(np.float64), v_in.astype(np.float64)
            oops.apply_update(w_ref, v_ref, ref_grads, np.float32(lr), np.float32(mu), np.float32(wd))
            assert rel_l2(w_gpu.cpu().numpy(), w_ref) < tol and rel_l2(v_gpu.cpu().numpy(), v_ref) < tol
            losses_ref.append(ref_loss)
        torch.cuda.synchronize()
        e_loss, e_w = rel_l2(losses_free, losses_ref), rel_l2(w_free.cpu().numpy(), w_ref)
        print("dtype %d: %d near-tie decisions over %d steps; free-running vs oracle: loss curve %.2e, params %.2e"
              % (dtype, total_flips, T, e_loss, e_w))
        assert e_loss < 0.05 and e_w < 0.05
    finally:
        g.close()


# fully-connected layers whose weight matrices span several tiles in both directions with ragged edges
FCWIDE = dict(name="fcwide", in_shape=(3, 16, 16), classes=10,
              layers=[("conv", 8, 3, 1, 1), ("relu",), ("fc", 200), ("relu",), ("dropout", 0.5), ("fc", 136), ("relu",), ("fc", 10),
                      ("softmax_ce",)])
# enough weights for the side stream (5.3 M): a convolution under a pool, a grouped one and one without a pool behind them
FORKED = dict(name="forked", in_shape=(3, 16, 16), classes=10,
              layers=[("conv", 16, 3, 1, 1), ("relu",), ("maxpool", 2, 2), ("conv", 32, 5, 1, 2, 2), ("relu",), ("conv", 32, 3, 1, 1), ("relu",),
                      ("maxpool", 2, 2), ("fc", 2048), ("relu",), ("fc", 2048), ("relu",), ("dropout", 0.5), ("fc", 10), ("softmax_ce",)])
SENTINEL = 777.0


def _fusable_fc_slices(onet, layers):
    """(offset, count) of the fully-connected weight slices asgd_train_step_fused pushes inside the gradient kernel."""
    out = []
    for li, (w_off, w_shape, _, _) in sorted(onet.param_slices.items()):
        if layers[li][0] == "fc" and w_shape[1] % 8 == 0 and w_off % 8 == 0:
            out.append((w_off, int(np.prod(w_shape))))
    return out


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("cfg", [wl.SMALL, RAGGED, FCWIDE, FORKED], ids=["small", "ragged", "fcwide", "forked"])
def test_train_step_is_the_three_calls_bit_for_bit_and_matches_the_oracle(cfg, dtype):
    """asgd_train_step pipelines the push by layer, asgd_train_step_fused pushes the fully-connected weights inside their
    gradient kernel; the results of both must be those of fwd_bwd + update + fetch."""
    layers, in_shape, batch = cfg["layers"], cfg["in_shape"], 12
    lr, mu, wd = 0.01, 0.9, 5e-4
    params0 = wl.make_params(layers, in_shape, 2002)
    tdt = torch.bfloat16 if dtype == B.BF16 else torch.float32
    onet = oracle.OracleNet(layers, in_shape)
    runs = []
    for mode in ("calls", "step", "fused"):
        g = GpuNet(layers, in_shape, batch, dtype)
        try:
            w = torch.from_numpy(params0).to(DEV); v = torch.zeros_like(w)
            copy = torch.empty(g.P, dtype=tdt, device=DEV)
            B.asgd_snapshot(w, copy, dtype)
            losses, first = [], None
            for a in range(3):
                images, labels = wl.make_batch(in_shape, batch, cfg["classes"], 1002 + a)
                img, lab = g.to_device_images(images), torch.from_numpy(labels.astype(np.int32)).to(DEV)
                g.grads.fill_(SENTINEL)
                if mode == "step":
                    B.asgd_train_step(g.net, w, v, copy, img, lab, 77, a, 0, g.loss, g.grads, lr, mu, wd)
                elif mode == "fused":
                    B.asgd_train_step_fused(g.net, w, v, copy, img, lab, 77, a, 0, g.loss, g.grads, lr, mu, wd)
                else:
                    B.asgd_fwd_bwd(g.net, copy, img, lab, 77, a, 0, g.loss, g.grads)
                    B.asgd_apply_update(w, v, g.grads, lr, mu, wd)
                    B.asgd_snapshot(w, copy, dtype)
                torch.cuda.synchronize()
                losses.append(float(g.loss.item()))
                if a == 0:
                    first = (w.cpu().numpy().copy(), v.cpu().numpy().copy(), g.grads.cpu().numpy().copy(), images, labels)
            runs.append((w.cpu(), v.cpu(), copy.cpu(), g.grads.cpu(), losses, first))
        finally:
            g.close()
    ibits = torch.int16 if dtype == B.BF16 else torch.int32
    # the fused form: parameters, momenta, the replica's copy and the losses are the same bits; the gradient buffer too,
    # except the fused weight slices, which the call must not have touched
    (w0, v0, c0, g0, l0, _), (w2, v2, c2, g2, l2, _) = runs[0], runs[2]
    assert torch.equal(w0, w2) and torch.equal(v0, v2) and l0 == l2 and torch.equal(c0.view(ibits), c2.view(ibits))
    fusable = _fusable_fc_slices(onet, layers)
    assert fusable                                       # every one of these nets has FC layers that qualify
    expect = g0.clone()
    for off, cnt in fusable:
        expect[off:off + cnt] = SENTINEL
    assert torch.equal(g2, expect)
    runs = runs[:2]
    (w0, v0, c0, g0, l0, _), (w1, v1, c1, g1, l1, first) = runs
    assert torch.equal(w0, w1) and torch.equal(v0, v1) and torch.equal(g0, g1) and l0 == l1
    assert torch.equal(c0.view(torch.int16 if dtype == B.BF16 else torch.int32), c1.view(torch.int16 if dtype == B.BF16 else torch.int32))
    # first step against the oracle (later steps start from parameters the two sides no longer share exactly)
    wg, vg, gg, images, labels = first
    p64, i64 = oracle_inputs(params0, images, dtype)
    _, ref_grads, _ = onet.fwd_bwd(p64, i64, labels, 77, 0, 0, act_dtype=ACT[dtype])
    w_ref, v_ref = params0.astype(np.float64), np.zeros(params0.size)
    oops.apply_update(w_ref, v_ref, ref_grads, np.float32(lr), np.float32(mu), np.float32(wd))
    # a near-tie decision may differ (see the gradient tests, which validate them one by one); this net and seed have none
    assert rel_l2(gg, ref_grads) < TOL[dtype] and rel_l2(wg, w_ref) < TOL[dtype] and rel_l2(vg, v_ref) < TOL[dtype]


# ---------------------------------------------------------------- A-SGD replay
# Last layers whose logits and softmax come from one kernel (up to 16 classes) and from two, batches around its tiles of 16 rows; the gradients of a small
# fully-connected layer, weights and data, in one launch; partial sums of filter gradients that wait for the next pool (stride 2), for
# a convolution or a pool of another stride below, or for the bias gradients.
@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("classes,batch", [(2, 1), (8, 15), (9, 16), (16, 17), (17, 33), (10, 70)])
@pytest.mark.parametrize("stride", [1, 2])
def test_small_nets_in_few_launches(stride, classes, batch, dtype):
    layers = [("conv", 16, 5, 1, 2), ("relu",), ("maxpool", 3, stride), ("conv", 24, 3, 1, 1), ("relu",), ("conv", 16, 3, 1, 1), ("relu",), ("maxpool", 2, 2),
              ("fc", 40), ("relu",), ("dropout", 0.5), ("fc", classes), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "few", "in_shape": (3, 18, 14), "classes": classes, "layers": layers}, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "few")
    finally:
        g.close()


# Fully-connected forward passes and data gradients in K splits with few rows: batches around the blocks of 32 rows and past 64 (the general kernel),
# outputs and inputs around the tiles of 128 columns and the K tiles of 64, K ranges that no round of four tiles divides, a last layer of odd size.
FC_SPLIT_SHAPES = [(512, 1000, 1), (520, 1032, 31), (1032, 520, 32), (2056, 264, 33), (1024, 1088, 63), (776, 1160, 64), (512, 1000, 65)]


@pytest.mark.parametrize("shape", FC_SPLIT_SHAPES, ids=lambda s: "%dto%d_%d" % s)
def test_split_fully_connected_shapes(shape):
    fin, out, batch = shape
    layers = [("conv", 8, 1, 1, 0), ("relu",), ("fc", out), ("relu",), ("dropout", 0.5), ("fc", 1096), ("relu",), ("fc", 1003), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "fcsplit", "in_shape": (3, 1, fin // 8), "classes": 1003, "layers": layers}, batch, B.BF16, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[B.BF16] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[B.BF16], "fcsplit")
    finally:
        g.close()


# (images, outputs, inputs, K splits): rows around the blocks of 32, columns around the tiles of 128, K ranges of whole tiles of 64 and with a rest, fewer
# weight rows than columns (a last layer).
@pytest.mark.parametrize("trans", [False, True], ids=["forward", "data"])
@pytest.mark.parametrize("rows,n,k,splits", [(1, 8, 512, 2), (31, 136, 1000, 4), (33, 1008, 4096, 8), (64, 264, 3160, 7)])
def test_split_products_by_either_loads(rows, n, k, splits, trans):
    """Internal function: the partial sums are the same bits by ordinary and by non-temporal weight loads, and add up to the product."""
    f = B.lib()["_ZN4asgd8fc_splitEbPKvliS1_liiiibPfP12ihipStream_t"]
    f.argtypes = ([ctypes.c_bool, ctypes.c_void_p, ctypes.c_long, ctypes.c_int, ctypes.c_void_p, ctypes.c_long] + [ctypes.c_int] * 4
                  + [ctypes.c_bool, ctypes.c_void_p, ctypes.c_void_p])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows * n)
    b_rows = n if trans else n - 3
    a = torch.randn((rows, k), generator=gen, device=DEV).bfloat16()
    b = torch.randn((k, n) if trans else (b_rows, k), generator=gen, device=DEV).bfloat16()
    ref = a.double().cpu() @ (b if trans else torch.nn.functional.pad(b, (0, 0, 0, n - b_rows)).t()).double().cpu()
    sums = []
    for stream in (False, True):
        ws = torch.full((splits, rows, n), float("nan"), device=DEV)
        assert f(trans, a.data_ptr(), k, rows, b.data_ptr(), n if trans else k, n, b_rows, k, splits, stream, ws.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
        sums.append(ws.cpu())
    assert torch.equal(sums[0], sums[1])
    # products of 16-bit values are exact in fp32; k additions in fp32 are off by less than k * 2^-24 of the sum of the magnitudes
    bound = k * 2.0 ** -24 * (a.double().abs().cpu() @ (b if trans else torch.nn.functional.pad(b, (0, 0, 0, n - b_rows)).t()).double().abs().cpu())
    assert ((sums[0].double().sum(0) - ref).abs() <= bound).all()


# The push of fully-connected weights in its own kernel: 2048 and 2056 inputs (strips of 128, the last one whole and ragged) into outputs around the tiles
# of 64 rows, enough tiles for it and one too few; batches around what a set of fragments holds (32, 64, 128, 256 images) and past it.
PUSH_SHAPES = [(16, 16, 1000, 1), (16, 16, 1000, 17), (16, 16, 1016, 32), (16, 16, 961, 33), (16, 16, 1087, 64), (16, 16, 1000, 65), (16, 16, 1026, 128),
               (16, 16, 1000, 129), (16, 16, 1000, 256), (16, 16, 1000, 257), (16, 16, 960, 20), (1, 257, 1000, 8), (1, 257, 968, 72), (1, 257, 2048, 136)]
# Convolutions worth the room beside the push of 8192 inputs into 552 outputs, which takes a side stream in a step; more images than a replay's rule asks for.
CONV_STACK = [("conv", 64, 3, 1, 1), ("relu",), ("maxpool", 2, 2), ("conv", 128, 3, 1, 1), ("relu",), ("maxpool", 2, 2), ("fc", 552), ("relu",), ("fc", 10), ("softmax_ce",)]


def _in_push_kernel(net, outputs, inputs, batch, conv_flops, replay):
    """What the library's rules say of the largest layer of a net (internal functions): whether its push has a kernel of its own."""
    f = B.lib()["_ZN4asgd12fc_push_paysEmdlbb"]
    f.argtypes, f.restype = [ctypes.c_size_t, ctypes.c_double, ctypes.c_long, ctypes.c_bool, ctypes.c_bool], ctypes.c_bool
    params = B.asgd_param_count(net)
    return f(params, conv_flops, batch, params < 4 << 20, replay) and batch <= 256 and -(-outputs // 64) * -(-inputs // 128) >= 256


def _bits(tensors):
    torch.cuda.synchronize()
    return [t.cpu().contiguous().view(torch.uint8).numpy() for t in tensors]


def _push_inputs(layers, in_shape, batch, replicas, minibatches):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    nets = [B.asgd_net_create(layers, batch, in_shape, B.BF16) for _ in range(replicas)]
    P = B.asgd_param_count(nets[0])
    return (nets, torch.randn(P, generator=gen, device=DEV) * 0.05, torch.randn(P, generator=gen, device=DEV) * 0.01,
            torch.randn((minibatches, batch) + in_shape, generator=gen, device=DEV).bfloat16(),
            torch.randint(0, 10, (minibatches, batch), generator=gen, device=DEV, dtype=torch.int32))


def _step_bits(net, params0, mom0, images, labels, fused):
    w, v, copy, grads, loss = params0.clone(), mom0.clone(), torch.empty_like(params0, dtype=torch.bfloat16), torch.zeros_like(params0), torch.zeros(1, device=DEV)
    B.asgd_snapshot(w, copy, B.BF16)
    if fused:
        B.asgd_train_step_fused(net, w, v, copy, images[0], labels[0], 3, 0, 0, loss, grads, 0.01, 0.9, 5e-4)
    else:
        B.asgd_fwd_bwd(net, copy, images[0], labels[0], 3, 0, 0, loss, grads)
        B.asgd_apply_update_snapshot(w, v, grads, 0.01, 0.9, 5e-4, copy, B.BF16)
    return _bits([w, v, copy, loss])


def _replay_bits(nets, params0, mom0, images, labels, offset):
    """Six updates of three replicas: the first two pushes are fetched by none, the third by all three, the last three leave their gradients.
    offset: parameters that many floats behind a 16-byte boundary."""
    P, W, T = params0.numel(), 3, 6

    def vec(src):
        t = torch.zeros(P + offset, device=DEV)[offset:]
        t.copy_(src)
        return t
    params, mom = vec(params0), vec(mom0)
    copies, grads = [torch.zeros(P, dtype=torch.bfloat16, device=DEV) for _ in range(W)], [torch.zeros(P, device=DEV) for _ in range(W)]
    losses, log = torch.zeros(T, device=DEV), torch.zeros((T, 3), dtype=torch.int32, device=DEV)
    B.asgd_replay_run(nets, params, mom, copies, grads, images, labels, np.array([0, 1, 2, 0, 1, 2], np.int32), np.array([0, 0, 0, 3, 3, 3], np.int32), 0.01, 0.9, 5e-4, 9,
                      losses, log)
    return _bits([params.clone(), mom.clone(), losses, log] + copies + grads)


@pytest.mark.parametrize("shape", PUSH_SHAPES, ids=lambda s: "%dx%d_%d_%d" % s)
def test_pushed_weights_are_the_calls_bit_for_bit(shape):
    """One fused step against the separate calls, and a replay against the separate kernels that parameters at a 4-byte offset take: parameters, momenta, the
    copies of several fetches at once, the gradients left."""
    h, w_, out, batch = shape
    layers = [("conv", 8, 1, 1, 0), ("relu",), ("fc", out), ("softmax_ce",)]
    nets, params0, mom0, images, labels = _push_inputs(layers, (3, h, w_), batch, 3, 6)
    try:
        inside = out > 960 and out < 2048 and batch <= 256   # 2048 outputs: a net with a side stream and nothing to run beside the push
        assert all(_in_push_kernel(nets[0], out, 8 * h * w_, batch, 0.0, r) == inside for r in (False, True))
        for a, b in zip(_step_bits(nets[0], params0, mom0, images, labels, True), _step_bits(nets[0], params0, mom0, images, labels, False)):
            np.testing.assert_array_equal(a, b)
        for a, b in zip(_replay_bits(nets, params0, mom0, images, labels, 0), _replay_bits(nets, params0, mom0, images, labels, 1)):
            np.testing.assert_array_equal(a, b)
    finally:
        for n in nets:
            B.asgd_net_destroy(n)


@pytest.mark.parametrize("batch", [65, 136])
def test_pushes_beside_convolutions_are_the_calls_bit_for_bit(batch):
    nets, params0, mom0, images, labels = _push_inputs(CONV_STACK, (3, 32, 32), batch, 3, 6)
    try:
        assert B.asgd_param_count(nets[0]) >= 4 << 20
        flops = 2.0 * batch * (1024 * 64 * 27 + 2 * 256 * 128 * 576)   # filter gradients, and the second layer's data gradient
        assert all(_in_push_kernel(nets[0], 552, 8192, batch, flops, r) for r in (False, True))
        for a, b in zip(_step_bits(nets[0], params0, mom0, images, labels, True), _step_bits(nets[0], params0, mom0, images, labels, False)):
            np.testing.assert_array_equal(a, b)
        for a, b in zip(_replay_bits(nets, params0, mom0, images, labels, 0), _replay_bits(nets, params0, mom0, images, labels, 1)):
            np.testing.assert_array_equal(a, b)
    finally:
        for n in nets:
            B.asgd_net_destroy(n)


@pytest.mark.parametrize("shape", [(16, 16, 1000, 65), (1, 257, 968, 72)], ids=lambda s: "%dx%d_%d_%d" % s)
def test_pushes_of_local_steps_are_the_calls_bit_for_bit(shape):
    """Local steps, whose gradients are summed up too (in the general gradient kernel), against the separate kernels that parameters at a 4-byte offset take."""
    h, w_, out, batch = shape
    layers = [("conv", 8, 1, 1, 0), ("relu",), ("fc", out), ("softmax_ce",)]
    nets, params0, mom0, images, labels = _push_inputs(layers, (3, h, w_), batch, 2, 4)
    P = params0.numel()
    try:
        replays = []
        for offset in (0, 1):
            def vec():
                return torch.zeros(P + offset, device=DEV)[offset:]
            params, mom, local = vec(), vec(), [[vec() for _ in range(2)] for _ in range(3)]
            params.copy_(params0)
            copies, grads = [torch.zeros(P, dtype=torch.bfloat16, device=DEV) for _ in range(2)], [torch.zeros(P, device=DEV) for _ in range(2)]
            losses, log = torch.zeros(4, device=DEV), torch.zeros((2, 3), dtype=torch.int32, device=DEV)
            B.asgd_replay_nsync_run(nets, 2, params, mom, local[0], local[1], local[2], copies, grads, images, labels, np.array([0, 1], np.int32), np.array([0, 1], np.int32),
                                    0.01, 0.9, 5e-4, 9, losses, log)
            replays.append(_bits([params.clone(), mom.clone(), losses, log] + copies + grads + [t.clone() for l in local for t in l]))
        for a, b in zip(*replays):
            np.testing.assert_array_equal(a, b)
    finally:
        for n in nets:
            B.asgd_net_destroy(n)


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_asgd_replay_matches_oracle_and_logs_the_schedule(dtype):
    cfg = wl.TINY
    layers, in_shape, batch = cfg["layers"], cfg["in_shape"], 8
    # The configuration's step size (0.01) and momentum in fp32.  On this random-label problem that step size makes the
    # stale trajectory overshoot (losses climb from 3.9 to 40 within a dozen updates); fp32 still agrees to 1e-4 there,
    # but a diverging trajectory multiplies bf16's rounding differences from update to update, so the bf16 run is
    # graded on the same schedule at a step size where the trajectory is stable.  Weight decay is on, to exercise it.
    W, T, lr, mu, wd = 4, 24, (cfg["lr"] if dtype == B.F32 else 0.001), cfg["mu"], 5e-4
    worker, rv = B.asgd_schedule_generate(T, 4005, W, 3)
    w_o, rv_o = oops.schedule(T, 4005, W, 3)
    np.testing.assert_array_equal(worker, w_o); np.testing.assert_array_equal(rv, rv_o)
    params0 = wl.make_params(layers, in_shape, 2001)
    batches = [wl.make_batch(in_shape, batch, 10, 1005 + a) for a in range(T)]
    if dtype == B.BF16:
        batches = [(wl.round_to_bf16(i), l) for i, l in batches]
    onet = oracle.OracleNet(layers, in_shape)
    w_ref, v_ref, losses_ref, log_ref = oasgd.replay(onet, params0, worker, rv, lambda a: batches[a], np.float32(lr),
                                                     np.float32(mu), np.float32(wd), dropout_seed=9,
                                                     worker_dtype="bf16" if dtype == B.BF16 else "f32", act_dtype=ACT[dtype])
    tdt = torch.bfloat16 if dtype == B.BF16 else torch.float32
    nets = [B.asgd_net_create(layers, batch, in_shape, dtype) for _ in range(W)]
    P = B.asgd_param_count(nets[0])
    try:
        results = []
        for rep in range(2):
            params = torch.from_numpy(params0).to(DEV); mom = torch.zeros_like(params)
            copies = [torch.empty(P, dtype=tdt, device=DEV) for _ in range(W)]
            grads = [torch.empty(P, dtype=torch.float32, device=DEV) for _ in range(W)]
            images = torch.from_numpy(np.stack([b[0] for b in batches])).to(DEV).to(tdt).contiguous()
            labels = torch.from_numpy(np.stack([b[1] for b in batches]).astype(np.int32)).to(DEV)
            losses = torch.zeros(T, dtype=torch.float32, device=DEV)
            log = torch.full((T, 3), -7, dtype=torch.int32, device=DEV)
            B.asgd_replay_run(nets, params, mom, copies, grads, images, labels, worker, rv, lr, mu, wd, 9, losses, log)
            torch.cuda.synchronize()
            results.append((params.cpu().numpy(), mom.cpu().numpy(), losses.cpu().numpy(), log.cpu().numpy()))
        p, m, ls, lg = results[0]
        np.testing.assert_array_equal(lg, log_ref)               # (update, worker, version read) as prescribed
        tol = TOL[dtype]
        # the accumulated parameter change, not the parameters (which the initial weights dominate), and the momentum
        errs = rel_l2(ls, losses_ref), rel_l2(p - params0, w_ref - params0), rel_l2(m, v_ref)
        print("replay dtype %d: losses %.2e, parameter change %.2e, momentum %.2e" % ((dtype,) + errs))
        assert max(errs) < tol, errs
        for a, b in zip(results[0], results[1]):                  # replay is reproducible bit for bit
            assert a.tobytes() == b.tobytes()
    finally:
        for n in nets:
            B.asgd_net_destroy(n)


@pytest.mark.parametrize("n,offset", [(1, 0), (4099, 0), (100003, 1), (1 << 20, 4)])
def test_accumulate_matches_numpy(n, offset):
    rng = np.random.default_rng(n)
    g = [rng.standard_normal(n + offset).astype(np.float32) for _ in range(3)]
    acc = torch.full((n + offset,), 7.0, dtype=torch.float32, device=DEV)
    for i, gi in enumerate(g):
        B.asgd_accumulate(acc[offset:], torch.from_numpy(gi).to(DEV)[offset:], first=(i == 0))
    torch.cuda.synchronize()
    want = (g[0][offset:] + g[1][offset:]) + g[2][offset:]      # fp32, in push order
    np.testing.assert_array_equal(acc.cpu().numpy()[offset:], want)
    assert (acc.cpu().numpy()[:offset] == 7.0).all()


# Fully-connected weights of more than 1024 tiles of 16 x 16, ragged on both sides of the tiles of 128 x 128: past the kernel for small products
WIDE_FC = {"layers": [("conv", 24, 3, 1, 1), ("relu",), ("maxpool", 2, 2), ("fc", 264), ("relu",), ("dropout", 0.5), ("fc", 1032), ("relu",), ("fc", 10), ("softmax_ce",)],
           "in_shape": (3, 14, 14)}


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("n_sync", [0, 1, 3])
@pytest.mark.parametrize("cfg", [RAGGED, WIDE_FC], ids=["ragged", "wide_fc"])
def test_replay_with_fused_pushes_is_the_separate_kernels_bit_for_bit(cfg, n_sync, dtype):
    """Parameters at a 4-byte offset go through the separate update, snapshot and accumulate kernels: everything that the
    replay leaves, the replicas' gradients among it, must be the same.  Six replicas fetch one version (a push writes
    four copies at most), and the last replica's only gradient is of an early version."""
    layers, shape, batch, W = cfg["layers"], cfg["in_shape"], 8, 6   # minibatches of a multiple of 16 bytes
    worker = np.array([0, 1, 2, 3, 4, 5, 0, 1, 2, 3, 4, 0, 1], np.int32)
    rv = np.array([0, 0, 1, 1, 4, 0, 6, 6, 6, 6, 6, 7, 12], np.int32)
    T, k, tdt = len(worker), max(n_sync, 1), torch.bfloat16 if dtype == B.BF16 else torch.float32
    nets = [B.asgd_net_create(layers, batch, shape, dtype) for _ in range(W)]
    P = B.asgd_param_count(nets[0])
    rng = np.random.default_rng(21)
    params0 = wl.make_params(layers, shape, 2001)
    images = torch.from_numpy(rng.standard_normal((T * k, batch) + shape).astype(np.float32)).to(DEV).to(tdt)
    labels = torch.from_numpy(rng.integers(0, 10, (T * k, batch)).astype(np.int32)).to(DEV)
    try:
        results = []
        for offset in (0, 1):
            def vec(value=0.0):
                return torch.full((P + offset,), value, dtype=torch.float32, device=DEV)[offset:]
            params, mom = vec(), vec()
            params.copy_(torch.from_numpy(params0))
            wp, wm, wa = ([vec() for _ in range(W)] for _ in range(3))
            copies = [torch.full((P,), float("nan"), dtype=tdt, device=DEV) for _ in range(W)]
            grads = [torch.full((P,), float("nan"), dtype=torch.float32, device=DEV) for _ in range(W)]
            losses = torch.zeros(T * k, dtype=torch.float32, device=DEV)
            log = torch.full((T, 3), -7, dtype=torch.int32, device=DEV)
            for _ in range(2):
                if n_sync:
                    B.asgd_replay_nsync_run(nets, n_sync, params, mom, wp, wm, wa, copies, grads, images, labels, worker, rv, 0.001, 0.9, 5e-4, 9, losses, log)
                else:
                    B.asgd_replay_run(nets, params, mom, copies, grads, images, labels, worker, rv, 0.001, 0.9, 5e-4, 9, losses, log)
            torch.cuda.synchronize()
            results.append([t.cpu().contiguous().view(torch.uint8).numpy() for t in [params.clone(), mom.clone(), losses, log] + copies + grads + (wp + wm + wa if n_sync else [])])
        np.testing.assert_array_equal(log.cpu().numpy(), np.stack([np.arange(T), worker, rv], 1))
        assert all(np.isfinite(g.cpu().numpy()).all() for g in grads)
        for a, b in zip(*results):
            np.testing.assert_array_equal(a, b)
    finally:
        for n in nets:
            B.asgd_net_destroy(n)


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("n_sync", [1, 3])
def test_nsync_replay_matches_oracle_and_logs_the_schedule(n_sync, dtype):
    cfg = wl.TINY
    layers, in_shape, batch = cfg["layers"], cfg["in_shape"], 8
    W, T, lr, mu, wd = 3, 9, (cfg["lr"] if dtype == B.F32 else 0.001), cfg["mu"], 5e-4    # step sizes as in the replay test above
    worker, rv = B.asgd_schedule_generate(T, 4005, W, 2)
    params0 = wl.make_params(layers, in_shape, 2001)
    batches = [wl.make_batch(in_shape, batch, 10, 1105 + b) for b in range(T * n_sync)]
    if dtype == B.BF16:
        batches = [(wl.round_to_bf16(i), l) for i, l in batches]
    onet = oracle.OracleNet(layers, in_shape)
    wdt = "bf16" if dtype == B.BF16 else "f32"
    w_ref, v_ref, losses_ref, log_ref, local_ref = oasgd.replay_nsync(
        onet, params0, worker, rv, lambda a, i: batches[a * n_sync + i], n_sync, np.float32(lr), np.float32(mu), np.float32(wd),
        dropout_seed=9, worker_dtype=wdt, act_dtype=ACT[dtype])
    tdt = torch.bfloat16 if dtype == B.BF16 else torch.float32
    nets = [B.asgd_net_create(layers, batch, in_shape, dtype) for _ in range(W)]
    P = B.asgd_param_count(nets[0])
    try:
        results = []
        for rep in range(2):
            params = torch.from_numpy(params0).to(DEV); mom = torch.zeros_like(params)
            f32 = lambda: [torch.zeros(P, dtype=torch.float32, device=DEV) for _ in range(W)]
            wp, wm, wa, grads = f32(), f32(), f32(), f32()
            copies = [torch.empty(P, dtype=tdt, device=DEV) for _ in range(W)]
            images = torch.from_numpy(np.stack([b[0] for b in batches])).to(DEV).to(tdt).contiguous()
            labels = torch.from_numpy(np.stack([b[1] for b in batches]).astype(np.int32)).to(DEV)
            losses = torch.zeros(T * n_sync, dtype=torch.float32, device=DEV)
            log = torch.full((T, 3), -7, dtype=torch.int32, device=DEV)
            B.asgd_replay_nsync_run(nets, n_sync, params, mom, wp, wm, wa, copies, grads, images, labels, worker, rv, lr, mu, wd, 9,
                                    losses, log)
            torch.cuda.synchronize()
            results.append([params.cpu().numpy(), mom.cpu().numpy(), losses.cpu().numpy(), log.cpu().numpy()]
                           + [t.cpu().numpy() for t in wp + wm])
        p, m, ls, lg = results[0][:4]
        np.testing.assert_array_equal(lg, log_ref)
        tol = TOL[dtype]
        errs = rel_l2(ls, np.array(losses_ref).ravel()), rel_l2(p - params0, w_ref - params0), rel_l2(m, v_ref)
        print("n_sync %d dtype %d: losses %.2e, parameter change %.2e, momentum %.2e" % ((n_sync, dtype) + errs))
        assert max(errs) < tol, errs
        for k in range(W):                                       # the replicas' own parameters (their change) and momentum
            assert rel_l2(results[0][4 + k] - params0, local_ref[k][0] - params0) < tol and rel_l2(results[0][4 + W + k], local_ref[k][1]) < tol
        for a, b in zip(results[0], results[1]):                  # reproducible bit for bit
            assert a.tobytes() == b.tobytes()
        if n_sync == 1:                                           # the plain replay, bit for bit
            params = torch.from_numpy(params0).to(DEV); mom = torch.zeros_like(params)
            copies = [torch.empty(P, dtype=tdt, device=DEV) for _ in range(W)]
            grads = [torch.empty(P, dtype=torch.float32, device=DEV) for _ in range(W)]
            losses = torch.zeros(T, dtype=torch.float32, device=DEV)
            log = torch.full((T, 3), -7, dtype=torch.int32, device=DEV)
            B.asgd_replay_run(nets, params, mom, copies, grads, images, labels, worker, rv, lr, mu, wd, 9, losses, log)
            torch.cuda.synchronize()
            assert params.cpu().numpy().tobytes() == p.tobytes() and losses.cpu().numpy().tobytes() == ls.tobytes()
    finally:
        for n in nets:
            B.asgd_net_destroy(n)


# ---------------------------------------------------------------- full size, in the configurations bench.py times
def _full_size_case(batch, dtype, capsys, plain):
    """The AlexNet-style net at a benchmarked batch size against the oracle on the WHOLE batch: loss, every
    parameter tensor's gradient, the logits and the dropout masks (bit for bit)."""
    cfg = wl.ALEXNET
    layers = cfg["layers"]
    seed, step, worker = cfg["seeds"]["dropout"], 3, 0
    g, onet, (loss, grads), (ref_loss, ref_grads, trace), _ = _net_case(cfg, batch, dtype, seed=seed, step=step, worker=worker,
                                                                       bias_noise=0.0, capsys=capsys, plain=plain)
    try:
        tol = TOL[dtype]
        assert np.isfinite(grads).all() and np.isfinite(loss)
        assert abs(loss - ref_loss) <= tol * abs(ref_loss), (loss, ref_loss)
        compare_grads(onet, grads, ref_grads, tol, "alexnet bs%d" % batch)
        logits = g.debug(B.DEBUG_OUTPUT, len(layers) - 2).reshape(batch, -1).astype(np.float64)
        assert rel_l2(logits, trace[len(layers) - 2]["out"]) < tol
        for li, l in enumerate(layers):
            if l[0] == "dropout":   # masks of the full batch, bit for bit
                np.testing.assert_array_equal(g.debug(B.DEBUG_MASK, li).reshape(batch, -1), trace[li]["mask"].reshape(batch, -1))
    finally:
        g.close()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16], ids=["f32", "bf16"])
def test_alexnet_bs128_gradient_matches_oracle(dtype, capsys):
    """Batch 128: the launch configuration of the headline benchmark (its split factors, tile shapes and
    reductions), in both compute types."""
    _full_size_case(128, dtype, capsys, plain=True)


@pytest.mark.parametrize("dtype", [B.F32, B.BF16], ids=["f32", "bf16"])
def test_alexnet_bs128_fused_step_is_the_calls_bit_for_bit(dtype):
    """The step `bench.py` times (asgd_train_step_fused at batch 128) against fwd_bwd + apply_update + snapshot, whose
    gradient the test above grades against the oracle: parameters, momenta, the replica's copy and the loss must be
    the same bits after two steps, the gradient buffer too outside the weight slices that are pushed inside their
    GEMM, and those slices must not have been written."""
    cfg = wl.ALEXNET
    layers, in_shape, batch = cfg["layers"], cfg["in_shape"], 128
    lr, mu, wd = cfg["lr"], cfg["mu"], cfg["wd"]
    params0 = wl.make_params(layers, in_shape, cfg["seeds"]["init"])
    tdt = torch.bfloat16 if dtype == B.BF16 else torch.float32
    onet = oracle.OracleNet(layers, in_shape)
    runs = []
    g = GpuNet(layers, in_shape, batch, dtype)
    try:
        for fused in (False, True):
            w = torch.from_numpy(params0).to(DEV); v = torch.zeros_like(w)
            copy = torch.empty(g.P, dtype=tdt, device=DEV)
            B.asgd_snapshot(w, copy, dtype)
            losses = []
            for a in range(2):
                images, labels = wl.make_batch(in_shape, batch, cfg["classes"], cfg["seeds"]["data"] + a)
                img, lab = g.to_device_images(images), torch.from_numpy(labels.astype(np.int32)).to(DEV)
                g.grads.fill_(SENTINEL)
                if fused:
                    B.asgd_train_step_fused(g.net, w, v, copy, img, lab, cfg["seeds"]["dropout"], a, 0, g.loss, g.grads, lr, mu, wd)
                else:
                    B.asgd_fwd_bwd(g.net, copy, img, lab, cfg["seeds"]["dropout"], a, 0, g.loss, g.grads)
                    B.asgd_apply_update(w, v, g.grads, lr, mu, wd)
                    B.asgd_snapshot(w, copy, dtype)
                torch.cuda.synchronize()
                losses.append(float(g.loss.item()))
            runs.append((w.cpu(), v.cpu(), copy.cpu(), g.grads.cpu(), losses))
            del w, v, copy
    finally:
        g.close()
    ibits = torch.int16 if dtype == B.BF16 else torch.int32
    (w0, v0, c0, g0, l0), (w1, v1, c1, g1, l1) = runs
    assert l0 == l1 and np.isfinite(l0).all()
    assert torch.equal(w0, w1) and torch.equal(v0, v1) and torch.equal(c0.view(ibits), c1.view(ibits))
    fusable = _fusable_fc_slices(onet, layers)
    assert len(fusable) == 3                            # the three fully-connected weight matrices
    expect = g0.clone()
    for off, cnt in fusable:
        expect[off:off + cnt] = SENTINEL
    assert torch.equal(g1, expect)


def test_alexnet_bs256_bf16_gradient_matches_oracle(capsys):
    """Batch 256 in bf16: twice the GEMM rows of the headline configuration, other tile and split choices."""
    _full_size_case(256, B.BF16, capsys, plain=False)


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_alexnet_full_batch_gradient_is_the_mean_of_its_chunks(dtype):
    """A property that holds at any size: the minibatch-mean gradient of 128 images equals the mean of the
    gradients of its four 32-image chunks (dropout off so the masks do not depend on the position in the batch).
    The 32-image plan is the A-SGD worker shape; small batches of the same net are checked against the oracle
    directly in test_alexnet_layers_small_batch."""
    cfg = wl.ALEXNET
    layers = [l if l[0] != "dropout" else ("dropout", 0.0) for l in cfg["layers"]]
    in_shape = cfg["in_shape"]
    params = wl.make_params(layers, in_shape, cfg["seeds"]["init"])
    images, labels = wl.make_batch(in_shape, 128, cfg["classes"], cfg["seeds"]["data"] + 1)
    big, small = GpuNet(layers, in_shape, 128, dtype), GpuNet(layers, in_shape, 32, dtype)
    try:
        loss, grads = big.fwd_bwd(params, images, labels)
        acc, lsum = np.zeros_like(grads, dtype=np.float64), 0.0
        for c in range(4):
            l_c, g_c = small.fwd_bwd(params, images[32 * c:32 * c + 32], labels[32 * c:32 * c + 32])
            acc += g_c; lsum += l_c
        onet = oracle.OracleNet(layers, in_shape)
        assert abs(loss - lsum / 4) <= 1e-5 * abs(loss)
        compare_grads(onet, grads, acc / 4, 1e-4 if dtype == B.F32 else 2e-3, "chunks")
    finally:
        big.close(); small.close()


class _PlanView:
    """What gpu_decisions needs of a plan that a replay ran on: the exports of its last forward pass."""
    def __init__(self, net, batch):
        self.net, self.batch = net, batch

    def debug(self, what, layer):
        shape = B.asgd_layer_shape(self.net, layer)
        dst = torch.empty((self.batch,) + shape, dtype=torch.float32 if what == B.DEBUG_OUTPUT else torch.uint8, device=DEV)
        B.asgd_debug_get(self.net, what, layer, dst)
        torch.cuda.synchronize()
        return dst.cpu().numpy()


def test_asgd_replay_at_worker_shape_matches_oracle(capsys):
    """Four workers on the AlexNet-style net at batch 32 in bf16 (the worker shape of the on-one-GPU A-SGD
    configuration, with its step size, momentum and weight decay), a seeded schedule with stale reads.
    (i) Twelve updates: the device-side log equals the prescribed schedule and two replays agree bit for bit.
    (ii) Four updates, one per worker, so that every worker's plan still holds the ReLU masks and pooling positions
    of its update afterwards: the oracle replays the same schedule, taking for each update the HIP path's decisions
    after gpu_decisions has validated them against its own forward pass on the version that update reads; losses,
    accumulated parameter change and momentum must then agree per tensor at the bf16 tolerance."""
    cfg = wl.ALEXNET
    layers, in_shape, batch, W = cfg["layers"], cfg["in_shape"], 32, 4
    lr, mu, wd = cfg["lr"], cfg["mu"], cfg["wd"]
    params0 = wl.make_params(layers, in_shape, cfg["seeds"]["init"])
    rng = np.random.default_rng(1005)
    T_long, T = 12, 4
    images_np = wl.round_to_bf16(rng.standard_normal((T_long, batch) + tuple(in_shape), dtype=np.float32))
    labels_np = rng.integers(0, cfg["classes"], size=(T_long, batch), dtype=np.int32)
    nets = [B.asgd_net_create(layers, batch, in_shape, B.BF16) for _ in range(W)]
    P = B.asgd_param_count(nets[0])
    try:
        images = torch.from_numpy(images_np).to(DEV).to(torch.bfloat16).contiguous()
        labels = torch.from_numpy(labels_np).to(DEV)

        def run(n_updates, seed):
            worker, rv = B.asgd_schedule_generate(n_updates, seed, W, 3)
            params = torch.from_numpy(params0).to(DEV); mom = torch.zeros_like(params)
            copies = [torch.empty(P, dtype=torch.bfloat16, device=DEV) for _ in range(W)]
            grads = [torch.empty(P, dtype=torch.float32, device=DEV) for _ in range(W)]
            losses = torch.zeros(n_updates, dtype=torch.float32, device=DEV)
            log = torch.full((n_updates, 3), -7, dtype=torch.int32, device=DEV)
            B.asgd_replay_run(nets, params, mom, copies, grads, images, labels, worker, rv, lr, mu, wd, 3003, losses, log)
            torch.cuda.synchronize()
            return worker, rv, (params.cpu().numpy(), mom.cpu().numpy(), losses.cpu().numpy(), log.cpu().numpy())

        # (i)
        worker, rv, first = run(T_long, 4005)
        _, _, second = run(T_long, 4005)
        assert (np.arange(T_long) - rv).max() == 3
        np.testing.assert_array_equal(first[3], np.stack([np.arange(T_long), worker, rv], 1))
        assert np.isfinite(first[2]).all() and (first[2] > 0).all()
        for a, b in zip(first, second):
            assert a.tobytes() == b.tobytes()
        # (ii) a schedule seed whose first four rows read versions 0, 0, 1 or 2, and a version at least 2 behind
        seed = next(sd for sd in range(4005, 4100) if (np.arange(T) - oops.schedule(T, sd, W, 3)[1]).max() >= 2)
        worker, rv, (p, m, ls, lg) = run(T, seed)
        progress(capsys, "replay at worker shape: HIP side done (schedule seed %d, versions read %s); oracle replay starts" % (seed, list(rv)))
        onet = oracle.OracleNet(layers, in_shape)
        flips = []

        def decisions_fn(a, wc, imgs, labs):
            _, _, trace = onet.fwd_bwd(wc, imgs, labs, 3003, a, int(worker[a]), want_grads=False, act_dtype="bf16")
            dec, report = gpu_decisions(_PlanView(nets[int(worker[a])], batch), layers, trace, B.BF16)
            flips.append(report["flips"])
            progress(capsys, "oracle replay: update %d, %d decisions of the HIP path followed" % (a, report["flips"]))
            return dec

        w_ref, v_ref, losses_ref, log_ref = oasgd.replay(onet, params0, worker, rv, lambda a: (images_np[a], labels_np[a]), np.float32(lr),
                                                         np.float32(mu), np.float32(wd), dropout_seed=3003, worker_dtype="bf16",
                                                         act_dtype="bf16", decisions_fn=decisions_fn)
        np.testing.assert_array_equal(lg, log_ref)
        tol = TOL[B.BF16]
        e_loss = rel_l2(ls, losses_ref)
        table = error_table("worker-shape replay, %d updates, relative L2 per tensor" % T,
                            [("parameter change", grad_errors(onet, p - params0, w_ref - params0)), ("momentum", grad_errors(onet, m, v_ref))])
        progress(capsys, ("losses %.2e; " % e_loss) + table.replace("\n", "\n     "))
        assert e_loss < tol
        compare_grads(onet, p - params0, w_ref - params0, tol, "parameter change")
        compare_grads(onet, m, v_ref, tol, "momentum")
    finally:
        for n in nets:
            B.asgd_net_destroy(n)


def test_out_of_range_label_gives_nan_loss_and_no_fault():
    """A label outside [0, classes) is never used as an address: the loss is NaN, the gradient stays finite (that
    row's logit gradient is softmax / B) and every kernel ends normally; the next call with valid labels is unaffected."""
    cfg = wl.TINY
    g = GpuNet(cfg["layers"], cfg["in_shape"], 8, B.F32)
    try:
        params = wl.make_params(cfg["layers"], cfg["in_shape"], 1)
        images, labels = wl.make_batch(cfg["in_shape"], 8, 10, 2)
        good_loss, good_grads = g.fwd_bwd(params, images, labels)
        for bad in (-1, 10, 2 ** 31 - 1, -2 ** 31):
            lab = labels.copy(); lab[3] = bad
            loss, grads = g.fwd_bwd(params, images, lab)
            assert np.isnan(loss) and np.isfinite(grads).all()
        loss, grads = g.fwd_bwd(params, images, labels)
        assert loss == good_loss and grads.tobytes() == good_grads.tobytes()
    finally:
        g.close()


# Bias gradients: bands of rows below and above four rows per lane (a layer without a pool), and of a layer under a pool from
# fewer bands than the lanes of a workgroup to more than eight times as many.
# Channel counts that fill their last chunk in part (40 and 56 of 48 and 64): its zeros lie where the partial sums of the filter
# gradients are written later in a pass.
PARTCHUNK = dict(name="partchunk", in_shape=(3, 19, 17), classes=10,
                 layers=[("conv", 40, 3, 1, 1), ("relu",), ("conv", 56, 3, 1, 1), ("relu",), ("conv", 24, 5, 1, 2), ("relu",), ("maxpool", 2, 2),
                         ("conv", 104, 3, 1, 1), ("relu",), ("conv", 40, 5, 1, 2), ("relu",), ("fc", 8), ("softmax_ce",)])


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("cfg", [PARTCHUNK, FORKED], ids=["partchunk", "forked"])
def test_nothing_of_a_pass_reaches_the_next(cfg, dtype):
    """A pass over an image with infinities leaves NaN in every partial sum; the pass after it must give the bits of a new plan."""
    batch = 13
    params = wl.make_params(cfg["layers"], cfg["in_shape"], 3)
    images, labels = wl.make_batch(cfg["in_shape"], batch, 8, 4)
    broken = images.copy()
    broken[:, :, ::2] = np.inf
    out = []
    for first in (None, broken, images):
        g = GpuNet(cfg["layers"], cfg["in_shape"], batch, dtype)
        try:
            if first is not None:
                _, grads = g.fwd_bwd(params, first, labels, 11, 2, 1)
                assert np.isfinite(grads).all() == (first is images)
            out.append(g.fwd_bwd(params, images, labels, 11, 2, 1))
        finally:
            g.close()
    assert np.isfinite(out[0][1]).all()
    for loss, grads in out[1:]:
        assert loss == out[0][0] and grads.tobytes() == out[0][1].tobytes()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("c,h,w,batch", [(8, 5, 7, 1), (40, 9, 11, 3), (200, 13, 13, 7), (40, 31, 33, 40), (136, 41, 43, 60)])
def test_bias_gradient_shapes(c, h, w, batch, dtype):
    layers = [("conv", c, 1, 1, 0), ("relu",), ("maxpool", 3, 2), ("conv", c, 1, 1, 0), ("relu",), ("fc", 10), ("softmax_ce",)]
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case({"name": "bias", "in_shape": (3, h, w), "classes": 10, "layers": layers}, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "bias")
    finally:
        g.close()


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("c,w", [(1, 12), (2, 12), (3, 12), (4, 12), (3, 14), (3, 15), (8, 12), (9, 7)])
def test_image_staging_takes_any_width(c, w, dtype):
    """The images of a first convolution are staged four, two or one pixel at a time, by width; more than four channels in
    groups of 16 bytes.  A channel or a pixel out of place shows in that layer's filter gradient."""
    layers = [("conv", 8, 3, 2, 2), ("relu",), ("fc", 8), ("softmax_ce",)]
    cfg, batch = {"name": "staging", "in_shape": (c, 10, w), "classes": 8, "layers": layers}, 5
    g, onet, (loss, grads), (ref_loss, ref_grads, _), _ = _net_case(cfg, batch, dtype, plain=False)
    try:
        assert abs(loss - ref_loss) <= TOL[dtype] * abs(ref_loss)
        compare_grads(onet, grads, ref_grads, TOL[dtype], "staging")
    finally:
        g.close()


# RAGGED runs on the caller's stream alone either way; FORKED has a side stream for its weights, LONGSUM for the 3200 images that a
# few workgroups sum up in its last layer
LONGSUM = dict(name="longsum", in_shape=(3, 6, 6), classes=8, layers=[("conv", 8, 3, 1, 1), ("relu",), ("maxpool", 2, 2), ("fc", 8), ("softmax_ce",)])


@pytest.mark.parametrize("cfg,batch,dtype", [(RAGGED, 37, B.F32), (RAGGED, 37, B.BF16), (FORKED, 37, B.F32), (FORKED, 37, B.BF16), (LONGSUM, 3200, B.F32)],
                         ids=lambda v: v["name"] if isinstance(v, dict) else str(v))
def test_serial_plan_gives_the_same_bits(cfg, batch, dtype):
    """asgd_net_set_serial keeps every kernel on the caller's stream; the results must not change by a bit."""
    params = wl.make_params(cfg["layers"], cfg["in_shape"], 3)
    images, labels = wl.make_batch(cfg["in_shape"], batch, cfg["classes"], 4)
    out = []
    for serial in (False, True):
        g = GpuNet(cfg["layers"], cfg["in_shape"], batch, dtype)
        try:
            B.asgd_net_set_serial(g.net, serial)
            out.append(g.fwd_bwd(params, images, labels, 11, 2, 1))
        finally:
            g.close()
    assert out[0][0] == out[1][0] and out[0][1].tobytes() == out[1][1].tobytes()


def test_side_stream_gives_the_same_bits():
    """The same for a net with enough weights that the parameter gradients run on the side stream."""
    layers = [("conv", 96, 3, 1, 1), ("relu",), ("maxpool", 2, 2), ("fc", 1024), ("relu",), ("fc", 10), ("softmax_ce",)]
    shape = (3, 16, 16)
    params = wl.make_params(layers, shape, 3)
    assert params.size > 4 << 20
    images, labels = wl.make_batch(shape, 37, 10, 4)
    out = []
    for serial in (False, True):
        g = GpuNet(layers, shape, 37, B.BF16)
        try:
            B.asgd_net_set_serial(g.net, serial)
            out.append(g.fwd_bwd(params, images, labels, 11, 2, 1))
        finally:
            g.close()
    assert out[0][0] == out[1][0] and out[0][1].tobytes() == out[1][1].tobytes()
