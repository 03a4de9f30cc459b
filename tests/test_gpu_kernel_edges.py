"""Edges of the kernels' own tilings and dispatch rules, against the fp64 oracle: counts around powers of two and
multiples of the wave, channel counts that do not divide a workgroup, images of one pixel."""
import numpy as np
import pytest
import torch

import paper_1901_06887_amd as mt
import workloads as wl
from gpu_common import compare, gpu_run, make_context, oracle_rows
from paper_1901_06887_amd import torch_io

pytestmark = pytest.mark.gpu


def mlp_fleet(n_tenants, n_requests, dims, dtype="f32", act=wl.ACT_RELU, seed=301, ids=None):
    tenants = {t: wl.make_model(wl.mlp_layers(list(dims), act), dtype, seed, t) for t in range(n_tenants)}
    rng = np.random.default_rng(seed)
    ids = rng.integers(0, n_tenants, n_requests) if ids is None else ids
    x = rng.standard_normal((n_requests, dims[0])).astype(np.float32)
    return wl.Workload("mlp", dtype, tenants, ids.astype(np.int32), wl.round_to_bf16(x) if dtype == "bf16" else x)


def check(w, what, ctx=None):
    ctx = ctx or make_context(w)
    gpu = gpu_run(ctx, w, poison=True)
    assert np.array_equal(ctx.last_counts(), np.bincount(w.tenant_ids, minlength=ctx.cfg.max_tenants)), what
    print("%s: worst per-tensor rel fro %.2e" % (what, compare(w, gpu, oracle_rows(w), what=what)), flush=True)
    return gpu


# tenants: one lane each up to 64, tables in LDS beyond; rows: 1024 is one row per lane of every wave
@pytest.mark.parametrize("n_tenants", [1, 63, 64, 65, 300])
@pytest.mark.parametrize("n_requests", [1, 64, 1024, 1025, 4097])
def test_segmentation_at_the_edges_of_its_register_paths(n_tenants, n_requests):
    w = mlp_fleet(n_tenants, n_requests, (8, 12, 5), seed=310 + n_tenants)
    ctx = make_context(w)
    one = check(w, "%d tenants, %d requests" % (n_tenants, n_requests), ctx)
    # the same rows as several submissions: same bits
    x, ids = torch_io.to_device(w.inputs, w.dtype), torch.from_numpy(w.tenant_ids).cuda()
    out = torch_io.alloc_outputs(n_requests, ctx.cfg.max_classes)
    cuts = sorted({0, n_requests // 3, n_requests // 2, n_requests})
    for a, b in zip(cuts[:-1], cuts[1:]):
        ctx.submit_batch(ids.data_ptr() + 4 * a, x.data_ptr() + a * x.stride(0) * x.element_size(), b - a, x.shape[1])
    ctx.run(torch.cuda.current_stream().cuda_stream, out.labels.data_ptr(), out.probs.data_ptr(), out.logits.data_ptr(),
            out.n_classes.data_ptr(), n_requests, ctx.cfg.max_classes)
    torch.cuda.synchronize()
    assert np.array_equal(out.logits.cpu().numpy().astype(np.float64), one[0]) and np.array_equal(out.labels.cpu().numpy(), one[2])


# more than 256 tenants: a tile list takes several steps of 256; more than 512: the histograms leave room for eight or four ranking waves.
# Models of one to three linear layers, a convolution, or none, at tenant numbers around the steps; few and many rows, one submission and three
@pytest.mark.parametrize("n_tenants", [257, 513, 1023, 1025, 2048])
@pytest.mark.parametrize("n_requests", [200, 5003])
def test_tile_lists_of_many_tenants(n_tenants, n_requests):
    edges = [t + d for t in range(0, n_tenants + 1, 256) for d in (-1, 0, 1, 2, 3)]
    hosts = sorted({t for t in edges if 0 <= t < n_tenants} | {n_tenants - 1} | set(range(5, n_tenants, 37)))
    tenants = {}
    for i, t in enumerate(hosts):
        if i % 4 == 3:
            layers = [wl.LayerSpec(wl.CONV, wl.ACT_RELU, 3, 8, 4, 4, 1, ksize=3, pad=1), wl.LayerSpec(wl.GAP, wl.ACT_NONE, 8, 8, 4, 4), wl.LayerSpec(wl.FC, wl.ACT_NONE, 8, 6)]
        else:
            layers = wl.mlp_layers([48, 20, 100, 5][:1] + [[5], [20, 7], [20, 100, 5]][i % 4], wl.ACT_RELU)
        tenants[t] = wl.make_model(layers, "f32", 312, t)
    rng = np.random.default_rng(312)
    ids = rng.choice(hosts, n_requests).astype(np.int32)
    ids[:len(hosts)] = hosts[:n_requests]                          # every model has a request, as far as they go
    ids = rng.permutation(ids)
    w = wl.Workload("many", "f32", tenants, ids, rng.standard_normal((n_requests, 48)).astype(np.float32))
    ctx = make_context(w, max_tenants=n_tenants)
    one = check(w, "%d tenants, %d requests" % (n_tenants, n_requests), ctx)
    x, d_ids = torch_io.to_device(w.inputs, "f32"), torch.from_numpy(ids).cuda()
    out = torch_io.alloc_outputs(n_requests, ctx.cfg.max_classes)
    cuts = [0, n_requests // 3, n_requests // 2, n_requests]
    for a, b in zip(cuts[:-1], cuts[1:]):
        ctx.submit_batch(d_ids.data_ptr() + 4 * a, x.data_ptr() + a * 48 * 4, b - a, 48)
    ctx.debug_poison()
    ctx.run(torch.cuda.current_stream().cuda_stream, out.labels.data_ptr(), out.probs.data_ptr(), out.logits.data_ptr(),
            out.n_classes.data_ptr(), n_requests, ctx.cfg.max_classes)
    torch.cuda.synchronize()
    assert np.array_equal(out.logits.cpu().numpy().astype(np.float64), one[0]) and np.array_equal(out.labels.cpu().numpy(), one[2])


@pytest.mark.parametrize("n_tenants", [300, 2048])
def test_big_tile_lists_of_many_tenants(monkeypatch, n_tenants):
    """Big tiles of tenants in different steps of a list, beside tenants that are too small for them."""
    monkeypatch.setenv("MT_BIG_MIN_TILES", "1")
    hosts = [3, 255, 256, n_tenants // 2 + 130, n_tenants - 1]
    tenants = {t: wl.make_model(wl.mlp_layers([64, 256, 200, 7], wl.ACT_GELU), "bf16", 313, t) for t in hosts}
    rng = np.random.default_rng(313)
    ids = rng.permutation(np.repeat(hosts, [2048, 40, 2304 + 130, 4096 + 100, 2500])).astype(np.int32)
    x = wl.round_to_bf16(rng.standard_normal((len(ids), 64)).astype(np.float32))
    w = wl.Workload("many-big", "bf16", tenants, ids, x)
    ctx = make_context(w, max_tenants=n_tenants)
    check(w, "%d tenants" % n_tenants, ctx)


@pytest.mark.parametrize("hw,channels,dtype", [((1, 1), 8, "f32"), ((9, 13), 72, "f32"), ((9, 13), 72, "bf16"), ((5, 7), 8, "bf16"),
                                               ((3, 3), 520, "bf16"), ((2, 5), 2056, "f32")])
def test_average_pooling_of_any_channel_count(hw, channels, dtype):
    h, w_ = hw
    layers = [wl.LayerSpec(wl.CONV, wl.ACT_RELU, 3, channels, h, w_, 1, ksize=1, pad=0), wl.LayerSpec(wl.GAP, wl.ACT_NONE, channels, channels, h, w_),
              wl.LayerSpec(wl.FC, wl.ACT_NONE, channels, 7)]
    tenants = {t: wl.make_model(layers, dtype, 320, t) for t in range(2)}
    rng = np.random.default_rng(320)
    x = rng.standard_normal((37, layers[0].in_len())).astype(np.float32)
    w = wl.Workload("gap", dtype, tenants, rng.integers(0, 2, 37).astype(np.int32), wl.round_to_bf16(x) if dtype == "bf16" else x)
    check(w, "%dx%dx%d %s" % (h, w_, channels, dtype))


# launches whose tiles split K: every window and stride, reductions from one brick to many (4, 8 and 16 waves), channel blocks
# with 8 of 32 channels, pixel tiles with a single pixel; against the oracle, and against the launches that do not split K
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k,stride,ci,co,hw", [(1, 1, 8, 8, (1, 1)), (1, 2, 16, 40, (5, 7)), (3, 1, 8, 72, (11, 3)), (3, 2, 24, 32, (9, 6)), (3, 1, 64, 96, (4, 8)),
                                               (3, 1, 200, 128, (7, 7)), (7, 2, 8, 64, (17, 13)), (7, 1, 40, 8, (6, 6)),
                                               # taps of whole chunks, images narrower than the window among them
                                               (3, 1, 128, 64, (1, 1)), (3, 1, 192, 40, (5, 2)), (3, 2, 160, 96, (9, 6)), (7, 1, 32, 72, (3, 4)), (3, 1, 288, 32, (7, 11))])
def test_convolutions_that_split_their_reduction(monkeypatch, dtype, k, stride, ci, co, hw):
    h, w_ = hw
    first = wl.LayerSpec(wl.CONV, wl.ACT_RELU, 3, ci, h, w_, 1, ksize=3, pad=1)
    mid = wl.LayerSpec(wl.CONV, wl.ACT_GELU, ci, co, h, w_, stride, ksize=k, pad=(k - 1) // 2)
    oh, ow = mid.out_hw()
    skip = [wl.LayerSpec(wl.CONV, wl.ACT_NONE, co, co, oh, ow, 1, ksize=1, pad=0), wl.LayerSpec(wl.ADD, wl.ACT_RELU, co, co, oh, ow, src2=2)]
    layers = [first, mid, *skip, wl.LayerSpec(wl.GAP, wl.ACT_NONE, co, co, oh, ow), wl.LayerSpec(wl.FC, wl.ACT_NONE, co, 9)]
    tenants = {t: wl.make_model(layers, dtype, 330 + k, t) for t in range(3)}
    rng = np.random.default_rng(330)
    x = rng.standard_normal((13, first.in_len())).astype(np.float32)
    w = wl.Workload("split", dtype, tenants, rng.integers(0, 3, 13).astype(np.int32), wl.round_to_bf16(x) if dtype == "bf16" else x)
    got = {}
    for tiles in ("0", "100000"):
        monkeypatch.setenv("MT_CONV_SPLIT_TILES", tiles)
        got[tiles] = check(w, "%dx%d s%d %d->%d %s, split up to %s tiles" % (k, k, stride, ci, co, dtype, tiles))
    # both sum fp32 products in fp32, in another order: a row's error is rounding noise, or (bf16) one flipped activation
    err = np.linalg.norm(got["0"][0] - got["100000"][0], axis=1) / np.linalg.norm(got["0"][0], axis=1)
    assert err.max() <= (5e-6 if dtype == "f32" else 1e-2)


# one layer index whose convolutions differ in pixels, channel blocks and reduction, beside tenants without any; requests spread, all the
# model's with the most pixels, all the one's with the most channels, and none a convolution's; submitted by ids and tenant by tenant
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows", [3, 70, 400])
@pytest.mark.parametrize("share", [(0.3, 0.3, 0.3, 0.1), (1, 0, 0, 0), (0, 1, 0, 0), (0, 0, 0, 1)])
def test_unlike_convolutions_at_one_layer_index(dtype, rows, share):
    conv = lambda ci, co, h, s, k: wl.LayerSpec(wl.CONV, wl.ACT_RELU, ci, co, h, h, s, ksize=k, pad=(k - 1) // 2)  # noqa: E731
    tail = lambda c, h, n: [wl.LayerSpec(wl.GAP, wl.ACT_NONE, c, c, h, h), wl.LayerSpec(wl.FC, wl.ACT_NONE, c, n)]  # noqa: E731
    models = [[conv(3, 8, 12, 1, 3), conv(8, 8, 12, 1, 3), *tail(8, 12, 5)], [conv(3, 96, 12, 2, 3), conv(96, 160, 6, 2, 3), *tail(160, 3, 7)],
              [conv(3, 16, 12, 2, 7), conv(16, 40, 6, 1, 1), *tail(40, 6, 3)], wl.mlp_layers([432, 40, 9], wl.ACT_RELU)]
    tenants = {t: wl.make_model(m, dtype, 335, t) for t, m in enumerate(models)}
    rng = np.random.default_rng(335)
    x = rng.standard_normal((rows, 432)).astype(np.float32)
    ids = np.sort(rng.choice(4, rows, p=share)).astype(np.int32)
    w = wl.Workload("unlike", dtype, tenants, ids, wl.round_to_bf16(x) if dtype == "bf16" else x)
    ctx = make_context(w, max_tenants=70)
    what = "%s, %d rows, %s" % (dtype, rows, share)
    check(w, what, ctx)
    d_x, out = torch_io.to_device(w.inputs, dtype), torch_io.alloc_outputs(rows, ctx.cfg.max_classes)
    for t in np.unique(ids):
        first, n = int(np.argmax(ids == t)), int((ids == t).sum())
        for at, part in ((first, n // 2), (first + n // 2, n - n // 2)):
            if part:
                ctx.submit(int(t), d_x.data_ptr() + at * 432 * d_x.element_size(), part)
    ctx.debug_poison()
    ctx.run(torch.cuda.current_stream().cuda_stream, out.labels.data_ptr(), out.probs.data_ptr(), out.logits.data_ptr(),
            out.n_classes.data_ptr(), rows, ctx.cfg.max_classes)
    torch.cuda.synchronize()
    got = (out.logits.cpu().numpy().astype(np.float64), out.probs.cpu().numpy().astype(np.float64), out.labels.cpu().numpy(), out.n_classes.cpu().numpy())
    compare(w, got, oracle_rows(w), what=what + ", by tenant")


# frames whose K loop moves in groups of four k steps inside a tap (64 bf16 or 32 fp32 channels): one, two and more groups per tap,
# an odd number of them in all, one to four channel blocks, images that fill half of the pixel slots, and a tenant in the same launch
# whose taps are not whole groups
@pytest.mark.parametrize("hw", [(7, 7), (14, 14), (5, 9)])
@pytest.mark.parametrize("dtype,ci,co", [("bf16", 64, 32), ("bf16", 64, 136), ("bf16", 128, 64), ("bf16", 192, 128), ("bf16", 320, 96),
                                         ("f32", 32, 24), ("f32", 96, 64), ("f32", 64, 128)])
def test_frame_convolutions_in_groups_of_k_steps(monkeypatch, dtype, ci, co, hw):
    monkeypatch.setenv("MT_CONV_SPLIT_TILES", "0")
    h, w_ = hw
    tenants = {}
    for t, mid in enumerate((ci, ci, ci + 16)):
        layers = [wl.LayerSpec(wl.CONV, wl.ACT_RELU, 3, mid, h, w_, 1, ksize=3, pad=1), wl.LayerSpec(wl.CONV, wl.ACT_RELU, mid, co, h, w_, 1, ksize=3, pad=1),
                  wl.LayerSpec(wl.GAP, wl.ACT_NONE, co, co, h, w_), wl.LayerSpec(wl.FC, wl.ACT_NONE, co, 9)]
        tenants[t] = wl.make_model(layers, dtype, 340, t)
    rng = np.random.default_rng(340)
    x = rng.standard_normal((17, 3 * h * w_)).astype(np.float32)
    w = wl.Workload("frames", dtype, tenants, rng.integers(0, 3, 17).astype(np.int32), wl.round_to_bf16(x) if dtype == "bf16" else x)
    check(w, "%dx%d %d->%d %s" % (h, w_, ci, co, dtype))


# tiles whose waves split K finish on all their waves: one and two column blocks (64 hidden outputs), class counts at the edges of a
# block and of the two, row counts at the edges of a tile, output rows that do not take 16-byte stores
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("classes", [1, 3, 31, 32, 33, 64, 65])
@pytest.mark.parametrize("rows,hidden", [(1, 24), (33, 64), (95, 200)])
def test_tiles_that_split_k_finish_their_rows(dtype, classes, rows, hidden):
    w = mlp_fleet(2, rows, (48, hidden, 40, classes), dtype=dtype, act=wl.ACT_GELU, seed=350)
    check(w, "%d rows, %d hidden, %d classes, %s" % (rows, hidden, classes, dtype))


def test_head_of_a_split_k_tile_on_infinite_and_undefined_logits():
    """A class whose logit is +-infinity or NaN: the label is what a walk from the first class finds, as the other heads."""
    C, cases = 5, ([np.inf, 1, 2, 3, 4], [-np.inf] * 5, [0, np.nan, 1, -np.inf, 1], [np.nan, 1, 2, 3, 4])
    w = mlp_fleet(len(cases), len(cases), (16, C), seed=351, ids=np.arange(len(cases)))
    for t, row in enumerate(cases):
        w.tenants[t].biases[0][:] = np.array(row, np.float32)
        w.tenants[t].weights[0][:] = 0
    lg, pr, lb, nc = gpu_run(make_context(w), w)
    assert lb.tolist() == [0, 0, 2, 0]
    assert np.isnan(pr[:, :C]).all()
    for t, row in enumerate(cases):
        assert np.array_equal(lg[t, :C], np.array(row), equal_nan=True)


# one to two column blocks finished by tiles that split K, up to four by the wide tiles, then the head kernel with a row in registers and without
@pytest.mark.parametrize("classes,no_split_k", [(5, "0"), (40, "0"), (40, "1"), (100, "1"), (100, "0"), (300, "0"), (1030, "0")])
def test_heads_on_infinite_and_undefined_logits(monkeypatch, classes, no_split_k):
    """A class whose logit is +-infinity or NaN: the label is what a walk from the first class finds, whichever kernel finishes the row."""
    monkeypatch.setenv("MT_NO_AUTO_SPLIT_K", no_split_k)
    C, cases = 5, ([np.inf, 1, 2, 3, 4], [-np.inf] * 5, [0, np.nan, 1, -np.inf, 1], [np.nan, 1, 2, 3, 4], [np.nan] * 5)
    w = mlp_fleet(len(cases), len(cases), (16, classes), seed=351, ids=np.arange(len(cases)))
    for t, row in enumerate(cases):
        w.tenants[t].biases[0][:] = np.nan if np.isnan(row).all() else -np.inf
        w.tenants[t].biases[0][:C] = np.array(row, np.float32)
        w.tenants[t].weights[0][:] = 0
    lg, pr, lb, nc = gpu_run(make_context(w), w)
    assert lb.tolist() == [0, 0, 2, 0, 0]
    assert np.isnan(pr[:, :C]).all()
    for t, row in enumerate(cases):
        assert np.array_equal(lg[t, :C], np.array(row), equal_nan=True)


# Padding columns of a hidden layer's activation stay zero whatever a row holds: 0 x Inf in a padding output would be NaN, and meet the
# zero-padded K of the next layer.  Linear hidden layers (one and two column blocks, a wider one with a ragged last block), in runs that split
# K, that do not, and that take big tiles; y = W x over the K real inputs: a row with an infinite input has infinite logits, not NaN.
def infinite_rows(dtype, dims, rows, hot):
    w = mlp_fleet(1, rows, dims, dtype=dtype, act=wl.ACT_NONE, seed=352)
    m = w.tenants[0]
    for layer in range(len(dims) - 2):
        m.weights[layer][:] = 1
    m.weights[-1][:] = np.array([-1, 2, 3], np.float32)[:, None]
    for b in m.biases:
        b[:] = 0
    w.inputs[:] = 1
    w.inputs[hot, 5] = np.inf
    return w


def check_infinite_rows(w, hot):
    lg, _, lb, _ = gpu_run(make_context(w), w, poison=True)
    cold = np.setdiff1d(np.arange(w.n_requests), hot)
    assert np.array_equal(lg[hot, :3], np.tile([-np.inf, np.inf, np.inf], (len(hot), 1))) and (lb[hot] == 1).all()
    assert np.isfinite(lg[cold]).all() and (lb[cold] == 2).all()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hidden", [(1,), (40,), (100,), (100, 7, 200)])
@pytest.mark.parametrize("no_split_k", ["0", "1"])
def test_infinite_inputs_leave_padding_columns_at_zero(monkeypatch, dtype, hidden, no_split_k):
    monkeypatch.setenv("MT_NO_AUTO_SPLIT_K", no_split_k)
    hot = np.array([0, 2, 34])
    check_infinite_rows(infinite_rows(dtype, (16, *hidden, 3), 37, hot), hot)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k", [64, 256])                       # a workgroup per big tile, one workgroup per CU walking them
def test_infinite_inputs_leave_padding_columns_of_big_tiles_at_zero(monkeypatch, dtype, k):
    monkeypatch.setenv("MT_BIG_MIN_TILES", "1")
    hot = np.array([0, 255, 256, 8191])
    check_infinite_rows(infinite_rows(dtype, (k, 200, 3), 8192, hot), hot)


def test_average_pooling_of_many_rows():
    """Launches of 1024 and more packed rows pool with smaller workgroups: odd channel counts, more chunks than threads."""
    for channels, dtype in ((72, "f32"), (8, "bf16"), (520, "f32")):
        layers = [wl.LayerSpec(wl.CONV, wl.ACT_RELU, 3, channels, 3, 5, 1, ksize=1, pad=0), wl.LayerSpec(wl.GAP, wl.ACT_NONE, channels, channels, 3, 5),
                  wl.LayerSpec(wl.FC, wl.ACT_NONE, channels, 7)]
        tenants = {t: wl.make_model(layers, dtype, 360, t) for t in range(2)}
        rng = np.random.default_rng(360)
        x = rng.standard_normal((1030, layers[0].in_len())).astype(np.float32)
        w = wl.Workload("gap", dtype, tenants, rng.integers(0, 2, 1030).astype(np.int32), wl.round_to_bf16(x) if dtype == "bf16" else x)
        check(w, "1030 rows of %d channels, %s" % (channels, dtype))


# pixels per thread around the eight loads in flight (one group of pixels, two, several rounds of them), an infinite value in the last
# pixel (taps past it are loaded and must not count), and many rows of many chunks
@pytest.mark.parametrize("rows,hw,channels,dtype", [(33, (1, 8), 8, "bf16"), (33, (3, 3), 16, "f32"), (7, (5, 13), 8, "bf16"), (5, (23, 23), 24, "f32"), (3, (27, 41), 8, "bf16"),
                                                    (1030, (16, 16), 72, "f32")])
def test_average_pooling_around_its_loads_in_flight(rows, hw, channels, dtype):
    h, w_ = hw
    layers = [wl.LayerSpec(wl.CONV, wl.ACT_RELU, 3, channels, h, w_, 1, ksize=1, pad=0), wl.LayerSpec(wl.GAP, wl.ACT_NONE, channels, channels, h, w_),
              wl.LayerSpec(wl.FC, wl.ACT_NONE, channels, 7)]
    w = wl.Workload("gap", dtype, {0: wl.make_model(layers, dtype, 361, 0)}, np.zeros(rows, np.int32), None)
    x = np.random.default_rng(361).standard_normal((rows, layers[0].in_len())).astype(np.float32)
    w.inputs = wl.round_to_bf16(x) if dtype == "bf16" else x
    check(w, "%d rows of %dx%dx%d, %s" % (rows, h, w_, channels, dtype))
    w.tenants[0].weights[0][:] = 1
    w.tenants[0].weights[2][:] = 1
    w.inputs[-1, -1] = np.inf
    lg = gpu_run(make_context(w), w)[0][:, :7]
    assert (lg[-1] == np.inf).all() and np.isfinite(lg[:-1]).all()


def test_convolution_outputs_on_both_sides_of_the_line_for_stores_through_l2():
    """44 images of 112x112x64 in bf16 are 70 MB, stored the ordinary way, 22 of them 35 MB, stored through L2: the same bits; some rows
    against the oracle."""
    layers = [wl.LayerSpec(wl.CONV, wl.ACT_RELU, 3, 64, 112, 112, 1, ksize=3, pad=1), wl.LayerSpec(wl.CONV, wl.ACT_RELU, 64, 64, 112, 112, 1, ksize=3, pad=1),
              wl.LayerSpec(wl.CONV, wl.ACT_NONE, 64, 64, 112, 112, 1, ksize=1, pad=0), wl.LayerSpec(wl.GAP, wl.ACT_NONE, 64, 64, 112, 112), wl.LayerSpec(wl.FC, wl.ACT_NONE, 64, 7)]
    x = wl.round_to_bf16(np.random.default_rng(362).standard_normal((44, layers[0].in_len())).astype(np.float32))
    w = wl.Workload("through", "bf16", {0: wl.make_model(layers, "bf16", 362, 0)}, np.zeros(44, np.int32), x)
    ctx = make_context(w)
    whole = gpu_run(ctx, w, poison=True)
    for a, b in ((0, 22), (22, 44)):
        part = gpu_run(ctx, w, ids=w.tenant_ids[a:b], inputs=w.inputs[a:b], poison=True)
        assert all(np.array_equal(p, q[a:b]) for p, q in zip(part, whole))
    rows = np.array([0, 21, 43])
    compare(w, tuple(v[rows] for v in whole), oracle_rows(w, rows), rows=rows, what="through", deep=True)


def first_conv_workload(dtype, rows, hw, ci, convs, pool=None, act=wl.ACT_RELU, seed=370):
    """Models that start with a convolution (k, stride, channels) of the same images, a max-pool (k, stride, pad) behind it or not, and a
    convolution behind that to which places matter."""
    tenants = {}
    for t, (k, stride, co) in enumerate(convs):
        h, w_ = hw
        layers = [wl.LayerSpec(wl.CONV, act, ci, co, h, w_, stride, ksize=k, pad=(k - 1) // 2)]
        h, w_ = layers[-1].out_hw()
        if pool:
            layers.append(wl.LayerSpec(wl.MAXPOOL, wl.ACT_NONE, co, co, h, w_, pool[1], ksize=pool[0], pad=pool[2]))
            h, w_ = layers[-1].out_hw()
        layers.append(wl.LayerSpec(wl.CONV, wl.ACT_RELU, co, 16, h, w_, 2, ksize=3, pad=1))
        h, w_ = layers[-1].out_hw()
        layers += [wl.LayerSpec(wl.GAP, wl.ACT_NONE, 16, 16, h, w_), wl.LayerSpec(wl.FC, wl.ACT_NONE, 16, 7)]
        tenants[t] = wl.make_model(layers, dtype, seed, t)
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((rows, ci * hw[0] * hw[1])).astype(np.float32)
    return wl.Workload("first", dtype, tenants, rng.integers(0, len(convs), rows).astype(np.int32), wl.round_to_bf16(x) if dtype == "bf16" else x)


# first convolutions on the submitted images: one to four channels, every window and stride (several in a launch), images of a pixel and
# of rows that are not whole groups of pixels, one to five channel blocks, every pool, tiles of one row, of a few and of whatever fits
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hw,ci,convs,pool,rows", [
    ((1, 1), 3, [(3, 1, 8)], None, 9), ((1, 3), 3, [(7, 2, 40), (1, 1, 8)], None, 1), ((5, 7), 1, [(3, 1, 72), (1, 2, 16)], None, 2), ((9, 6), 2, [(7, 1, 24)], None, 9),
    ((11, 13), 4, [(3, 2, 32), (7, 1, 136)], None, 4), ((40, 66), 3, [(3, 1, 40), (3, 1, 96)], None, 99), ((70, 33), 3, [(3, 2, 8), (1, 1, 64), (7, 2, 32)], None, 3),
    ((2, 2), 3, [(3, 1, 8)], (2, 2, 0), 1), ((8, 8), 3, [(7, 2, 32), (3, 1, 160)], (3, 2, 1), 9), ((13, 10), 1, [(3, 1, 72)], (2, 1, 1), 5), ((15, 22), 4, [(3, 2, 24), (1, 1, 64)], (3, 1, 1), 99),
    ((90, 61), 3, [(7, 2, 64), (3, 1, 40)], (3, 2, 1), 5), ((64, 150), 3, [(3, 1, 64)], (3, 2, 0), 99), ((33, 120), 2, [(3, 1, 96)], (2, 2, 1), 1), ((61, 57), 3, [(7, 1, 128)], (3, 1, 0), 7)])
def test_first_convolutions_on_the_submitted_images(monkeypatch, dtype, hw, ci, convs, pool, rows):
    monkeypatch.setenv("MT_FIRST_ROWS", str(rows))
    monkeypatch.setenv("MT_CONV_SPLIT_TILES", "0")
    w = first_conv_workload(dtype, 11, hw, ci, convs, pool, act={1: wl.ACT_GELU, 2: wl.ACT_NONE}.get(ci, wl.ACT_RELU))
    what = "%s %s x%d %s %s tiles of %d rows" % (dtype, hw, ci, convs, pool, rows)
    print(what, flush=True)
    ctx = make_context(w)
    one = check(w, what, ctx)
    # rows that start and lie at odd addresses: the same bits
    n_in, es = w.inputs.shape[1], 2 if dtype == "bf16" else 4
    x = torch_io.to_device(np.concatenate([w.inputs, np.zeros((11, 1), np.float32)], axis=1), dtype).reshape(-1)
    flat = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")
    flat[1:] = x
    ids, out = torch.from_numpy(w.tenant_ids).cuda(), torch_io.alloc_outputs(11, ctx.cfg.max_classes)
    ctx.submit_batch(ids.data_ptr(), flat.data_ptr() + es, 11, n_in + 1)
    ctx.run(torch.cuda.current_stream().cuda_stream, out.labels.data_ptr(), out.probs.data_ptr(), out.logits.data_ptr(), out.n_classes.data_ptr(), 11, ctx.cfg.max_classes)
    torch.cuda.synchronize()
    assert np.array_equal(out.logits.cpu().numpy().astype(np.float64), one[0])
    ctx.close()
    # staged images and a max-pool of its own: the same bits in bf16, the same products in another order in fp32
    monkeypatch.setenv("MT_NO_CONV_FIRST", "1")
    ctx = make_context(w)
    staged = gpu_run(ctx, w, poison=True)
    if dtype == "bf16":
        assert np.array_equal(staged[0], one[0])
    else:
        assert np.linalg.norm(staged[0] - one[0]) <= 5e-6 * np.linalg.norm(one[0])
    ctx.close()


# a first convolution and the 3x3 convolution behind it in one launch: one to four blocks of second channels, both strides of both, images of a pixel, of
# several tiles and of rows that fill a tile badly; beside models that do not take it (too many channels, a large window, a max-pool), which leaves both layers a launch
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hw,models,rows", [
    ((1, 1), [(3, 1, 16, 1, 8)], 9), ((2, 9), [(1, 1, 32, 2, 40), (3, 2, 48, 1, 128)], 9), ((16, 16), [(3, 1, 32, 2, 64), (3, 1, 64, 1, 96), (3, 1, 16, 1, 128)], 3),
    ((35, 29), [(3, 1, 48, 1, 40), (3, 2, 64, 2, 32)], 99), ((21, 100), [(3, 1, 16, 1, 16), (1, 2, 16, 1, 8)], 1), ((9, 11), [(3, 1, 32, 1, 40), (3, 1, 16, 1, 136), (7, 2, 16, 1, 8)], 9), ((33, 130), [(3, 1, 16, 2, 72)], 99)])
def test_first_convolutions_with_the_ones_behind_them(monkeypatch, dtype, hw, models, rows):
    monkeypatch.setenv("MT_FIRST_ROWS", str(rows))
    monkeypatch.setenv("MT_CONV_SPLIT_TILES", "0")
    tenants = {}
    for t, (k, s0, c0, s1, c1) in enumerate(models):
        layers = [wl.LayerSpec(wl.CONV, wl.ACT_GELU if t else wl.ACT_RELU, 3, c0, *hw, s0, ksize=k, pad=(k - 1) // 2)]
        layers.append(wl.LayerSpec(wl.CONV, wl.ACT_RELU, c0, c1, *layers[-1].out_hw(), s1, ksize=3, pad=1))
        layers.append(wl.LayerSpec(wl.CONV, wl.ACT_RELU, c1, 8, *layers[-1].out_hw(), 2, ksize=3, pad=1))
        layers += [wl.LayerSpec(wl.GAP, wl.ACT_NONE, 8, 8, *layers[-1].out_hw()), wl.LayerSpec(wl.FC, wl.ACT_NONE, 8, 5)]
        tenants[t] = wl.make_model(layers, dtype, 372, t)
    h, w_ = (hw[0] - 1) // 2 + 1, (hw[1] - 1) // 2 + 1
    tenants[len(models)] = wl.make_model([wl.LayerSpec(wl.CONV, wl.ACT_RELU, 3, 16, *hw, 1, ksize=3, pad=1), wl.LayerSpec(wl.MAXPOOL, wl.ACT_NONE, 16, 16, *hw, 2, ksize=3, pad=1),
                                          wl.LayerSpec(wl.CONV, wl.ACT_RELU, 16, 8, h, w_, 1, ksize=3, pad=1), wl.LayerSpec(wl.GAP, wl.ACT_NONE, 8, 8, h, w_),
                                          wl.LayerSpec(wl.FC, wl.ACT_NONE, 8, 5)], dtype, 372, 9)
    x = np.random.default_rng(372).standard_normal((23, 3 * hw[0] * hw[1])).astype(np.float32)
    ids = np.random.default_rng(373).integers(0, len(tenants), 23).astype(np.int32)
    for apart in (True, False):                                      # with and without the model that is served apart
        if not apart:
            del tenants[len(models)]
        ids_ = ids if apart else ids % len(models)
        w = wl.Workload("pair", dtype, tenants, ids_, wl.round_to_bf16(x) if dtype == "bf16" else x)
        what = "%s %s %s tiles of %d rows" % (dtype, hw, models, rows)
        print(what, flush=True)
        ctx = make_context(w)
        one, launches = check(w, what, ctx), ctx.stats()["last_run_launches"]
        ctx.close()
        monkeypatch.setenv("MT_NO_CONV_PAIR", "1")                   # two launches: the same bits in both types
        ctx = make_context(w)
        got = gpu_run(ctx, w, poison=True)
        monkeypatch.delenv("MT_NO_CONV_PAIR")
        assert np.array_equal(got[0], one[0]), what
        takes = not apart and all(k <= 3 and c1 <= 128 for k, _, _, _, c1 in models)
        assert ctx.stats()["last_run_launches"] == launches + takes, what
        ctx.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k,stride,pool", [(1, 1, None), (3, 1, None), (7, 2, None), (3, 1, (3, 2, 1))])
def test_infinite_pixels_stay_inside_their_windows(dtype, k, stride, pool):
    """Linear layers of ones over an image with one infinite pixel: the mean over the outputs is infinite if some window holds the pixel, and never NaN."""
    h, w_ = 12, 14
    layers = [wl.LayerSpec(wl.CONV, wl.ACT_NONE, 3, 8, h, w_, stride, ksize=k, pad=(k - 1) // 2)]
    h, w_ = layers[-1].out_hw()
    if pool:
        layers.append(wl.LayerSpec(wl.MAXPOOL, wl.ACT_NONE, 8, 8, h, w_, pool[1], ksize=pool[0], pad=pool[2]))
        h, w_ = layers[-1].out_hw()
    layers += [wl.LayerSpec(wl.GAP, wl.ACT_NONE, 8, 8, h, w_), wl.LayerSpec(wl.FC, wl.ACT_NONE, 8, 3)]
    m = wl.make_model(layers, dtype, 371, 0)
    for l, s in enumerate(layers):
        if s.kind in (wl.CONV, wl.FC):
            m.weights[l][:] = 1
            m.biases[l][:] = 0
    x = np.ones((12 * 14 + 1, 12 * 14 * 3), np.float32)
    x[np.arange(12 * 14), np.arange(12 * 14) * 3 + 1] = -np.inf      # request p: pixel p; the last one: none
    w = wl.Workload("inf", dtype, {0: m}, np.zeros(len(x), np.int32), x)
    lg = gpu_run(make_context(w), w, poison=True)[0][:, :3]
    assert np.isfinite(lg[-1]).all() and not np.isnan(lg).any()
    ch, cw = layers[0].out_hw()
    for p, row in enumerate(lg[:-1]):
        y, xx = divmod(p, 14)
        holds = np.outer(np.abs(np.arange(ch) * stride - y) <= k // 2, np.abs(np.arange(cw) * stride - xx) <= k // 2)      # convolution outputs whose window holds the pixel
        if pool:                                                     # a maximum is infinite where all of its window is
            cut = lambda v, o: v[max(o * pool[1] - pool[2], 0):o * pool[1] - pool[2] + pool[0]]  # noqa: E731
            holds = np.array([[cut(cut(holds, oy).T, ox).all() for ox in range(w_)] for oy in range(h)])
        assert np.array_equal(row, np.full(3, -np.inf)) == holds.any() and np.isinf(row).all() == holds.any(), p


def test_first_convolutions_with_infinite_filters(monkeypatch):
    """Filters that are not finite take the staged path: the same bits, undefined and infinite logits among them."""
    w = first_conv_workload("bf16", 7, (9, 10), 3, [(3, 1, 16), (7, 2, 40)], (3, 2, 1))
    w.tenants[0].weights[0][3, 1, 0, 2] = np.inf
    monkeypatch.setenv("MT_FIRST_ROWS", "9")                         # (images as small as these are staged otherwise)
    got = []
    for off in ("0", "1"):
        monkeypatch.setenv("MT_NO_CONV_FIRST", off)
        got.append(gpu_run(make_context(w), w, poison=True)[0])
    assert np.array_equal(got[0], got[1], equal_nan=True) and np.isfinite(got[0][w.tenant_ids == 1]).all() and not np.isfinite(got[0][w.tenant_ids == 0]).all()


# runs whose first launch does the batcher's work: rows at the edges of a wave's 64 and of what it takes, one tenant and all 64, models of two to four
# layers and of few and many classes, rows of unknown tenants and of tenants without a model; the same bits and counts as with the batcher
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_tenants", [1, 9, 64])
@pytest.mark.parametrize("rows", [1, 33, 64, 65, 200, 256, 257])
def test_small_runs_without_a_batcher(monkeypatch, dtype, n_tenants, rows):
    shapes = ([48, 24, 5], [48, 64, 40, 130], [48, 200, 33, 7, 64])
    tenants = {t: wl.make_model(wl.mlp_layers(shapes[t % 3], wl.ACT_RELU), dtype, 380, t) for t in range(n_tenants) if t != 7}
    rng = np.random.default_rng(380)
    x = rng.standard_normal((rows, 48)).astype(np.float32)
    ids = rng.integers(0, n_tenants, rows).astype(np.int32)
    ids[ids == 7] = 3
    w = wl.Workload("entry", dtype, tenants, ids, wl.round_to_bf16(x) if dtype == "bf16" else x)
    odd = ids.copy()
    odd[rng.random(rows) < 0.2] = rng.choice([-1, n_tenants, 1 << 30, min(7, n_tenants)])
    got = {}
    for off in ("0", "1"):
        monkeypatch.setenv("MT_NO_ENTRY", off)
        ctx = make_context(w, max_tenants=n_tenants)
        got[off] = [check(w, "%s, %d tenants, %d rows" % (dtype, n_tenants, rows), ctx) if off == "0" else gpu_run(ctx, w, poison=True)]
        launches = ctx.stats()["last_run_launches"]
        got[off].append(gpu_run(ctx, w, ids=odd, poison=True))
        got[off].append((ctx.last_counts(), [ctx.tenant_account(t)["requests"] for t in tenants]))
        one = torch_io.to_device(w.inputs, dtype)                    # all of them one tenant's, named by the submission
        out = torch_io.alloc_outputs(rows, ctx.cfg.max_classes)
        ctx.submit(0, one.data_ptr(), rows)
        ctx.run(torch.cuda.current_stream().cuda_stream, out.labels.data_ptr(), out.probs.data_ptr(), out.logits.data_ptr(), out.n_classes.data_ptr(), rows, ctx.cfg.max_classes)
        torch.cuda.synchronize()
        got[off].append((out.logits.cpu().numpy(), out.labels.cpu().numpy(), ctx.last_counts()))
        got[off + "n"] = launches
        ctx.close()
    for a, b in zip(got["0"], got["1"]):
        assert all(np.array_equal(u, v) for u, v in zip(a, b))
    assert got["0n"] == got["1n"] - (rows <= 256 and (n_tenants < 64 or rows <= 64))      # (64 tenants and more rows: ordinary tiles)


# the lists of first convolutions, alone and with the ones behind them: more tenants than a wave has lanes, several steps of a list, and batches that are
# ranked by a kernel of their own; models of one and of two tiles a request, MLPs between them
@pytest.mark.parametrize("n_tenants,rows", [(65, 300), (300, 900), (1025, 1500), (5, 8300), (300, 8300)])
@pytest.mark.parametrize("pair", [True, False])
def test_lists_of_first_convolutions_of_many_tenants_and_requests(monkeypatch, n_tenants, rows, pair):
    monkeypatch.setenv("MT_FIRST_ROWS", "5")
    monkeypatch.setenv("MT_CONV_SPLIT_TILES", "0")                   # (another order of the sums)
    tenants = {}
    for t in range(n_tenants):
        if t % 5 == 2:
            layers = wl.mlp_layers([192, 32, 6], wl.ACT_RELU)
        else:
            layers = [wl.LayerSpec(wl.CONV, wl.ACT_RELU, 3, 16, 8, 8, 1 + t % 2, ksize=3, pad=1)]
            layers.append(wl.LayerSpec(wl.CONV, wl.ACT_RELU, 16, 8, *layers[0].out_hw(), 1, ksize=3 if pair else 1, pad=int(pair)))
            layers.append(wl.LayerSpec(wl.CONV, wl.ACT_RELU, 8, 8, *layers[1].out_hw(), 2, ksize=3, pad=1))
            layers += [wl.LayerSpec(wl.GAP, wl.ACT_NONE, 8, 8, *layers[2].out_hw()), wl.LayerSpec(wl.FC, wl.ACT_NONE, 8, 6)]
        tenants[t] = wl.make_model(layers, "bf16", 390, t)
    rng = np.random.default_rng(390)
    w = wl.Workload("lists", "bf16", tenants, rng.integers(0, n_tenants, rows).astype(np.int32), wl.round_to_bf16(rng.standard_normal((rows, 192)).astype(np.float32)))
    got, launches = {}, {}
    for off in ("", "MT_NO_CONV_PAIR", "MT_NO_CONV_FIRST"):
        if off:
            monkeypatch.setenv(off, "1")
        ctx = make_context(w)
        got[off], launches[off] = gpu_run(ctx, w, poison=True), ctx.stats()["last_run_launches"]
        assert np.array_equal(ctx.last_counts(), np.bincount(w.tenant_ids, minlength=n_tenants))
        ctx.close()
    assert launches["MT_NO_CONV_PAIR"] == launches[""] + pair and launches["MT_NO_CONV_FIRST"] == launches["MT_NO_CONV_PAIR"] + 1
    for off in ("MT_NO_CONV_PAIR", "MT_NO_CONV_FIRST"):
        assert all(np.array_equal(a, b) for a, b in zip(got[""], got[off])), off
    pick = np.sort(rng.choice(rows, 250, replace=False))
    compare(w, tuple(v[pick] for v in got[""]), oracle_rows(w, pick), rows=pick, what="lists")


# a tile finds its tenant's facts in LDS with up to 32 or 64 tenants, by loads of its own beyond: the first, the last and a middle one of them, few requests
# (tiles that split K) and many, against the oracle and, to the bit, against a context of so many tenants that every kernel takes the other way
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_tenants", [3, 32, 33, 64, 65])
@pytest.mark.parametrize("rows", [5, 300])
def test_facts_of_few_and_many_tenants(dtype, n_tenants, rows):
    hosts = [0, n_tenants // 2, n_tenants - 1]
    layers = [wl.resnet18_layers(hw=24, widths=(16, 32, 64, 72), classes=10), wl.cnn_layers(hw=24, chans=(3, 32, 64, 128), strides=(1, 1, 2)),
              wl.mlp_layers([24 * 24 * 3, 200, 72, 7], wl.ACT_RELU)]
    models = [wl.make_model(m, dtype, 380, i) for i, m in enumerate(layers)]
    rng = np.random.default_rng(380)
    x = rng.standard_normal((rows, 24 * 24 * 3)).astype(np.float32)
    at = rng.integers(0, 3, rows)
    at[:3] = [0, 1, 2]
    gpu = []
    for ids, n in ((hosts, n_tenants), ([5, 100, 299], 300)):
        w = wl.Workload("facts", dtype, {t: models[i] for i, t in enumerate(ids)}, np.asarray(ids, np.int32)[at], wl.round_to_bf16(x) if dtype == "bf16" else x)
        ctx = make_context(w, max_tenants=n)
        gpu.append(gpu_run(ctx, w, poison=True))
    compare(w, gpu[1], oracle_rows(w), what="%d tenants, %d rows" % (n_tenants, rows), deep=dtype == "bf16")
    assert all(np.array_equal(a, b) for a, b in zip(*gpu))


# layer 0 does the batcher's work in runs of any tiles: rows at the edges of a wave's share and of the range, one tenant to a full wave of them, tiles of one to four
# column blocks and rows that fill none; requests of nobody.  Against the oracle, and to the bit against the batcher's launch
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_tenants", [1, 9, 64])
@pytest.mark.parametrize("rows", [320, 513, 1024, 4095, 4096, 4097])
def test_runs_of_any_tiles_without_a_batcher(monkeypatch, dtype, n_tenants, rows):
    shapes = ([48, 24, 5], [48, 64, 40, 130], [48, 200, 33, 7, 64])
    tenants = {t: wl.make_model(wl.mlp_layers(shapes[t % 3], wl.ACT_RELU), dtype, 395, t) for t in range(n_tenants) if t != 7}
    rng = np.random.default_rng(395)
    x = rng.standard_normal((rows, 48)).astype(np.float32)
    ids = np.minimum(rng.zipf(1.3, rows) - 1, n_tenants - 1).astype(np.int32)
    ids[ids == 7] = 3
    w = wl.Workload("entry", dtype, tenants, ids, wl.round_to_bf16(x) if dtype == "bf16" else x)
    odd = ids.copy()
    odd[rng.random(rows) < 0.2] = rng.choice([-1, n_tenants, 255, 1 << 30, min(7, n_tenants)])
    got = {}
    for off in ("0", "1"):
        monkeypatch.setenv("MT_NO_ENTRY", off)
        ctx = make_context(w, max_tenants=n_tenants)
        got[off] = [check(w, "%s, %d tenants, %d rows" % (dtype, n_tenants, rows), ctx) if off == "0" else gpu_run(ctx, w, poison=True)]
        launches = ctx.stats()["last_run_launches"]
        got[off].append(gpu_run(ctx, w, ids=odd, poison=True))
        got[off].append((ctx.last_counts(), [ctx.tenant_account(t)["requests"] for t in tenants]))
        one = torch_io.to_device(w.inputs, dtype)                    # all of them one tenant's, named by the submission
        out = torch_io.alloc_outputs(rows, ctx.cfg.max_classes)
        ctx.submit(0, one.data_ptr(), rows)
        ctx.run(torch.cuda.current_stream().cuda_stream, out.labels.data_ptr(), out.probs.data_ptr(), out.logits.data_ptr(), out.n_classes.data_ptr(), rows, ctx.cfg.max_classes)
        torch.cuda.synchronize()
        got[off].append((out.logits.cpu().numpy(), out.labels.cpu().numpy(), ctx.last_counts()))
        got[off + "n"] = launches
        ctx.close()
    for a, b in zip(got["0"], got["1"]):
        assert all(np.array_equal(u, v) for u, v in zip(a, b))
    assert got["0n"] == got["1n"] - (rows <= 4096)


# layer 0 reads rows of any length at any address: lengths around whole chunks and steps, rows that begin at odd elements with undefined values behind each, in tiles that split K (few
# rows and many without the batcher) and of four column blocks (more tenants than it takes, a row or two each), several submissions.  Against the oracle, and to the bit against staged rows
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_in", [1, 3, 7, 8, 9, 31, 63, 64, 65, 301])
@pytest.mark.parametrize("rows,n_tenants", [(19, 3), (700, 3), (90, 70)])
def test_rows_of_any_length_at_any_address(monkeypatch, dtype, n_in, rows, n_tenants):
    shapes = ([n_in, 40, 5], [n_in, 200, 70], [n_in, 300, 64, 7])
    tenants = {t: wl.make_model(wl.mlp_layers(shapes[t % 3], wl.ACT_RELU), dtype, 396, t) for t in range(n_tenants)}
    rng = np.random.default_rng(396)
    x = rng.standard_normal((rows, n_in)).astype(np.float32)
    ids = rng.integers(0, n_tenants, rows).astype(np.int32)
    w = wl.Workload("any", dtype, tenants, ids, wl.round_to_bf16(x) if dtype == "bf16" else x)
    stride = n_in + 4 + n_in % 2                                     # even: every row begins at an odd element
    buf = np.full(rows * stride + 1, np.nan, np.float32)
    for r in range(rows):
        buf[1 + r * stride:1 + r * stride + n_in] = w.inputs[r]
    d_buf, d_ids = torch_io.to_device(buf[None], dtype), torch.from_numpy(ids).cuda()
    at, es = d_buf.data_ptr() + d_buf.element_size(), d_buf.element_size()
    got = {}
    for off in ("0", "1"):
        monkeypatch.setenv("MT_NO_FUSED_GATHER", off)
        ctx = make_context(w, max_tenants=n_tenants)
        got[off] = [check(w, "%s %d x %d" % (dtype, rows, n_in), ctx)]
        for cuts in ([0, rows], [0, rows // 3, rows // 2, rows]):
            out = torch_io.alloc_outputs(rows, ctx.cfg.max_classes)
            for a, b in zip(cuts[:-1], cuts[1:]):
                ctx.submit_batch(d_ids.data_ptr() + 4 * a, at + a * stride * es, b - a, stride)
            ctx.debug_poison()
            ctx.run(torch.cuda.current_stream().cuda_stream, out.labels.data_ptr(), out.probs.data_ptr(), out.logits.data_ptr(), out.n_classes.data_ptr(), rows, ctx.cfg.max_classes)
            torch.cuda.synchronize()
            got[off].append((out.logits.cpu().numpy().astype(np.float64), out.probs.cpu().numpy().astype(np.float64), out.labels.cpu().numpy(), out.n_classes.cpu().numpy()))
            assert all(np.array_equal(u, v) for u, v in zip(got[off][0], got[off][-1]))
        ctx.close()
    assert all(np.array_equal(u, v) for u, v in zip(got["0"][0], got["1"][0]))


# the same in tiles of four column blocks and two row blocks, whose second one is full, ragged or missing, at odd strides (rows begin at odd and even elements by turns): without the
# batcher, behind it, and in several submissions.  Against the oracle, and to the bit against staged rows
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_in", [1, 3, 7, 8, 9, 31, 63, 64, 65, 301])
@pytest.mark.parametrize("counts", [(33, 64, 255), (95, 32, 401)])
def test_wide_tiles_read_rows_of_any_length_at_any_address(monkeypatch, dtype, n_in, counts):
    monkeypatch.setenv("MT_NO_AUTO_SPLIT_K", "1")
    rows = sum(counts)
    shapes = ([n_in, 130, 5], [n_in, 200, 70], [n_in, 300, 64, 7])
    tenants = {t: wl.make_model(wl.mlp_layers(shapes[t], wl.ACT_RELU), dtype, 398, t) for t in range(3)}
    rng = np.random.default_rng(398)
    x = rng.standard_normal((rows, n_in)).astype(np.float32)
    ids = rng.permutation(np.repeat(np.arange(3), counts)).astype(np.int32)
    w = wl.Workload("wide any", dtype, tenants, ids, wl.round_to_bf16(x) if dtype == "bf16" else x)
    stride = n_in + 4 + (n_in + 1) % 2
    assert stride % 2
    buf = np.full(rows * stride + 1, np.nan, np.float32)
    for r in range(rows):
        buf[1 + r * stride:1 + r * stride + n_in] = w.inputs[r]
    d_buf, d_ids = torch_io.to_device(buf[None], dtype), torch.from_numpy(ids).cuda()
    at, es = d_buf.data_ptr() + d_buf.element_size(), d_buf.element_size()
    got, launches = {}, {}
    for entry, gather in (("0", "0"), ("1", "0"), ("0", "1")):
        monkeypatch.setenv("MT_NO_ENTRY", entry)
        monkeypatch.setenv("MT_NO_FUSED_GATHER", gather)
        ctx = make_context(w, max_tenants=3)
        got[entry, gather], launches[entry, gather] = [], []
        for cuts in ([0, rows], [0, rows // 3, rows // 2, rows]):
            out = torch_io.alloc_outputs(rows, ctx.cfg.max_classes)
            for a, b in zip(cuts[:-1], cuts[1:]):
                ctx.submit_batch(d_ids.data_ptr() + 4 * a, at + a * stride * es, b - a, stride)
            ctx.debug_poison()
            ctx.run(torch.cuda.current_stream().cuda_stream, out.labels.data_ptr(), out.probs.data_ptr(), out.logits.data_ptr(), out.n_classes.data_ptr(), rows, ctx.cfg.max_classes)
            torch.cuda.synchronize()
            got[entry, gather].append((out.logits.cpu().numpy().astype(np.float64), out.probs.cpu().numpy().astype(np.float64), out.labels.cpu().numpy(), out.n_classes.cpu().numpy()))
            launches[entry, gather].append(ctx.stats()["last_run_launches"])
        ctx.close()
    first = got["0", "0"][0]
    compare(w, first, oracle_rows(w), what="%s %s x %d" % (dtype, counts, n_in))
    assert all(np.array_equal(u, v) for runs in got.values() for g in runs for u, v in zip(first, g))
    # layers; with the batcher's launch and, staged, that of the rows (one submission: layer 0 has the batcher's work where it reads the rows)
    assert launches["0", "0"] == [3, 4] and launches["1", "0"] == [4, 4] and launches["0", "1"] == [5, 5]


# last layers of 33 to 128 classes finished by tiles of all their column blocks in runs whose tiles split K: classes at the edges of a block and of the range, sums shorter than
# the waves that share them, rows that fill a tile and not; beside a model whose only layer is such a one, the head does them all.  Against the oracle
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("classes", [32, 33, 64, 65, 97, 128, 129])
@pytest.mark.parametrize("rows", [1, 32, 70])
def test_small_runs_finish_wide_last_layers_in_their_tiles(monkeypatch, dtype, classes, rows):
    shapes = ([40, 24, classes], [40, 200, 72, classes], [40, 136, 5])
    models = [wl.make_model(wl.mlp_layers(s, wl.ACT_RELU), dtype, 397, i) for i, s in enumerate(shapes + ([40, 40],))]
    rng = np.random.default_rng(397)
    x = rng.standard_normal((rows, 40)).astype(np.float32)
    for n in (3, 4):                                                 # with the model of one layer, and without
        tenants = dict(enumerate(models[:n]))
        w = wl.Workload("whole", dtype, tenants, (np.arange(rows) % n).astype(np.int32), wl.round_to_bf16(x) if dtype == "bf16" else x)
        launches = []
        for off in ("0", "1"):
            monkeypatch.setenv("MT_NO_FUSED_HEAD", off)
            ctx = make_context(w)
            check(w, "%s, %d classes, %d rows, %d models" % (dtype, classes, rows, n), ctx)
            launches.append(ctx.stats()["last_run_launches"])
            ctx.close()
        if n == 3:
            assert launches[0] == launches[1] - (classes <= 128)
        else:
            assert launches[0] == launches[1]


# on either side of the line for tiles of all a last layer's column blocks (sums of a last layer, its blocks): the launches that the estimate says, the oracle's results
@pytest.mark.parametrize("dtype,k,classes", [("bf16", 1344, 128), ("bf16", 1408, 97), ("bf16", 4096, 64), ("bf16", 4160, 33), ("f32", 128, 100), ("f32", 192, 65), ("f32", 512, 64), ("f32", 576, 40)])
def test_wide_last_layers_around_the_line_of_whole_tiles(dtype, k, classes):
    tenants = {t: wl.make_model(wl.mlp_layers([40, k, classes], wl.ACT_RELU), dtype, 399, t) for t in range(2)}
    x = np.random.default_rng(399).standard_normal((45, 40)).astype(np.float32)
    w = wl.Workload("line", dtype, tenants, (np.arange(45) % 2).astype(np.int32), wl.round_to_bf16(x) if dtype == "bf16" else x)
    ctx = make_context(w)
    launches = ctx.estimate_run(np.bincount(w.tenant_ids))["launches"]
    check(w, "%s %d %d" % (dtype, k, classes), ctx)
    assert ctx.stats()["last_run_launches"] == launches
    ctx.close()


# frames of which one tile fewer fits a compute unit with their tenants' facts beside them: a launch that starts at once has the facts ahead, a larger one of the same tenants not.
# The same images in both, and against the oracle
@pytest.mark.parametrize("dtype,hw,chans", [("bf16", 8, (3, 192, 192, 192)), ("bf16", 10, (3, 128, 64, 128)), ("f32", 8, (3, 96, 96, 96))])
def test_frames_with_and_without_facts_beside_them(dtype, hw, chans):
    es, frames = 2 if dtype == "bf16" else 4, []
    for cin, cout in zip(chans[1:], chans[2:]):
        t = mt.debug_conv_row_tiling(hw, hw, cin, elem_size=es)
        grid = lambda rows, t=t: -(-rows // t["images_per_tile"]) * t["tiles_per_image"]  # noqa: E731
        frames.append([mt.debug_conv_frame_ahead(3, -(-cout // 32), t["frame_bytes"], grid(rows)) for rows in (160, 1600)])
    assert [True, False] in frames
    tenants = {t: wl.make_model(wl.cnn_layers(hw=hw, chans=chans, strides=(1,) * (len(chans) - 1)), dtype, 400, t) for t in range(3)}
    rng = np.random.default_rng(400)
    x = rng.standard_normal((1600, hw * hw * 3)).astype(np.float32)
    w = wl.Workload("frames", dtype, tenants, rng.integers(0, 3, 1600).astype(np.int32), wl.round_to_bf16(x) if dtype == "bf16" else x)
    ctx = make_context(w)
    every, few = gpu_run(ctx, w, poison=True), gpu_run(ctx, w, ids=w.tenant_ids[:160], inputs=w.inputs[:160], poison=True)
    ctx.close()
    # (the pooling launch adds an image's 64 pixels in another order from some number of rows on: fp32 logits and probabilities may differ by 64 roundings of 2^-24)
    for a, b in zip(every, few):
        assert np.array_equal(a[:160], b) or (dtype == "f32" and np.linalg.norm(a[:160] - b) <= 64 * 2.0 ** -24 * np.linalg.norm(b))
    assert np.array_equal(every[2][:160], few[2])
    pick = np.arange(0, 1600, 53)
    compare(w, tuple(v[pick] for v in every), oracle_rows(w, pick), rows=pick, what="frames")
