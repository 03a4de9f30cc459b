"""What the runtime's speed is measured on: whole serving passes through the public entry points.

A pass is what a worker does with the requests that are waiting: submit them (one batch of mixed tenants whose ids are
already in device memory, or one call per tenant), run, and have labels, probabilities, logits and class counts of every
request in submission order.  A case names the models the worker hosts and the requests of one pass; `prepare` sets up
what a worker has in hand before the requests arrive: a context with the models registered, the requests in device
memory, the output buffers and the streams.  Model and request values follow the repository's workloads: weights
N(0, 1/fan_in), biases N(0, 0.01), inputs N(0, 1) or U(0, 1), a batch normalisation behind every convolution of the
residual models, tenants drawn uniformly or by Zipf popularity.

The keys of a case
  kind      mlp (`hidden`: the widths of the hidden layers; or `choices`: every tenant draws its depth from
            depth_lo..depth_hi linear layers and each hidden width from these), cnn (3x3 convolutions over an
            h x w image, then a global average pool and a linear layer), resnet (18 layers with skip connections,
            `width` channels in the first stage), fleet (tenants take turns at being an MLP, a CNN and a residual
            net, all fed the same hw x hw x 3 requests)
  dtype     bf16 or f32 (weights, inputs and hidden activations)
  tenants, requests, skew (Zipf exponent, 0: uniform), act (relu, gelu, none), inputs (normal, uniform), classes
  submit    batch: one mt_submit_batch; tenant: one mt_submit per tenant and chunk of at most `chunk` rows
  streams   runs in flight, each over requests and outputs of its own, on as many streams
"""
import math

import torch

import paper_1901_06887_amd as mt

ACTS = {"none": mt.MT_ACT_NONE, "relu": mt.MT_ACT_RELU, "gelu": mt.MT_ACT_GELU}
MT_EFULL = 6
BASE = {"dtype": "bf16", "act": "relu", "inputs": "normal", "skew": 0.0, "submit": "batch", "chunk": 32, "streams": 1}


def listed():
    return [dict(BASE, **c) for c in (
        # the smallest call: one request to one of a few small models, submitted by its tenant; launches and latency
        {"name": "mlp_one_request", "kind": "mlp", "tenants": 8, "requests": 1, "in_dim": 784, "hidden": "1024,1024", "classes": 10,
         "submit": "tenant"},
        # a small fp32 batch: four tenants, some sixteen requests each
        {"name": "mlp_f32_small", "kind": "mlp", "dtype": "f32", "tenants": 4, "requests": 64, "in_dim": 256, "hidden": "512,512", "classes": 10},
        # the ordinary batch of a worker with many small models, popularity skewed; weights decide
        {"name": "mlp_zipf", "kind": "mlp", "tenants": 64, "requests": 4096, "in_dim": 784, "hidden": "1024,1024", "classes": 10, "skew": 1.1,
         "inputs": "uniform"},
        # the same worker with three runs in flight on three streams
        {"name": "mlp_zipf_three_runs", "kind": "mlp", "tenants": 64, "requests": 4096, "in_dim": 784, "hidden": "1024,1024", "classes": 10, "skew": 1.1,
         "inputs": "uniform", "streams": 3},
        # many tenants whose models all differ in depth and width
        {"name": "mlp_mixed_depths", "kind": "mlp", "tenants": 256, "requests": 16384, "in_dim": 1024, "choices": "512,1024,2048", "depth_lo": 2,
         "depth_hi": 6, "classes": 100, "skew": 1.2},
        # odd sizes everywhere, GELU, requests arriving tenant by tenant in small pieces
        {"name": "mlp_ragged", "kind": "mlp", "tenants": 24, "requests": 777, "in_dim": 301, "hidden": "333,520,97", "classes": 37, "act": "gelu",
         "skew": 0.8, "submit": "tenant", "chunk": 64},
        # large batches through wide models: arithmetic decides
        {"name": "mlp_wide_gelu", "kind": "mlp", "tenants": 8, "requests": 32768, "in_dim": 4096, "hidden": "4096,4096,4096", "classes": 1000,
         "act": "gelu"},
        # small images through small CNNs
        {"name": "cnn_batch", "kind": "cnn", "tenants": 32, "requests": 2048, "h": 32, "w": 32, "chans": "3,32,64,128", "strides": "1,2,2", "classes": 10},
        # an fp32 CNN over images that are neither square nor powers of two
        {"name": "cnn_f32_odd", "kind": "cnn", "dtype": "f32", "tenants": 6, "requests": 150, "h": 29, "w": 35, "chans": "3,24,40,72", "strides": "1,1,2",
         "classes": 33},
        # 18-layer residual nets on full-size images: a batch, and the single request
        {"name": "resnet_batch", "kind": "resnet", "tenants": 4, "requests": 64, "hw": 224, "width": 64, "classes": 1000},
        {"name": "resnet_one_request", "kind": "resnet", "tenants": 4, "requests": 1, "hw": 224, "width": 64, "classes": 1000, "submit": "tenant"},
        # MLPs, CNNs and residual nets side by side in one worker
        {"name": "fleet", "kind": "fleet", "tenants": 12, "requests": 600, "hw": 32, "width": 32, "classes": 40, "skew": 0.8},
    )]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _size(rng, lo, hi, multiple):
    """A size spread over its logarithm; half of them round, half as they come."""
    v = _log_int(rng, lo, hi)
    return max(multiple, v // multiple * multiple) if rng.random() < 0.5 else v


def draw(rng):
    while True:
        kind = rng.choice(["mlp", "mlp", "mlp", "cnn", "cnn", "resnet", "fleet"])
        c = dict(BASE, kind=kind, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), act=rng.choice(["relu", "relu", "gelu"]),
                 skew=rng.choice([0.0, 0.8, 1.1, 1.2]), submit=rng.choice(["batch", "batch", "tenant"]), chunk=rng.randint(1, 64),
                 streams=rng.choice([1, 1, 1, 1, 2, 3]))
        if kind == "mlp":
            c.update(tenants=_log_int(rng, 1, 256), requests=_log_int(rng, 1, 32768), in_dim=_size(rng, 24, 4096, 64), classes=_size(rng, 3, 1000, 8))
            if rng.random() < 0.3:
                c.update(choices=",".join(str(_size(rng, 64, 2048, 64)) for _ in range(3)), depth_lo=2, depth_hi=rng.randint(2, 6))
            else:
                c.update(hidden=",".join(str(_size(rng, 24, 4096, 64)) for _ in range(rng.randint(1, 4))))
        elif kind == "cnn":
            n = rng.randint(1, 4)
            c.update(tenants=_log_int(rng, 1, 64), requests=_log_int(rng, 1, 4096), h=rng.randint(8, 64), classes=rng.choice([4, 10, 33, 100]),
                     chans=",".join(["3"] + [str(8 * _log_int(rng, 1, 16)) for _ in range(n)]), strides=",".join(str(rng.choice([1, 2])) for _ in range(n)))
            c["w"] = c["h"] if rng.random() < 0.5 else rng.randint(8, 64)
        elif kind == "resnet":
            c.update(tenants=_log_int(rng, 1, 8), requests=_log_int(rng, 1, 256), hw=8 * rng.randint(4, 28), width=8 * _log_int(rng, 2, 8), classes=rng.choice([10, 100, 1000]))
        else:
            c.update(tenants=_log_int(rng, 3, 48), requests=_log_int(rng, 3, 4096), hw=rng.choice([16, 24, 32]), width=rng.choice([16, 32]), classes=rng.choice([10, 40]))
        p, f, act = _cost(c)
        if c["submit"] == "tenant" and c["requests"] > 64 * c["chunk"]:
            c["chunk"] = -(-c["requests"] // 64)                        # a worker's calls per run, not its rows
        # no larger than the largest listed case in weights and operations, and activations that leave room for three contexts
        if p <= 3.0e8 and f * c["streams"] * (8 if c["dtype"] == "f32" else 1) <= 3.5e12 and act * c["streams"] <= 6e9:
            return c


# ---- models -----------------------------------------------------------------------------------------------------------
def _mlp(dims, act):
    return [mt.layer_spec(mt.MT_FC, ACTS[act] if i < len(dims) - 2 else mt.MT_ACT_NONE, dims[i], dims[i + 1]) for i in range(len(dims) - 1)]


def _cnn(h, w, chans, strides, classes, act):
    layers = []
    for i, s in enumerate(strides):
        layers.append(mt.layer_spec(mt.MT_CONV2D, ACTS[act], chans[i], chans[i + 1], h, w, s, ksize=3, pad=1))
        h, w = (h - 1) // s + 1, (w - 1) // s + 1
    layers.append(mt.layer_spec(mt.MT_GAP, mt.MT_ACT_NONE, chans[-1], chans[-1], h, w))
    layers.append(mt.layer_spec(mt.MT_FC, mt.MT_ACT_NONE, chans[-1], classes))
    return layers


def _resnet(hw, width, classes):
    conv = lambda act, ci, co, h, s, k, src=0: mt.layer_spec(mt.MT_CONV2D, act, ci, co, h, h, s, ksize=k, pad=(k - 1) // 2, src=src)  # noqa: E731
    L = [conv(mt.MT_ACT_RELU, 3, width, hw, 2, 7)]
    h = (hw - 1) // 2 + 1
    L.append(mt.layer_spec(mt.MT_MAXPOOL, mt.MT_ACT_NONE, width, width, h, h, 2, ksize=3, pad=1))
    h = (h - 1) // 2 + 1
    ci = width
    for stage in range(4):
        co = width << stage
        for block in range(2):
            s = 2 if stage > 0 and block == 0 else 1
            x = len(L)                                                  # source code of the block's input
            h2 = (h - 1) // s + 1
            L += [conv(mt.MT_ACT_RELU, ci, co, h, s, 3), conv(mt.MT_ACT_NONE, co, co, h2, 1, 3)]
            main = len(L)
            if s != 1 or ci != co:
                L.append(conv(mt.MT_ACT_NONE, ci, co, h, s, 1, src=x))
                L.append(mt.layer_spec(mt.MT_ADD, mt.MT_ACT_RELU, co, co, h2, h2, src=main, src2=len(L)))
            else:
                L.append(mt.layer_spec(mt.MT_ADD, mt.MT_ACT_RELU, co, co, h2, h2, src2=x))
            ci, h = co, h2
    L.append(mt.layer_spec(mt.MT_GAP, mt.MT_ACT_NONE, ci, ci, h, h))
    L.append(mt.layer_spec(mt.MT_FC, mt.MT_ACT_NONE, ci, classes))
    return L


def _ints(text):
    return [int(v) for v in text.split(",")]


def _in_len(case):
    if case["kind"] == "mlp":
        return case["in_dim"]
    return 3 * case["h"] * case["w"] if case["kind"] == "cnn" else 3 * case["hw"] ** 2


def _layers(case, tenant, pick):
    """Layer list of one tenant; `pick(n)` draws from 0 .. n-1."""
    kind = case["kind"]
    if kind == "fleet":
        kind = ("mlp", "cnn", "resnet")[tenant % 3]
        hw, width = case["hw"], case["width"]
        if kind == "mlp":
            return _mlp([3 * hw * hw, 8 * width, 4 * width, case["classes"]], case["act"])
        if kind == "cnn":
            return _cnn(hw, hw, [3, width, 2 * width, 4 * width], [1, 2, 2], case["classes"], case["act"])
        return _resnet(hw, width, case["classes"])
    if kind == "mlp":
        if "choices" in case:
            options = _ints(case["choices"])
            depth = case["depth_lo"] + pick(case["depth_hi"] - case["depth_lo"] + 1)
            hidden = [options[pick(len(options))] for _ in range(depth - 1)]
        else:
            hidden = _ints(case["hidden"])
        return _mlp([case["in_dim"], *hidden, case["classes"]], case["act"])
    if kind == "cnn":
        return _cnn(case["h"], case["w"], _ints(case["chans"]), _ints(case["strides"]), case["classes"], case["act"])
    return _resnet(case["hw"], case["width"], case["classes"])


def _params(s):
    return (s.in_features * s.out_features * (s.kh * s.kw if s.kind == mt.MT_CONV2D else 1)) if s.kind in (mt.MT_FC, mt.MT_CONV2D) else 0


def _out_hw(s):
    return ((s.in_h + 2 * s.pad - s.kh) // s.stride + 1) * ((s.in_w + 2 * s.pad - s.kw) // s.stride + 1)


def _model_cost(layers):
    """(weights and biases of one model in values, operations of one request, most values of a request between two layers)"""
    params = flops = width = 0
    for s in layers:
        px = _out_hw(s) if s.kind == mt.MT_CONV2D else 1
        params += _params(s) + (s.out_features if _params(s) else 0)
        flops += 2 * px * _params(s)
        width = max(width, s.in_features * max(1, s.in_h * s.in_w), s.out_features * px)
    return params, flops, width


def _shares(case):
    """Expected share of the requests per popularity rank."""
    p = [(k + 1) ** -case["skew"] for k in range(case["tenants"])]
    return [v / sum(p) for v in p]


def _averages(case):
    """Expected (weights, operations per request, width) of a tenant's model."""
    if "choices" in case:
        options = _ints(case["choices"])
        m, depths = sum(options) / len(options), range(case["depth_lo"], case["depth_hi"] + 1)
        macs = sum(case["in_dim"] * m + (d - 2) * m * m + m * case["classes"] for d in depths) / len(depths)
        return macs + sum((d - 1) * m + case["classes"] for d in depths) / len(depths), 2 * macs, max(case["in_dim"], *options)
    n = min(3, case["tenants"]) if case["kind"] == "fleet" else 1
    each = [_model_cost(_layers(case, t, None)) for t in range(n)]
    return sum(e[0] for e in each) / n, sum(e[1] for e in each) / n, max(e[2] for e in each)


def _cost(case):
    """(registered weights, operations, bytes of one run's activations) of a case."""
    params, flops, width = _averages(case)
    es = 2 if case["dtype"] == "bf16" else 4
    return params * case["tenants"], flops * case["requests"], 3 * es * width * (case["requests"] + 32 * min(case["tenants"], case["requests"]))


# ---- the measured path ------------------------------------------------------------------------------------------------
class _Model:
    def __init__(self, layers, dtype, g):
        self.layers, self.weights, self.biases, self.bn, self.bn_eps = layers, [], [], None, 1e-5
        residual = any(s.kind == mt.MT_ADD for s in layers)
        bn = []
        for s in layers:
            if not _params(s):
                self.weights.append(None), self.biases.append(None), bn.append(None)
                continue
            k = s.in_features * (s.kh * s.kw if s.kind == mt.MT_CONV2D else 1)
            w = torch.randn(s.out_features, k, generator=g, device="cuda") * k ** -0.5
            w = w.to(torch.bfloat16).view(torch.int16).cpu().numpy().view("uint16") if dtype == "bf16" else w.cpu().numpy()
            self.weights.append(w)
            self.biases.append((torch.randn(s.out_features, generator=g, device="cuda") * 0.1).cpu().numpy())
            if residual and s.kind == mt.MT_CONV2D:
                n = torch.randn(2, s.out_features, generator=g, device="cuda") * 0.1
                u = torch.rand(2, s.out_features, generator=g, device="cuda") + 0.5
                bn.append(tuple(v.cpu().numpy() for v in (u[0], n[0], n[1], u[1])))       # gamma, beta, mean, variance
            else:
                bn.append(None)
        if any(b is not None for b in bn):
            self.bn = bn


def prepare(case, seed):
    g = torch.Generator("cuda").manual_seed(seed * 1000003 + 11)
    host = torch.Generator().manual_seed(seed * 1000003 + 12)
    pick = lambda n: int(torch.randint(n, (1,), generator=host))  # noqa: E731
    R, T, n_in = case["requests"], case["tenants"], _in_len(case)
    plans = [_layers(case, t, pick) for t in range(T)]
    code = mt.MT_BF16 if case["dtype"] == "bf16" else mt.MT_F32
    prints = [mt.model_footprint(p, code) for p in plans]
    ctx = mt.Context(T, R, max(f["min_width"] for f in prints), max(f["n_classes"] for f in prints), sum(f["arena_bytes"] for f in prints) + (1 << 20),
                     code, 0, case["streams"])
    for t in range(T):
        m = _Model(plans[t], case["dtype"], g)
        ctx.register_model(t, m.layers, m.weights, m.biases, m.bn, m.bn_eps)
    share = torch.tensor(_shares(case))[torch.randperm(T, generator=host)]                # popularity rank -> tenant
    jobs = []
    for j in range(case["streams"]):
        ids = torch.multinomial(share, R, replacement=True, generator=host).to(torch.int32)
        x = torch.randn(R, n_in, generator=g, device="cuda") if case["inputs"] == "normal" else torch.rand(R, n_in, generator=g, device="cuda")
        x = x.to(torch.bfloat16) if case["dtype"] == "bf16" else x
        calls = []
        if case["submit"] == "tenant":                                                    # (tenant, first row, rows): each tenant's rows lie together
            ids = ids.sort().values
            counts = torch.bincount(ids.long(), minlength=T).tolist()
            at = 0
            pieces = []
            for t, n in enumerate(counts):
                pieces += [(t, at + a, min(case["chunk"], n - a)) for a in range(0, n, case["chunk"])]
                at += n
            calls = [pieces[i] for i in torch.randperm(len(pieces), generator=host).tolist()]   # they arrive in any order
        n_out = ctx.cfg.max_classes
        out = mt.Served(torch.empty(R, dtype=torch.int32, device="cuda"), torch.empty(R, n_out, device="cuda"), torch.empty(R, n_out, device="cuda"),
                        torch.empty(R, dtype=torch.int32, device="cuda"))
        jobs.append({"ids": ids.cuda(), "x": x, "calls": calls, "out": out, "stream": torch.cuda.Stream() if case["streams"] > 1 else None})
    return {"ctx": ctx, "jobs": jobs}


def _serve(ctx, job, stream):
    if not job["calls"]:
        return mt.serve(ctx, job["ids"], job["x"], job["out"], stream)
    base, row = job["x"].data_ptr(), job["x"].stride(0) * job["x"].element_size()
    for t, first, n in job["calls"]:
        ctx.submit(t, base + first * row, n)
    o = job["out"]
    args = (stream.cuda_stream, o.labels.data_ptr(), o.probs.data_ptr(), o.logits.data_ptr(), o.n_classes.data_ptr(), o.labels.numel(), o.probs.shape[1])
    try:
        ctx.run(*args)
    except mt.MtError as e:
        if e.status != MT_EFULL:
            raise
        stream.synchronize()            # eight runs of several submissions are still queued: a worker waits and calls again
        ctx.run(*args)
    return o


def run(state):
    here = torch.cuda.current_stream()
    outs = []
    for job in state["jobs"]:
        if job["stream"] is not None:
            job["stream"].wait_stream(here)
    for job in state["jobs"]:
        o = _serve(state["ctx"], job, job["stream"] or here)
        outs.append((o.labels, o.probs, o.logits, o.n_classes))
    for job in state["jobs"]:
        if job["stream"] is not None:
            here.wait_stream(job["stream"])
    return outs


def work(case):
    """Requests read once, the weights of the tenants expected to have requests read once, predictions written once."""
    params, flops, _ = _averages(case)
    es, R, n = 2 if case["dtype"] == "bf16" else 4, case["requests"], case["streams"]
    active = sum(1.0 - (1.0 - p) ** (R * n) for p in _shares(case))     # runs in flight share the weights
    return {"bytes": active * params * es + n * R * (_in_len(case) * es + 2 * 4 * case["classes"] + 8), "flops": n * R * flops}


def tolerance(case):
    """About four times what the path differs by from itself in 64 bits (and, for the linear layers, with sums in another order).

    fp32: up to 6e-7 of the norm, 2e-6 at the largest value.  bf16: a hidden activation that lies on a rounding boundary goes the
    other way in another summation order, and the layers behind it amplify that: 1e-4 to 6.4e-4 of the norm over many requests of
    shallow models (largest value 7e-3), up to 1e-2 of a single request's, which is what counts in small batches; 1.2e-3 (2.8e-2)
    with residual nets among the models, 2e-3 to 9e-3 (4.1e-2) for full-size residual nets, whose every request holds several such values.
    Labels: no difference seen; a few near ties are allowed."""
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-5, "differ": 1e-3}
    if case["kind"] == "resnet":
        return {"rel": 2e-2, "max": 0.17, "differ": 1e-2}
    if case["requests"] < 100:
        return {"rel": 1e-2, "max": 0.1, "differ": 1e-2}
    return {"rel": 5e-3, "max": 0.12, "differ": 2e-3} if case["kind"] == "fleet" else {"rel": 2.5e-3, "max": 3e-2, "differ": 1e-3}
