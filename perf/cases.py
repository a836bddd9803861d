"""Workloads of the codec and of its products, for timing and comparison.

A case is one call (or one block's calls) of the library as a program makes it:

  gemv    batch-1 decode: one grouped fused GEMV per activation (q/k/v, o,
          gate/up, down of a block), plans and workspaces kept;
  gemm    M tokens through one projection (batched decode, prefill chunks);
  encode  one matrix, or a category's stack, into planes;
  decode  planes back to a dense matrix;
  train   one codec-training step: loss and gradient of a mini-batch, Adam.

The encoded layers that the products and the decode read are made here in
plain torch from Gaussian weights with 1% large input columns (a stand-in for
a stored compressed checkpoint); they follow the documented layout, and the
64-bit results are computed from the same planes.
"""
import math
from types import SimpleNamespace

import torch

import paper_2607_08643_amd as bsq

DEV = "cuda"
PAYLOAD_MAX = {0: 127.0, 1: 448.0, 2: 57344.0}
BLOCK_8B = [[(4096, 4096), (1024, 4096), (1024, 4096)], [(4096, 4096)], [(12288, 4096), (12288, 4096)],
            [(4096, 12288)]]


# ---------------------------------------------------------------- the cases
def _case(name, op, **kw):
    c = {"name": name, "op": op, "d": 8, "b": 0, "stages": 2, "protect": 1, "fmt": 0, "lora": 0, "dtype": "bf16"}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one 256 x 256 fp32 layer, all latency
        _case("gemv-tiny-f32", "gemv", shape="256x256", protect=0, dtype="fp32"),
        # one decode token through one 4096/12288 block (q/k/v, o, gate/up,
        # down: four grouped launches), an adapter on every projection
        _case("token-block-d8-lora", "gemv", shape="block", lora=16),
        # the largest group of a batch-1 token: gate and up of a 5120/25600 block
        _case("token-gateup-d8", "gemv", shape="25600+25600x5120"),
        # the same 4096/12288 block at half the code rate, FP8 protected columns
        _case("token-block-d16-e4m3", "gemv", shape="block", d=16, fmt=1),
        # batched decode: 16 sequences through an attention output projection
        _case("gemm-16-d8-lora", "gemm", shape="4096x4096", M=16, lora=16),
        # batched decode: 64 sequences through a gate projection, half rate
        _case("gemm-64-d16-lora", "gemm", shape="12288x4096", M=64, lora=16, d=16),
        # 256 tokens through a down projection (long inputs)
        _case("gemm-256-d8-lora", "gemm", shape="4096x12288", M=256, lora=16),
        # prefill: a ragged chunk of 2000 tokens through a gate projection
        _case("gemm-2000-d8-lora", "gemm", shape="12288x4096", M=2000, lora=16),
        # quantising one projection (a checkpoint walked matrix by matrix)
        _case("encode-one-d8", "encode", shape="12288x4096", mats=1),
        # quantising a category's stack of layers in one call, half rate
        _case("encode-stack-d16", "encode", shape="4096x4096", mats=8, d=16),
        # a dense bf16 copy of one projection with odd sizes
        _case("decode-ragged-d8", "decode", shape="11003x5000", mats=1),
        # one training step of a stage codec on 65,536 chunks of a category
        _case("train-64k-d8", "train", shape="4096x4096", mats=4, n=65536, b=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["gemv", "gemv", "gemm", "gemm", "gemm", "encode", "decode", "train"])
    d = rng.choice([8, 8, 16])
    c = _case("", op, d=d, stages=rng.choice([2, 2, 2, 2, 1, 3]), fmt=rng.choice([0, 0, 1]),
              lora=rng.choice([0, 16]))
    del c["name"]
    dim = lambda lo, hi: _log_int(rng, lo, hi)  # noqa: E731
    cols = lambda lo, hi: max(1, dim(lo, hi) // d) * d  # noqa: E731
    if op == "gemv":
        rows = [dim(64, 25600) for _ in range(rng.choice([1, 1, 2, 3]))]
        c["shape"] = "%sx%d" % ("+".join(map(str, rows)), min(cols(256, 25600), 262144000 // sum(rows) // d * d))
        if rng.random() < 0.15:
            c.update(shape="%dx%d" % (dim(64, 1024), cols(256, 1024)), dtype="fp32", lora=0)
    elif op == "gemm":
        M, rows = dim(2, 2048), dim(64, 12288)
        c.update(M=M, shape="%dx%d" % (rows, max(256, min(cols(256, 12288), 100000000000 // (M * rows) // d * d))))
    elif op in ("encode", "decode"):
        rows, mats = dim(256, 12288), rng.choice([1, 1, 2, 4, 8])
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        most = (100000000 if dtype == "bf16" else 50000000) // (mats * rows) // d * d
        c.update(mats=mats, lora=0, dtype=dtype, shape="%dx%d" % (rows, max(256, min(cols(256, 12288), most))))
    else:
        c.update(n=dim(4096, 131072), b=rng.choice([8, 8, 16]), shape="4096x4096", mats=1, stages=1, fmt=0, lora=0,
                 protect=0, dtype=rng.choice(["bf16", "bf16", "fp32"]))
    return c


# ---------------------------------------------------------------- inputs
def _groups(c):
    """The case's groups of (d_out, d_in) that share an activation."""
    if c["shape"] == "block":
        return BLOCK_8B
    rows, cols = c["shape"].split("x")
    return [[(int(r), int(cols)) for r in rows.split("+")]]


def _dims(c):
    return _groups(c)[0][0]


def _k(c, d_in):
    return (d_in + 99) // 100 if c["protect"] else 0


def _dtype(c):
    return torch.float32 if c["dtype"] == "fp32" else torch.bfloat16


def _config(c):
    linear = c["op"] == "train"
    b = c["b"] or c["d"]
    return bsq.Config(d=c["d"], stages=c["stages"], kind=bsq.DEC_MLP, hidden=b, protect_num=c["protect"],
                      protect_den=100, protect_format=c["fmt"], codebook_bits=b,
                      encoder=bsq.ENC_LINEAR if linear else bsq.ENC_IDENTITY)


def _gen(seed, *more):
    s = int(seed) & 0xFFFFFFFF
    for m in more:
        s = (s * 1000003 + int(m) + 1) & 0x7FFFFFFFFFFF
    return torch.Generator(device=DEV).manual_seed(s)


def _uniform(g, shape, fan_in):
    return (torch.rand(shape, generator=g, device=DEV) * 2 - 1) / math.sqrt(fan_in)


def _decoders(c, seed, category=0):
    b, d, h = c["b"] or c["d"], c["d"], c["b"] or c["d"]
    out = []
    for s in range(c["stages"]):
        g = _gen(seed, 11, category, s)
        out.append(SimpleNamespace(W1=_uniform(g, (h, b), b), b1=_uniform(g, (h,), b), W2=_uniform(g, (d, h), h),
                                   b2=_uniform(g, (d,), h)))
    return out


def _tables(c, decs):
    """Every stage decoder on all 2^b codes, fp64 [2^b][d]."""
    b = c["b"] or c["d"]
    codes = torch.arange(1 << b, device=DEV)
    q = (((codes[:, None] >> torch.arange(b, device=DEV)) & 1) * 2 - 1).double() / math.sqrt(b)
    return [torch.relu(q @ D.W1.double().T + D.b1.double()) @ D.W2.double().T + D.b2.double() for D in decs]


def _weight(c, g, mats, d_out, d_in):
    W = torch.randn((mats, d_out, d_in), generator=g, device=DEV) * 0.02
    k = _k(c, d_in)
    for m in range(mats if k else 0):
        W[m][:, torch.randperm(d_in, generator=g, device=DEV)[:k]] *= 10
    return W.to(_dtype(c))


def _tiled(c, plane):
    """[d_out][C] as 64-row x 16-chunk tiles, padded with zeros."""
    rows, C = plane.shape
    R, P = (rows + 63) // 64 * 64, (C + 15) // 16 * 16
    t = torch.zeros((R, P), dtype=plane.dtype, device=DEV)
    t[:rows, :C] = plane
    return t.view(R // 64, 64, P // 16, 16).transpose(1, 2).contiguous()


def _compress(c, W, tabs, want):
    """One encoded matrix in plain torch: per stage (codes, gains) [d_out][C],
    then the protected columns, their stored bytes and scales. want(s, codes,
    gains, y): called per stage with the decoded vectors."""
    d = c["d"]
    d_out, d_in = W.shape
    k = _k(c, d_in)
    W = W.float()
    idx = q8 = scale = None
    keep = torch.ones(d_in, device=DEV)
    if k:
        idx = W.double().square().sum(0).topk(k).indices.sort().values
        keep[idx] = 0
        cols = W[:, idx]
        scale = cols.abs().amax(0) / PAYLOAD_MAX[c["fmt"]]
        v = cols / scale
        q8 = v.round().clamp(-127, 127).to(torch.int8) if c["fmt"] == 0 else v.to(
            torch.float8_e4m3fn if c["fmt"] == 1 else torch.float8_e5m2).view(torch.int8)
    keep = keep.view(1, -1, d)
    r = W.view(d_out, -1, d) * keep
    shift = torch.arange(d, device=DEV)
    for s in range(c["stages"]):
        code = ((r >= 0).int() << shift).sum(-1, dtype=torch.int32)
        y = tabs[s].float()[code.long()] * keep
        gain = torch.nan_to_num((r * y).sum(-1) / y.square().sum(-1), 0.0, 0.0, 0.0).half()
        r = r - gain.float()[..., None] * y
        want(s, code, gain, y)
    return idx, q8, scale


def _stored_layer(c, cfg, W, tabs):
    """The encoded layer of W."""
    d_out, d_in = W.shape
    L = bsq.layer_empty(cfg, d_out, d_in, 1, DEV)

    def put(s, code, gain, _y):
        L.codes[s].copy_(_tiled(c, code).to(torch.uint8) if c["d"] == 8 else _tiled(c, code).to(torch.int16))
        L.gains[s].copy_(_tiled(c, gain))

    idx, q8, scale = _compress(c, W, tabs, put)
    if idx is not None:
        L.idx.copy_(idx)
        L.scale.copy_(scale)
        L.q8.zero_()
        L.q8[:, :idx.numel()] = q8
        bit = torch.zeros(L.bits.numel() * 32, dtype=torch.int64, device=DEV)
        bit[idx] = 1
        word = (bit.view(-1, 32) << torch.arange(32, device=DEV)).sum(1)
        L.bits.copy_(torch.where(word >= 1 << 31, word - (1 << 32), word))
    return L


def _decoded(c, W, tabs):
    """The fp64 matrix that the stored form of W stands for."""
    d_out, d_in = W.shape
    out = torch.zeros((d_out, d_in // c["d"], c["d"]), dtype=torch.float64, device=DEV)

    def add(s, code, gain, _y):
        out.add_(gain.double()[..., None] * tabs[s][code.long()])

    idx, q8, scale = _compress(c, W, tabs, add)
    out = out.view(d_out, d_in)
    if idx is not None:
        v = q8.double() if c["fmt"] == 0 else q8.view(
            torch.float8_e4m3fn if c["fmt"] == 1 else torch.float8_e5m2).double()
        out[:, idx] = v * scale.double()
    return out


def _members(c, seed):
    """Per group: the activation, and per member its weight, decoders and adapter."""
    for gi, group in enumerate(_groups(c)):
        g = _gen(seed, 23, gi)
        d_in = group[0][1]
        shape = (c["M"], d_in) if c["op"] == "gemm" else (d_in,)
        x = torch.randn(shape, generator=g, device=DEV).to(_dtype(c))
        mem = []
        for mi, (d_out, _) in enumerate(group):
            W = _weight(c, g, 1, d_out, d_in)[0]
            lora = None
            if c["lora"]:
                lora = tuple((torch.randn(s, generator=g, device=DEV) * 0.01).to(torch.bfloat16)
                             for s in ((c["lora"], d_in), (d_out, c["lora"])))
            mem.append((W, _decoders(c, seed, 16 * gi + mi), lora))
        yield x, mem


def _aligned_ws(n, zero=False):
    t = (torch.zeros if zero else torch.empty)(n + 256, dtype=torch.uint8, device=DEV)
    return t[(-t.data_ptr()) % 256:][:n]


def prepare(case, seed):
    c, cfg = case, _config(case)
    st = SimpleNamespace(c=c, cfg=cfg)
    if c["op"] in ("gemv", "gemm"):
        st.calls = []
        for x, mem in _members(c, seed):
            codecs = [bsq.bsq_codec_prepare(cfg, decs, DEV) for _, decs, _ in mem]
            layers = [_stored_layer(c, cfg, W, _tables(c, decs)) for W, decs, _ in mem]
            loras = [l for _, _, l in mem]
            if c["op"] == "gemv":
                st.calls.append(bsq.GemvPlan(cfg, codecs, layers, x, loras=loras if c["lora"] else None,
                                             y_dtype=_dtype(c)))
            else:
                L = layers[0]
                ws = _aligned_ws(bsq.bsq_workspace_bytes(cfg, bsq.OP_GEMM, 1, L.d_out, L.d_in, c["M"]))
                out = torch.empty((c["M"], L.d_out), dtype=torch.bfloat16, device=DEV)
                st.calls.append((codecs[0], L, x, loras[0], out, ws))
        return st
    d_out, d_in = _dims(c)
    W = _weight(c, _gen(seed, 31), c["mats"], d_out, d_in)
    if c["op"] == "train":
        b, d, h = c["b"], c["d"], c["b"]
        g = _gen(seed, 37)
        st.chunks = W
        st.idx = torch.randint(0, W.numel() // d, (c["n"],), generator=g, device=DEV)
        st.theta = torch.cat([_uniform(g, (b * d,), d), _uniform(g, (h * b,), b), _uniform(g, (h,), b),
                              _uniform(g, (d * h,), h), _uniform(g, (d,), h)])
        st.m, st.v = torch.zeros_like(st.theta), torch.zeros_like(st.theta)
        st.grad, st.loss = torch.empty_like(st.theta), torch.empty(4, device=DEV)
        st.hp, st.step = bsq.TrainHyper(), 0
        st.ws = _aligned_ws(bsq.bsq_train_workspace_bytes(cfg, c["n"]))
        return st
    st.codec = bsq.bsq_codec_prepare(cfg, _decoders(c, seed), DEV)
    if c["op"] == "encode":
        st.W = W if c["mats"] > 1 else W[0]
        st.out = bsq.layer_empty(cfg, d_out, d_in, c["mats"], DEV)
        st.ws = _aligned_ws(bsq.bsq_workspace_bytes(cfg, bsq.OP_ENCODE, c["mats"], d_out, d_in))
        st.err = torch.zeros(1, dtype=torch.int32, device=DEV)
        return st
    tabs = _tables(c, _decoders(c, seed))
    Ls = [_stored_layer(c, cfg, W[m], tabs) for m in range(c["mats"])]
    st.layer = Ls[0]
    if c["mats"] > 1:
        one = lambda f: None if f(Ls[0]) is None else torch.stack([f(L) for L in Ls])  # noqa: E731
        st.layer = bsq.Layer(cfg, [one(lambda L, s=s: L.codes[s]) for s in range(c["stages"])],
                             [one(lambda L, s=s: L.gains[s]) for s in range(c["stages"])], one(lambda L: L.idx),
                             one(lambda L: L.q8), one(lambda L: L.scale), d_out, d_in, c["mats"],
                             one(lambda L: L.bits))
    st.out = torch.empty(tuple(W.shape) if c["mats"] > 1 else (d_out, d_in), dtype=_dtype(c), device=DEV)
    return st


def run(st):
    op = st.c["op"]
    if op == "gemv":
        return [plan() for plan in st.calls]
    if op == "gemm":
        return [bsq.bsq_gemm(st.cfg, codec, L, X, lora=lora, out=out, ws=ws)
                for codec, L, X, lora, out, ws in st.calls]
    if op == "encode":
        L = bsq.bsq_encode(st.cfg, st.codec, st.W, out=st.out, ws=st.ws, err=st.err, check=False)
        return {"codes": list(L.codes), "gains": list(L.gains), "idx": L.idx, "q8": L.q8, "scale": L.scale,
                "bits": L.bits, "err": st.err}
    if op == "decode":
        return bsq.bsq_decode(st.cfg, st.codec, st.layer, out=st.out)
    st.step += 1
    bsq.bsq_train_grad(st.cfg, st.hp, st.chunks, st.theta, idx=st.idx, grad=st.grad, loss=st.loss, ws=st.ws)
    bsq.bsq_train_adam(st.cfg, st.hp, st.step, st.theta, st.grad, st.m, st.v)
    return {"grad": st.grad, "loss": st.loss, "theta": st.theta, "m": st.m, "v": st.v}


# ---------------------------------------------------------------- work, tolerance, 64-bit results
def _stored_bytes(c, d_out, d_in):
    """Code and gain planes, protected bytes, scales, indices and bitmap."""
    k = _k(c, d_in)
    n = d_out * (d_in // c["d"]) * c["stages"] * (2 + (c["d"] // 8))
    return n + (d_out * k + 8 * k + d_in // 8 if k else 0)


def work(case):
    c = case
    es = 4 if c["dtype"] == "fp32" else 2
    if c["op"] in ("gemv", "gemm"):
        M = c.get("M", 1)
        nb = fl = 0
        for group in _groups(c):
            nb += M * group[0][1] * es
            for d_out, d_in in group:
                nb += _stored_bytes(c, d_out, d_in) + M * d_out * es + 2 * c["lora"] * (d_out + d_in)
                fl += 2 * M * (d_out * d_in + c["lora"] * (d_out + d_in))
        return {"bytes": nb, "flops": fl}
    d_out, d_in = _dims(c)
    n = c["mats"] * d_out * d_in
    if c["op"] == "train":
        d, b, h, N = c["d"], c["b"], c["b"], c["n"]
        return {"bytes": N * (8 + es * d) + 28 * (b * d + h * b + h + d * h + d),
                "flops": 6 * N * (b * d + h * b + d * h)}
    # encode: per weight and stage the two sums of the gain and the residual; decode: one multiply-add
    per = 6 if c["op"] == "encode" else 2
    return {"bytes": n * es + c["mats"] * _stored_bytes(c, d_out, d_in), "flops": per * c["stages"] * n}


def tolerance(case):
    """encode and decode are bit-exact by definition. The bf16 products round
    decoded values or weights to bf16 and their outputs to bf16; the fp32
    product and the training step keep 32-bit sums."""
    c = case
    if c["op"] in ("encode", "decode"):
        return "exact"
    if c["op"] == "train":
        return {"rel": 2e-5, "max": 1e-3}
    if c["dtype"] == "fp32":
        return {"rel": 2e-6, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.1}


def _exact_train(c, seed):
    """One step in fp64: the straight-through loss, its gradient and Adam."""
    st = prepare(c, seed)
    b, d, h, hp = c["b"], c["d"], c["b"], bsq.TrainHyper()
    th = st.theta.double().requires_grad_()
    E, W1, b1, W2, b2 = torch.split(th, [b * d, h * b, h, d * h, d])
    x = st.chunks.view(-1, d)[st.idx].double()
    z = x @ E.view(b, d).T
    nz = z.norm(dim=1, keepdim=True)
    u = torch.where(nz > 0, z / nz.clamp_min(1e-300), torch.zeros_like(z))
    q = torch.where(z >= 0, 1.0, -1.0).double() / math.sqrt(b)
    a = torch.relu((u + (q - u).detach()) @ W1.view(h, b).T + b1)
    xh = a @ W2.view(d, h).T + b2
    H = lambda s: -(s * s.log() + (1 - s) * (1 - s).log())  # noqa: E731
    s = torch.sigmoid(2 * hp.tau * u / math.sqrt(b))
    rec, com = (xh - x).square().sum(1).mean(), (u - q).square().sum(1).mean()
    ent = H(s).sum(1).mean() - hp.gamma * H(s.mean(0)).sum()
    loss = rec + hp.lambda_c * com + hp.lambda_e * ent
    g, = torch.autograd.grad(loss, th)
    m, v = (1 - hp.beta1) * g, (1 - hp.beta2) * g * g
    theta = th.detach() - hp.lr * (m / (1 - hp.beta1)) / ((v / (1 - hp.beta2)).sqrt() + hp.eps)
    return {"grad": g, "loss": torch.stack([loss, rec, com, ent]).detach(), "theta": theta, "m": m, "v": v}


def exact(case, seed):
    c = case
    if c["op"] == "train":
        return _exact_train(c, seed)
    if c["op"] in ("gemv", "gemm"):
        outs = []
        for x, mem in _members(c, seed):
            ys = []
            for W, decs, lora in mem:
                X = x.double()
                y = X @ _decoded(c, W, _tables(c, decs)).T
                if lora is not None:
                    y = y + (X @ lora[0].double().T) @ lora[1].double().T
                ys.append(y)
            outs.append(ys)
        return outs if c["op"] == "gemv" else [ys[0] for ys in outs]
    d_out, d_in = _dims(c)
    W = _weight(c, _gen(seed, 31), c["mats"], d_out, d_in)
    tabs = _tables(c, _decoders(c, seed))
    if c["op"] == "decode":
        out = torch.stack([_decoded(c, W[m], tabs) for m in range(c["mats"])])
        return out if c["mats"] > 1 else out[0]
    # encode: the first stage's gains and the scales; later stages code the
    # rounded residual, so they have no value of their own in 64 bits
    gains, scales = [], []
    for m in range(c["mats"]):
        w = W[m].double()
        keep = torch.ones(d_in, device=DEV, dtype=torch.float64)
        if c["protect"]:
            idx = w.square().sum(0).topk(_k(c, d_in)).indices.sort().values
            keep[idx] = 0
            scales.append(w[:, idx].abs().amax(0) / PAYLOAD_MAX[c["fmt"]])
        r, kc = (w * keep).view(d_out, -1, c["d"]), keep.view(1, -1, c["d"])
        code = ((r >= 0).int() << torch.arange(c["d"], device=DEV)).sum(-1)
        y = tabs[0][code.long()] * kc
        gains.append(_tiled(c, torch.nan_to_num((r * y).sum(-1) / y.square().sum(-1), 0.0, 0.0, 0.0)))
    one = lambda v: torch.stack(v) if c["mats"] > 1 else v[0]  # noqa: E731
    none = [None] * (c["stages"] - 1)
    return {"codes": [None] * c["stages"], "gains": [one(gains)] + none, "idx": None, "q8": None,
            "scale": one(scales) if scales else None, "bits": None, "err": None}
