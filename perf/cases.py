"""The calls whose time matters to a user of this library, as measurable cases.

A case is a dict of plain values. `kind` says which entry points a pass calls:

  layer    binding.layer_forward (inference: no saved activations)
  train    binding.layer_forward(save=True), then binding.layer_backward
  decode   binding.DecodeSession.step, once per token of one whole block
           (the last of these steps appends the block to the proxy cache)
  prefill  binding.DecodeSession.prefill over the next T tokens

Sizes are the workloads of this repository's synth.py, its tests' ragged and
image shapes, and generic ones between them. Weights are N(0, 0.02^2) as in
those workloads, biases likewise, activations and upstream gradients N(0, 1),
and a cache holds rows of the size that the model's own append writes.
"""
import math

import torch

from paper_2608_23463_amd import binding as B

STD = 0.02
EPS = 1e-6
TOKEN_CAUSAL, BLOCK_CAUSAL, BIDIRECTIONAL = 0, 1, 2
GATED, ADD, AFFINE, GATED_HEAD = 0, 1, 2, 3


def _layer(name, kind, batch, seq, d_fine, d_proxy, head_dim, factors, dtype="bf16", mask=TOKEN_CAUSAL,
           injection=GATED, image=0, extended=True, stacked=False):
    c = {"kind": kind, "batch": batch, "seq": seq, "d_fine": d_fine, "d_proxy": d_proxy, "head_dim": head_dim,
         "factors": factors, "dtype": dtype, "mask": mask, "injection": injection, "image": image,
         "extended": extended, "stacked": stacked}
    return dict(c, name=name) if name else c


def _gen(name, kind, batch, d, head_dim, factors, n0, tokens, dtype="bf16", ragged=False):
    c = {"kind": kind, "batch": batch, "d": d, "head_dim": head_dim, "factors": factors, "n0": n0,
         "tokens": tokens, "dtype": dtype, "ragged": ragged}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a million-token document through one layer: the headline workload
        _layer("layer_1M_d1024", "layer", 1, 1 << 20, 1024, 1024, 64, "64"),
        # the same layer at an ordinary long-context length, in the plain bf16
        # arithmetic that the model is trained in
        _layer("layer_64k_d1024", "layer", 1, 65536, 1024, 1024, 64, "64", extended=False),
        # the language model's history stream: 64-wide tokens, 512-wide proxies
        _layer("layer_1M_lm", "layer", 1, 1 << 20, 64, 512, 64, "64"),
        # a short text in single precision (evaluation against another implementation)
        _layer("layer_4k_fp32", "layer", 1, 4096, 256, 256, 64, "64", dtype="fp32"),
        # a small vision batch: 32 x 32 images in 4 x 4 patches, seen both ways,
        # one training step of a layer
        _layer("train_image_64x32x32", "train", 64, 1024, 192, 192, 64, "16", mask=BIDIRECTIONAL, image=32),
        # training step of a layer in the middle of a stack, on a batch of
        # texts whose length is no multiple of the block
        _layer("train_4x5000_d512", "train", 4, 5000, 512, 512, 64, "64", stacked=True),
        # long-context training step of the wide factorised layer
        _layer("train_256k_d2048", "train", 1, 1 << 18, 2048, 2048, 128, "8x8"),
        # batch serving against long caches: 64 tokens of 32 sequences, one block
        _gen("decode_B32_n16k", "decode", 32, 1024, 64, "64", 16384, 64),
        # one interactive user in the middle of a conversation
        _gen("decode_B1_n1500", "decode", 1, 512, 64, "64", 1500, 64),
        # continuous batching: sequences of many lengths, each at its own position
        _gen("decode_ragged_B12", "decode", 12, 1024, 64, "8x8", 6000, 64, ragged=True),
        # the next 4,096 tokens of a batch against its long caches
        _gen("prefill_B32_T4096", "prefill", 32, 1024, 64, "64", 16384, 4096),
        # a short prompt of one user, nothing cached yet
        _gen("prefill_B1_T700", "prefill", 1, 512, 64, "64", 0, 700),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _seconds(case):
    """A rough cost, the same for every implementation, to bound the draws."""
    w = work(case)
    return w["flops"] / (1e15 if case["dtype"] == "bf16" else 1e14) + w["bytes"] / 5e12


def draw(rng):
    most = max(_seconds(c) for c in listed())
    while True:
        dtype = "fp32" if rng.random() < 0.15 else "bf16"
        what = rng.choice(["layer", "layer", "train", "train", "image", "decode", "decode", "ragged", "prefill",
                           "prefill"])
        head_dim = rng.choice([64, 64, 128])
        factors = rng.choice(["16", "32", "64", "64", "128", "4x4", "8x8", "4x16"])
        p = _block(factors)
        if what == "image":
            side = rng.choice([2, 4, 8])
            w, h = side * rng.randint(3, 40), side * rng.randint(3, 40)
            d = 64 * rng.randint(2, 12)
            c = _layer(None, rng.choice(["layer", "train"]), _log(rng, 1, 64), w * h, d, d, 64, str(side * side),
                       dtype, rng.choice([BIDIRECTIONAL, BLOCK_CAUSAL]), GATED, w)
            tokens, ok = c["batch"] * w * h, side > 2 or w * h <= 4096
        elif what in ("layer", "train"):
            dp = head_dim * rng.randint(2, 16)
            df = rng.choice([dp, dp, 64, 8 * rng.randint(8, 128)])
            batch = _log(rng, 1, 8)
            c = _layer(None, what, batch, _log(rng, 500, (1 << 20) // batch), df, dp, head_dim, factors, dtype,
                       rng.choice([TOKEN_CAUSAL, TOKEN_CAUSAL, BLOCK_CAUSAL]),
                       rng.choice([GATED, GATED, GATED, ADD, AFFINE]), 0, rng.random() < 0.7, rng.random() < 0.5)
            tokens, ok = batch * c["seq"], c["seq"] <= 32768 * p and (what == "layer" or c["seq"] <= 8192 * p)
        else:
            d = head_dim * rng.randint(2, 16 if head_dim == 64 else 8)
            batch = _log(rng, 1, 48)
            n0 = 0 if rng.random() < 0.15 else _log(rng, 30, 16384)
            tokens = p if what != "prefill" else _log(rng, 40, 4096)
            c = _gen(None, "prefill" if what == "prefill" else "decode", batch, d, head_dim, factors, n0, tokens,
                     dtype, what == "ragged" and n0 > 0)
            tokens, ok = batch * tokens, batch * d * n0 <= 32 * 1024 * 16384
        if ok and tokens <= (1 << 20 if dtype == "bf16" else 1 << 15) and _seconds(c) <= most:
            return c


# ---------------------------------------------------------------- sizes

def _factors(case_or_text):
    t = case_or_text if isinstance(case_or_text, str) else case_or_text["factors"]
    return [int(k) for k in t.split("x")]


def _block(factors):
    return math.prod(_factors(factors))


def _dims(case, fine, proxy):
    """Widths d_0 .. d_M of the compression levels."""
    return [fine] + [proxy] * len(_factors(case))


def _work_layer(c):
    es = 2 if c["dtype"] == "bf16" else 4
    ks, df, dp = _factors(c), c["d_fine"], c["d_proxy"]
    m = -(-c["seq"] // _block(c["factors"]))
    tok, rows = c["batch"] * c["seq"], c["batch"] * m
    d = _dims(c, df, dp)
    nh = dp // c["head_dim"]
    wts = 4 * dp * dp
    flops = 2 * 4 * rows * dp * dp
    r = rows
    for j in reversed(range(len(ks))):  # level j + 1 has r rows
        wts += 2 * ks[j] * d[j] * d[j + 1]
        flops += 2 * 2 * r * ks[j] * d[j] * d[j + 1]
        r *= ks[j]
    pairs = m * m if c["mask"] == BIDIRECTIONAL else m * (m + 1) // 2
    flops += 4 * c["batch"] * pairs * dp
    gate = {GATED: df * 2 * df, ADD: 0, AFFINE: 2 * df * df, GATED_HEAD: nh * 2 * df}[c["injection"]]
    wts += gate
    flops += 2 * tok * gate
    byt = es * (2 * tok * df + rows * dp * (2 if c["stacked"] else 1) + wts)
    if c["kind"] == "train":  # twice the products, the gradients in and out, fp32 weight gradients
        flops *= 3
        byt += es * (2 * tok * df + rows * dp * (2 if c["stacked"] else 0) + wts) + 4 * wts
    return {"bytes": byt, "flops": flops}


def _lengths(c):
    """Cached rows of every sequence at the start of the pass."""
    if not c["ragged"]:
        return [c["n0"]] * c["batch"]
    return [max(1, c["n0"] * (b * 7 % c["batch"] + 1) // c["batch"]) for b in range(c["batch"])]


def _slots(c):
    """Filled slots of the current block at the start of the pass."""
    p = _block(c["factors"])
    return [b * 5 % p if c["ragged"] else 0 for b in range(c["batch"])]


def _work_gen(c):
    es = 2 if c["dtype"] == "bf16" else 4
    d, bsz, p = c["d"], c["batch"], _block(c["factors"])
    ks, dd = _factors(c), _dims(c, d, d)
    t, nh = c["tokens"], c["d"] // c["head_dim"]
    blocks = bsz * (t // p)
    comp_w = sum(k * a * b for k, a, b in zip(ks, dd, dd[1:]))
    flops = 2 * bsz * t * d * (4 * d + nh) + 2 * blocks * 2 * d * d
    r = blocks
    for j in reversed(range(len(ks))):
        flops += 2 * r * ks[j] * dd[j] * dd[j + 1]
        r *= ks[j]
    w_step, w_app = 4 * d * d + nh * d, comp_w + 2 * d * d
    if c["kind"] == "prefill":
        seen = bsz * sum(c["n0"] + i // p + i % p + 1 for i in range(t))
        flops += 4 * d * seen
        byt = es * (2 * bsz * t * d + 2 * bsz * c["n0"] * d + w_step + w_app + 2 * blocks * d)
    else:
        rows = t * sum(_lengths(c)) + bsz * t * (p + 1) // 2  # every step reads the cache and the block so far
        flops += 4 * d * rows
        byt = es * (2 * d * rows + 2 * bsz * t * d + t * w_step + w_app + 2 * blocks * d)
    return {"bytes": byt, "flops": flops}


def work(case):
    return _work_layer(case) if case["kind"] in ("layer", "train") else _work_gen(case)


# ---------------------------------------------------------------- inputs

class _Draw:
    """Normal samples from one seed, made on the GPU in the case's type."""

    def __init__(self, case, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        self.dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def __call__(self, *shape, std=1.0):
        return torch.empty(shape, dtype=self.dtype, device="cuda").normal_(0.0, std, generator=self.gen)

    def linear(self, out, inp):
        return self(out, inp, std=STD), self(out, std=STD)


def _layer_inputs(c, seed):
    dr = _Draw(c, seed)
    ks, df, dp = _factors(c), c["d_fine"], c["d_proxy"]
    d = _dims(c, df, dp)
    m = -(-c["seq"] // _block(c["factors"]))
    w = {"compress": [dr.linear(d[j + 1], ks[j] * d[j]) for j in range(len(ks))]}
    for name in "qkvo":
        w[name] = dr.linear(dp, dp)
    w["decompress"] = [dr.linear(ks[j] * d[j], d[j + 1]) for j in range(len(ks))]
    if c["injection"] == GATED:
        w["gate"] = dr.linear(df, 2 * df)
    elif c["injection"] == GATED_HEAD:
        w["gate"] = dr.linear(dp // c["head_dim"], 2 * df)
    elif c["injection"] == AFFINE:
        w["affine"] = dr.linear(2 * df, df)
    s = {"weights": w, "x": dr(c["batch"], c["seq"], df), "h_in": None, "dy": None, "dh_out": None}
    if c["stacked"]:
        s["h_in"] = dr(c["batch"], m, dp)
    if c["kind"] == "train":
        s["dy"] = dr(c["batch"], c["seq"], df)
        if c["stacked"]:
            s["dh_out"] = dr(c["batch"], m, dp)
    return s


def _gen_inputs(c, seed):
    dr = _Draw(c, seed)
    ks, d, p = _factors(c), c["d"], _block(c["factors"])
    dd = _dims(c, d, d)
    nh, dh = d // c["head_dim"], c["head_dim"]
    w = {"rms_gamma": 1.0 + dr(d, std=0.1)}
    for name in "qkvo":
        w[name] = dr.linear(d, d)
    w["alpha"] = dr.linear(nh, d)
    w["compress"] = [dr.linear(dd[j + 1], ks[j] * dd[j]) for j in range(len(ks))]
    w["k_proxy"], w["v_proxy"] = dr.linear(d, d), dr.linear(d, d)
    # rows as the append writes them: the spread of a chain of N(0, 0.02^2) maps
    std = math.prod(STD * math.sqrt(k * a) for k, a in zip(ks, dd)) * STD * math.sqrt(d)
    n_cap = c["n0"] + c["tokens"] // p + 2
    s = {"weights": w}
    for name in ("k_cache", "v_cache"):
        s[name] = torch.zeros((c["batch"], nh, n_cap, dh), dtype=dr.dtype, device="cuda")
        s[name][:, :, :c["n0"]] = dr(c["batch"], nh, c["n0"], dh, std=min(std, 4.0))
    # decode: one [B, d] row block per step; prefill: the chunk
    s["x"] = dr(c["tokens"], c["batch"], d) if c["kind"] == "decode" else dr(c["batch"], c["tokens"], d)
    if c["ragged"]:  # the slots that are filled already
        s["blk"] = [dr(c["batch"], p, d), dr(c["batch"], nh, p, dh), dr(c["batch"], nh, p, dh)]
    return s


def prepare(case, seed):
    if case["kind"] in ("layer", "train"):
        s = _layer_inputs(case, seed)
        s["cfg"] = B.layer_config(case["batch"], case["seq"], case["d_fine"], case["d_proxy"],
                                  case["d_proxy"] // case["head_dim"], case["head_dim"], _factors(case), (),
                                  case["dtype"], case["mask"], case["injection"], case["image"],
                                  B.PF_PRECISION_EXTENDED if case["extended"] else B.PF_PRECISION_BF16)
    else:
        s = _gen_inputs(case, seed)
        cfg = B.decode_config(case["batch"], case["d"], case["d"] // case["head_dim"], case["head_dim"],
                              _factors(case), (), case["dtype"], EPS)
        s["session"] = ses = B.DecodeSession(cfg, s["weights"], s["k_cache"], s["v_cache"], n=case["n0"],
                                             ragged=case["ragged"], n_seq=_lengths(case), j_seq=_slots(case))
        s["y"] = torch.empty_like(s["x"])
        if case["ragged"]:
            for t, v in zip((ses.x_blk, ses.k_loc, ses.v_loc), s["blk"]):
                t.copy_(v)
            s["lengths"], s["slots"] = _lengths(case), _slots(case)
            # where each sequence's block lands: one row at its own length
            s["appended"] = (torch.arange(case["batch"], device="cuda"), slice(None),
                             torch.tensor(s["lengths"], device="cuda"))
    s["case"] = case
    return s


# ---------------------------------------------------------------- a pass

def run(s):
    c = s["case"]
    if c["kind"] == "layer":
        x_out, h_out, _ = B.layer_forward(s["cfg"], s["weights"], s["x"], s["h_in"])
        return {"x_out": x_out, "h_out": h_out}
    if c["kind"] == "train":
        x_out, h_out, saved = B.layer_forward(s["cfg"], s["weights"], s["x"], s["h_in"], save=True)
        dx, dh_in, grads = B.layer_backward(s["cfg"], s["weights"], s["x"], s["h_in"], saved, s["dy"], s["dh_out"])
        # the key bias moves every logit of a row alike, so its gradient is
        # zero and what comes back is the rounding of terms that cancel
        grads["k"] = (grads["k"][0],)
        return {"x_out": x_out, "h_out": h_out, "dx": dx, "dh_in": dh_in, "grads": grads}
    ses = s["session"]
    # the cache as it was before the block: its rows below n0 are only read
    if c["ragged"]:
        ses.n_seq[:] = s["lengths"]
        ses.j_seq[:] = s["slots"]
    else:
        ses.state.n, ses.state.j = c["n0"], 0
    new = slice(c["n0"], c["n0"] + c["tokens"] // ses.x_blk.shape[1])  # the rows that are appended
    if c["kind"] == "prefill":
        ses.prefill(s["x"], s["y"])
        left = c["tokens"] % ses.x_blk.shape[1]  # tokens of an unfinished block stay in the local slots
        return {"y": s["y"], "k_loc": ses.k_loc[:, :, :left], "v_loc": ses.v_loc[:, :, :left],
                "k_rows": s["k_cache"][:, :, new], "v_rows": s["v_cache"][:, :, new]}
    for t in range(c["tokens"]):
        ses.step(s["x"][t], s["y"][t])
    at = s["appended"] if c["ragged"] else (slice(None), slice(None), new)
    return {"y": s["y"], "k_loc": ses.k_loc, "v_loc": ses.v_loc, "k_rows": s["k_cache"][at], "v_rows": s["v_cache"][at]}


# ---------------------------------------------------------------- in 64 bits

def _f64(v):
    if isinstance(v, torch.Tensor):
        return v.double()
    if isinstance(v, dict):
        return {k: _f64(x) for k, x in v.items()}
    if isinstance(v, (list, tuple)):
        return [_f64(x) for x in v]
    return v


def _lin(x, wb):
    return torch.nn.functional.linear(x, wb[0], wb[1])


def _attend(q, k, v, causal):
    """softmax(q k^T / sqrt(dh)) v of one head, in chunks of query rows."""
    out = []
    for r0 in range(0, q.shape[0], 4096):
        qc = q[r0:r0 + 4096]
        keys = r0 + qc.shape[0] if causal else k.shape[0]
        sc = qc @ k[:keys].T / math.sqrt(q.shape[1])
        if causal:
            rows = torch.arange(r0, r0 + qc.shape[0], device=q.device)[:, None]
            sc = sc.masked_fill(torch.arange(keys, device=q.device)[None, :] > rows, -math.inf)
        out.append(torch.softmax(sc, -1) @ v[:keys])
    return torch.cat(out)


def _patches(x, w, p, back):
    """Raster order <-> patch order of [L, d] tokens of a w-wide image."""
    h = x.shape[0] // w
    shape = (h // p, w // p, p, p, x.shape[1]) if back else (h // p, p, w // p, p, x.shape[1])
    return x.reshape(shape).permute(0, 2, 1, 3, 4).reshape(x.shape)


def _exact_sequence(c, w, x, h_in):
    ks, dh, L = _factors(c), c["head_dim"], x.shape[0]
    p = math.prod(ks)
    side = math.isqrt(p)
    if c["image"]:
        x = _patches(x, c["image"], side, False)
    elif L % p:
        x = torch.cat([x, x.new_zeros(p - L % p, x.shape[1])])
    z = x
    for k, wb in zip(ks, w["compress"]):
        z = _lin(z.reshape(z.shape[0] // k, -1), wb)
    h = z if h_in is None else h_in + z
    q, k, v = (_lin(h, w[n]) for n in "qkv")
    o = torch.cat([_attend(q[:, i:i + dh], k[:, i:i + dh], v[:, i:i + dh], c["mask"] != BIDIRECTIONAL)
                   for i in range(0, h.shape[1], dh)], 1)
    u = _lin(o, w["o"])
    if c["mask"] == TOKEN_CAUSAL:
        u = torch.cat([torch.zeros_like(u[:1]), u[:-1]])
    for j in reversed(range(len(ks))):
        u = _lin(u, w["decompress"][j]).reshape(u.shape[0] * ks[j], -1)
    if c["injection"] == ADD:
        y = x + u
    elif c["injection"] == AFFINE:
        st = _lin(u, w["affine"])
        d = x.shape[1]
        y = (1 + st[:, :d]) * x * torch.rsqrt((x * x).mean(1, keepdim=True) + EPS) + st[:, d:]
    else:
        g = torch.sigmoid(_lin(torch.cat([x, u], 1), w["gate"]))
        y = x + g.repeat_interleave(x.shape[1] // g.shape[1], 1) * u
    return (_patches(y, c["image"], side, True) if c["image"] else y[:L]), h


def _exact_layer(c, seed):
    s = _f64(_layer_inputs(c, seed))
    train = c["kind"] == "train"
    w = s["weights"]
    flat = [t for v in w.values() for wb in (v if isinstance(v[0], (list, tuple)) else [v]) for t in wb]
    ins = [s["x"]] + ([s["h_in"]] if c["stacked"] else [])
    if train:
        for t in flat + ins:
            t.requires_grad_()
    xs, hs = [], []
    with torch.set_grad_enabled(train):
        for b in range(c["batch"]):
            y, h = _exact_sequence(c, w, s["x"][b], s["h_in"][b] if c["stacked"] else None)
            if train:  # one sequence at a time, the gradients add up
                loss = (y * s["dy"][b]).sum() + ((h * s["dh_out"][b]).sum() if c["stacked"] else 0.0)
                loss.backward()
            xs.append(y.detach())
            hs.append(h.detach())
    out = {"x_out": torch.stack(xs), "h_out": torch.stack(hs)}
    if train:
        def grad(v):
            return [grad(t) for t in v] if isinstance(v, (list, tuple)) else v.grad
        g = {n: grad(v) for n, v in w.items()}
        g["k"] = (g["k"][0],)
        g.setdefault("gate", None)
        g.setdefault("affine", None)
        out.update(dx=s["x"].grad, dh_in=s["h_in"].grad if c["stacked"] else None, grads=g)
    return out


def _exact_gen(c, seed):
    s = _f64(_gen_inputs(c, seed))
    w, p, ks = s["weights"], _block(c["factors"]), _factors(c)
    bsz, d, dh = c["batch"], c["d"], c["head_dim"]
    nh, T = d // dh, c["tokens"]
    x = s["x"].transpose(0, 1) if c["kind"] == "decode" else s["x"]  # [B, T, d]
    kc, vc = s["k_cache"], s["v_cache"]
    k_loc, v_loc = (s["blk"][1:] if c["ragged"] else [x.new_zeros(bsz, nh, p, dh) for _ in range(2)])
    lengths, slots = _lengths(c), _slots(c)
    y = torch.empty_like(x)
    for b in range(bsz):
        n0, j0 = lengths[b], slots[b]
        u = x[b] * torch.rsqrt((x[b] * x[b]).mean(1, keepdim=True) + EPS) * w["rms_gamma"]
        q, k, v = (_lin(u, w[n]).reshape(T, nh, dh).transpose(0, 1) for n in "qkv")
        al = torch.sigmoid(_lin(u, w["alpha"]))
        # the tokens from the start of the current block on
        xb = torch.cat([s["blk"][0][b, :j0], x[b]]) if c["ragged"] else x[b]
        k = torch.cat([k_loc[b, :, :j0], k], 1)
        v = torch.cat([v_loc[b, :, :j0], v], 1)
        full = xb.shape[0] // p
        z = xb[:full * p]
        for f, wb in zip(ks, w["compress"]):
            z = _lin(z.reshape(z.shape[0] // f, -1), wb) if full else z
        for cache, n in ((kc, "k_proxy"), (vc, "v_proxy")):
            if full:
                cache[b, :, n0:n0 + full] = _lin(z, w[n]).reshape(full, nh, dh).transpose(0, 1)
        a = torch.empty(T, nh, dh, dtype=x.dtype, device=x.device)
        pos = torch.arange(j0, j0 + T, device=x.device)
        own = torch.arange(k.shape[1], device=x.device)[None, :]
        rows = torch.arange(n0 + full, device=x.device)[None, :]
        hide_own = (own > pos[:, None]) | (own < (pos // p * p)[:, None])
        hide_row = rows >= n0 + (pos // p)[:, None]
        for h in range(nh):
            sc = (q[h] @ k[h].T / math.sqrt(dh)).masked_fill(hide_own, -math.inf)
            a[:, h] = torch.softmax(sc, 1) @ v[h]
            if n0 + full:
                sc = (q[h] @ kc[b, h, :n0 + full].T / math.sqrt(dh)).masked_fill(hide_row, -math.inf)
                mx = sc.max(1, keepdim=True).values
                e = torch.exp(sc - torch.where(mx.isfinite(), mx, torch.zeros_like(mx)))
                a[:, h] += al[:, h:h + 1] * ((e @ vc[b, h, :n0 + full]) / e.sum(1, keepdim=True).clamp_min(1e-300))
        y[b] = x[b] + _lin(a.reshape(T, d), w["o"])
        for t in range(max(0, T - p), T):  # what the local slots hold afterwards
            k_loc[b, :, (j0 + t) % p], v_loc[b, :, (j0 + t) % p] = k[:, j0 + t], v[:, j0 + t]
    new = slice(c["n0"], c["n0"] + T // p)
    if c["ragged"]:
        at = torch.arange(bsz, device=x.device), slice(None), torch.tensor(lengths, device=x.device)
    else:
        at = slice(None), slice(None), new
    if c["kind"] == "decode":
        return {"y": y.transpose(0, 1), "k_loc": k_loc, "v_loc": v_loc, "k_rows": kc[at], "v_rows": vc[at]}
    return {"y": y, "k_loc": k_loc[:, :, :T % p], "v_loc": v_loc[:, :, :T % p], "k_rows": kc[at], "v_rows": vc[at]}


def exact(case, seed):
    if case["kind"] in ("layer", "train"):
        return _exact_layer(case, seed)
    with torch.no_grad():
        return _exact_gen(case, seed)


def tolerance(case):
    """About four times the error against 64 bits that was measured over the
    listed and some 50 drawn cases (largest 2-norm / largest single value):
    fp32 5e-7 / 3e-6, its gradients 1.4e-6 / 9e-6; bf16 decode and prefill
    2.9e-3 / 1.3e-2; bf16 layers 3.4e-3 / 2.2e-2, with plain bf16 logits
    6.8e-3 / 0.1. Gradients inherit the rounding of sharp logits: 6.3e-3 / 4e-2
    where the layer is narrow, 2.3e-2 / 0.26 where it is wide or plain."""
    train = case["kind"] == "train"
    if case["dtype"] == "fp32":
        return {"rel": 6e-6, "max": 4e-5} if train else {"rel": 2e-6, "max": 1.2e-5}
    if case["kind"] in ("decode", "prefill"):
        return {"rel": 1.2e-2, "max": 5e-2}
    sharp = not case["extended"] or train and case["d_proxy"] > 1024
    if train:
        return {"rel": 3e-2, "max": 1.0} if sharp else {"rel": 2.5e-2, "max": 0.16}
    return {"rel": 2.7e-2, "max": 0.4} if sharp else {"rel": 1.4e-2, "max": 0.1}
