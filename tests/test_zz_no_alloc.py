"""proxy_decode_step_static, the decode step that allocates nothing, against
proxy_decode_step with a caller workspace (through the C ABI).

Two sessions decode the same tokens from the same state, one through each
entry point; outputs, counters and caches must be bit-identical (the two
share every kernel). Two calls in a row, the second on a smaller shape
(fewer sequences, narrower model, shorter cache), each starting two tokens
before the end of a block, so a step appends a block through the static
scratch too. The static scratch keeps the previous call's contents, so the
second call also shows that nothing in it needs clearing.
"""
import numpy as np
import pytest

from paper_2608_23463_amd import synth
from paper_2608_23463_amd.synth import DecodeShape
from helpers import dev, dev_weights
from test_gpu_decode import make_session

pytestmark = pytest.mark.gpu

CALLS = [
    ("32 x 1024, 16,384 rows", DecodeShape(32, 1024, 16, 64, (64,), n0=16384, steps=3)),
    ("3 x 256, 2,000 rows", DecodeShape(3, 256, 4, 64, (16,), n0=2000, steps=3)),
]


def test_static_scratch_step_matches_workspace_step(gpu):
    import torch
    for label, shape in CALLS:
        print(f"[no-alloc decode] {label}", flush=True)
        inp = synth.decode_inputs(shape, 9000 + shape.batch)
        a = make_session(shape, inp)
        b = make_session(shape, inp)
        j0 = shape.block - 2
        rng = np.random.default_rng(shape.batch)
        for name in ("x_blk", "k_loc", "v_loc"):
            slots = getattr(a, name)
            full = synth.bf16_round(rng.standard_normal(tuple(slots.shape)).astype(np.float32))
            val = dev(full, shape.dtype)
            getattr(a, name).copy_(val)
            getattr(b, name).copy_(val)
        a.state.j = b.state.j = j0
        for t in range(shape.steps):
            x_t = dev(inp["x"][t], shape.dtype)
            ya = a.step(x_t)
            yb = b.step_static(x_t)
            torch.cuda.synchronize()
            assert torch.equal(ya, yb), (label, t)
        assert (a.n, a.j) == (b.n, b.j) == (shape.n0 + 1, (j0 + shape.steps) % shape.block)
        n = a.n
        assert torch.equal(a.k_cache[:, :, :n], b.k_cache[:, :, :n]), label
        assert torch.equal(a.v_cache[:, :, :n], b.v_cache[:, :, :n]), label


def test_static_step_past_the_full_plans_scratch(gpu):
    """512 sequences of 32 heads over 2,000 rows: the partials of the short
    slices alone take more than the 64 MiB, so the step takes the plan with
    less scratch, through either entry point: outputs and appended rows are
    bit-identical, as they are over 100 rows, where the full plan fits."""
    import torch
    B = gpu
    nb, nh, d, p = 512, 32, 2048, 4
    w = dev_weights(synth.decode_inputs(DecodeShape(1, d, nh, 64, (p,), n0=0, steps=1), 9100)["weights"], "bf16")
    gen = torch.Generator(device="cuda").manual_seed(9101)

    def rnd(*s):
        return torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)

    blk, kl, vl, xs = rnd(nb, p, d), rnd(nb, nh, p, 64), rnd(nb, nh, p, 64), rnd(3, nb, d)
    for n in (2000, 100):
        kc, vc = rnd(nb, nh, n + 2, 64), rnd(nb, nh, n + 2, 64)
        out = []
        for static in (False, True):
            s = B.DecodeSession(B.decode_config(nb, d, nh, 64, (p,)), w, kc.clone(), vc.clone(), n=n)
            s.x_blk.copy_(blk)
            s.k_loc.copy_(kl)
            s.v_loc.copy_(vl)
            s.state.j = p - 2
            print(f"[no-alloc decode] 512 x 2048, n = {n}, static {static}", flush=True)
            ys = [(s.step_static if static else s.step)(xs[t]) for t in range(3)]
            torch.cuda.synchronize()
            out.append((torch.stack(ys), s.k_cache, s.v_cache))
        for a, b in zip(*out):
            assert torch.equal(a, b), n


def test_static_step_appends_in_passes(gpu):
    """19 sequences with blocks of 2,000 tokens: the append's partials and
    level outputs do not fit beside each other, so without a workspace it runs
    in passes of a few blocks, cut along K as the whole batch is: bit-identical."""
    import torch
    B = gpu
    nb, nh, dh, factors = 19, 7, 128, (4, 100, 5)
    d, p, n = nh * dh, 2000, 11
    gen = torch.Generator(device="cuda").manual_seed(9102)

    def rnd(*s, std=1.0):
        return torch.randn(s, generator=gen, device="cuda") * std

    lin = lambda o, i: (rnd(o, i, std=0.02), rnd(o, std=0.02))
    w = {"rms_gamma": torch.ones(d, device="cuda"), "alpha": lin(nh, d), "compress": [lin(d, k * d) for k in factors]}
    for name in ("q", "k", "v", "o", "k_proxy", "v_proxy"):
        w[name] = lin(d, d)
    kc, vc, xs = rnd(nb, nh, n + 2, dh), rnd(nb, nh, n + 2, dh), rnd(3, nb, d)
    blk, kl, vl = rnd(nb, p, d), rnd(nb, nh, p, dh), rnd(nb, nh, p, dh)
    out = []
    for static in (False, True):
        print(f"[no-alloc decode] 19 x 896 fp32, blocks of 2,000, static {static}", flush=True)
        s = B.DecodeSession(B.decode_config(nb, d, nh, dh, factors, dtype="fp32"), w, kc.clone(), vc.clone(), n=n)
        s.x_blk.copy_(blk)
        s.k_loc.copy_(kl)
        s.v_loc.copy_(vl)
        s.state.j = p - 2
        ys = [(s.step_static if static else s.step)(xs[t]) for t in range(3)]
        torch.cuda.synchronize()
        out.append((torch.stack(ys), s.k_cache, s.v_cache))
    for a, b in zip(*out):
        assert torch.isfinite(a).all() and torch.equal(a, b)
