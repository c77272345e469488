"""GEMM launches and their epilogues: grouped launches, bias gradients formed inside the weight-gradient
GEMM, and the split-K reduction over lanes, at the sizes where they can go
wrong: widths at and just past the 128 and 256 tiles, one to a few proxies
against long reductions (many slices of few chunks), token counts that are no
multiple of the K step, and gradient sets with members left out."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2608_23463_amd import synth
from paper_2608_23463_amd.synth import LayerShape
from helpers import dev, dev_weights
from test_gpu_backward import compare, run_gpu_backward

pytestmark = pytest.mark.gpu

SHAPES = {
    # 128-wide operands: one tile per product, the narrowest fused bias sums
    "d128_rows37": LayerShape(1, 16 * 37, 128, 128, 2, 64, (16,)),
    # one chunk past a tile edge: the last tile holds 8 rows and 8 columns
    "d136_dp192": LayerShape(2, 8 * 61, 136, 192, 3, 64, (8,)),
    # past two 128 tiles, ragged tokens, a compression of 3 rows over K = 16,896
    "d264_dp256_m3": LayerShape(1, 64 * 2 + 5, 264, 256, 4, 64, (64,)),
    # the 256 tiles of long reductions: 16,640 token rows
    "d256_rows16k": LayerShape(1, 32 * 520, 256, 256, 2, 128, (32,), mask=synth.BLOCK_CAUSAL),
    # under the tiles: the register-path kernel and the column-sum passes
    "d72_dp64": LayerShape(2, 8 * 33, 72, 64, 1, 64, (8,)),
    # transposed per-head stores: runs of rows (m a multiple of 8, or one sequence)
    # with padding columns, and 2-byte stores (two sequences of 21 proxies)
    "cols_m24_B2": LayerShape(2, 8 * 24, 128, 128, 2, 64, (8,)),
    "cols_m37_B1": LayerShape(1, 8 * 37, 128, 128, 1, 128, (8,), mask=synth.BIDIRECTIONAL),
    "cols_m21_B2": LayerShape(2, 8 * 21, 128, 128, 2, 64, (8,)),
    # stores through the row map: a real tail of one token, patches of an odd grid
    "pad_tail1_B3": LayerShape(3, 8 * 9 + 1, 136, 128, 2, 64, (8,)),
    "pad_tail1_add": LayerShape(2, 8 * 9 + 1, 72, 64, 1, 64, (4, 2), injection=synth.INJECT_ADD),
    "affine_d144": LayerShape(1, 8 * 130, 144, 128, 2, 64, (8,), injection=synth.INJECT_AFFINE),
    "fp32_d136": LayerShape(1, 8 * 70, 136, 128, 2, 64, (8,), dtype="fp32"),
    "fp32_affine_rows8k": LayerShape(1, 16 * 520, 40, 64, 1, 64, (16,), dtype="fp32", injection=synth.INJECT_AFFINE),
}


@pytest.mark.parametrize("name", SHAPES)
def test_gradients_at_tile_edges(gpu, name):
    shape = SHAPES[name]
    print(f"[case {name}] {shape}", flush=True)
    inp = synth.layer_inputs(shape, 4100 + sorted(SHAPES).index(name), with_dy=True)
    res = run_gpu_backward(shape, inp)
    ref = oracle.layer_backward(inp["x"], inp["weights"], shape.factors, shape.n_heads, inp["dy"], shape.mask,
                                injection=shape.injection)
    compare(shape, inp, res, ref, name)


@pytest.mark.parametrize("missing", ["q", "k v o", "gate", "compress decompress"])
def test_gradients_left_out(gpu, missing):
    """A NULL dw skips that gradient; the others (and every bias gradient)
    equal the full call's bit for bit, within the workspace the size query gave."""
    import torch
    B = gpu
    shape = LayerShape(1, 64 * 20, 256, 256, 4, 64, (64,))
    print(f"[left out: {missing}]", flush=True)
    inp = synth.layer_inputs(shape, 4200, with_dy=True)
    cfg = B.config_from_shape(shape)
    w, x, dy = dev_weights(inp["weights"], "bf16"), dev(inp["x"], "bf16"), dev(inp["dy"], "bf16")
    _, _, saved = B.layer_forward(cfg, w, x, save=True)
    dx, _, full = B.layer_backward(cfg, w, x, None, saved, dy)

    def fresh(pair, drop):
        return tuple(None if drop and i == 0 else torch.full_like(t, float("nan")) for i, t in enumerate(pair))

    some = {}
    for key, val in full.items():
        drop = key in missing.split()
        some[key] = [fresh(p, drop) for p in val] if isinstance(val, list) else (fresh(val, drop) if val else None)
    dx2 = torch.full_like(dx, float("nan"))
    ws = torch.full((B.layer_workspace_size(cfg, True),), 255, dtype=torch.uint8, device="cuda")
    st = B.load().proxy_layer_backward(ctypes.byref(cfg), ctypes.byref(B.layer_weights(w)), x.data_ptr(), None,
                                       saved.data_ptr(), dy.data_ptr(), None, dx2.data_ptr(), None,
                                       ctypes.byref(B.layer_grads(some)), ws.data_ptr(), ws.numel(),
                                       torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st == B.PF_OK, B.last_error()
    assert torch.equal(dx, dx2)
    for key, val in full.items():
        for a, b in zip(val if isinstance(val, list) else [val or ()], some[key] if isinstance(val, list) else [some[key] or ()]):
            for i, (p, q) in enumerate(zip(a, b)):
                if q is None:
                    continue
                if i == 1 and key in missing.split():  # formed by its own column-sum pass
                    err = float((p - q).abs().max() / p.abs().max().clamp_min(1e-30))
                    assert np.isfinite(err) and (key == "k" or err <= 1e-4), (key, err)
                else:
                    assert torch.equal(p, q), (key, i)


@pytest.mark.parametrize("data", ["mean", "small after large"])
def test_bias_gradient_of_a_long_reduction(gpu, data):
    """Bias gradients formed inside the weight-gradient GEMM over K slices of
    8,192 rows, against the 64-bit column sums of the same bf16 values (with
    the additive injection the decompression's bias gradient is that of dY).
    A lane adds chains of at most 128 values, so the error of a sum of positive
    values is at most about 128 half-units in the last place: 128 * 2^-24 = 8e-6.
    One chain over the slice loses every 2^-20 that follows the 256s: 1.5e-5."""
    import torch
    B = gpu
    shape = LayerShape(1, 1 << 17, 1024, 1024, 16, 64, (2, 64), injection=synth.INJECT_ADD)
    gen = torch.Generator(device="cuda").manual_seed(5)
    std = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=gen)
    lin = lambda o, i: (std(o, i), std(o))
    w = {"compress": [lin(1024, 2048), lin(1024, 65536)], "decompress": [lin(2048, 1024), lin(65536, 1024)],
         **{n: lin(1024, 1024) for n in "qkvo"}}
    x = std(1, shape.seq_len, 1024)
    if data == "mean":
        dy = (1.0 + 5.0 * std(1, shape.seq_len, 1024).float()).to(torch.bfloat16)
    else:
        dy = torch.full((1, shape.seq_len, 1024), 2.0 ** -20, dtype=torch.bfloat16, device="cuda")
        dy[:, :32] = 0.0
        dy[:, :2] = dy[:, 16:18] = 256.0  # rows 0 and 8 of the [L / 2, 2 * 1024] operand
    cfg = B.config_from_shape(shape)
    _, _, saved = B.layer_forward(cfg, w, x, save=True)
    _, _, g = B.layer_backward(cfg, w, x, None, saved, dy)
    torch.cuda.synchronize()
    ref = dy.view(-1, 2048).double().sum(0)
    err = float(((g["decompress"][0][1].double() - ref).abs() / ref).max())
    print(f"  bias gradient over {shape.seq_len // 2} rows: {err:.2e}", flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("batch,tokens,heads", [(7, 610, 10), (1, 250, 8), (2, 1002, 8)])
def test_fp32_projections_error_of_short_chains(gpu, batch, tokens, heads):
    """fp32 Q, K and V in one launch: the K and V of a prefill's unfinished
    block against 64 bits. A sum of K products in chains of K / 2 is off by
    about 1.3e-8 sqrt(K) of the result (2-norms; 3.3e-7 measured at K = 640),
    one chain by sqrt(2) times that; the bound lies halfway."""
    import torch
    B = gpu
    d, p = heads * 64, 64
    gen = torch.Generator(device="cuda").manual_seed(4190 + tokens)

    def rnd(*shape, std=1.0):
        return torch.randn(shape, generator=gen, device="cuda") * std

    lin = lambda o, i: (rnd(o, i, std=0.05), torch.zeros(o, device="cuda"))
    w = {"rms_gamma": torch.ones(d, device="cuda"), "alpha": lin(heads, d), "compress": [lin(d, p * d)]}
    for name in ("q", "k", "v", "o", "k_proxy", "v_proxy"):
        w[name] = lin(d, d)
    print(f"[case {batch} x {tokens} x {d}]", flush=True)
    s = B.DecodeSession(B.decode_config(batch, d, heads, 64, (p,), dtype="fp32"), w, rnd(batch, heads, 20, 64),
                        rnd(batch, heads, 20, 64), n=2)
    x = rnd(batch, tokens, d)
    s.prefill(x)
    torch.cuda.synchronize()
    tail = tokens % p
    xt = x[:, tokens - tail:].double().cpu()
    u = xt / torch.sqrt((xt * xt).mean(-1, keepdim=True) + 1e-6)
    for name, got in (("k", s.k_loc), ("v", s.v_loc)):
        ref = (u.reshape(-1, d) @ w[name][0].double().cpu().T).reshape(batch, tail, heads, 64).transpose(1, 2)
        err = float((got[:, :, :tail].double().cpu() - ref).norm() / ref.norm())
        print(f"  {name}: {err:.2e} ({err / d ** 0.5:.2e} sqrt(K))", flush=True)
        assert err <= 1.55e-8 * d ** 0.5


def test_bias_gradient_of_few_rows(gpu):
    """fp32 bias gradients over 31 rows: chains of eight values and two joins,
    so at most ten roundings of 2^-24, where one chain loses each of the thirty
    2^-25 that follow a one (8.9e-7)."""
    import torch
    B = gpu
    shape = LayerShape(1, 16 * 31, 64, 64, 1, 64, (16,), dtype="fp32", injection=synth.INJECT_ADD)
    inp = synth.layer_inputs(shape, 4180, with_dy=True)
    inp["dy"][:] = 2.0 ** -25
    inp["dy"][:, :16] = 1.0
    print(f"[case] {shape}", flush=True)
    db = run_gpu_backward(shape, inp)[2]["decompress"][0][1].double().cpu()
    err = float((db - (1.0 + 30 * 2.0 ** -25)).abs().max())
    print(f"  {err:.2e}", flush=True)
    assert err <= 10 * 2.0 ** -24
