"""Decode steps of one to seventeen sequences (the projection kernels stage 4,
8, 16 or 32 rows, and the output map merges small partials itself) and short
cache slices, at the sizes where they can go wrong: widths of one to four
16-byte chunks per lane, head counts that are no multiple of four, caches at
and around the slice edges, empty caches, positions per sequence, and steps
across an append; and a sequence's bits in any batch.
"""
import numpy as np
import pytest

import oracle
from paper_2608_23463_amd import synth
from helpers import TOL, dev, dev_weights, host

pytestmark = pytest.mark.gpu

CASES = {
    # name: (batch, n_heads, head_dim, dtype, cached rows)
    "B1_d128_empty": (1, 2, 64, "bf16", 0),
    "B1_d64_n1": (1, 1, 64, "bf16", 1),
    "B1_d576_n127": (1, 9, 64, "bf16", 127),
    "B2_d512_n128": (2, 8, 64, "bf16", 128),
    "B3_d640_n129_dh128": (3, 5, 128, "bf16", 129),
    "B4_d1024_n700": (4, 16, 64, "bf16", 700),
    "B4_d2048_n300_dh128": (4, 16, 128, "bf16", 300),   # four chunks per lane
    "B2_d2048_n40": (2, 32, 64, "bf16", 40),            # two rows of four chunks
    "B2_d512_fp32_n150": (2, 8, 64, "fp32", 150),
    "B2_d512_n700_merged": (2, 8, 64, "bf16", 700),      # two rows in the merged output map
    "B4_d256_fp32_n90": (4, 4, 64, "fp32", 90),
    "B4_d1024_n3000_combine": (4, 16, 64, "bf16", 3000),  # more channels than the merge takes
    "merge_past_B1_d1024_n16500": (1, 16, 64, "bf16", 16500),  # 17 slices: partials past the merge's bound
    "merge_B1_d1024_n16380": (1, 16, 64, "bf16", 16380),       # 16, at the bound
    "B8_d320_n90": (8, 5, 64, "bf16", 90),              # two staged rows per wave
    "B9_d512_n200": (9, 8, 64, "bf16", 200),            # four
    "B16_d1024_n60_dh128": (16, 8, 128, "bf16", 60),
    "B17_d256_fp32_n33": (17, 4, 64, "fp32", 33),       # eight
    "B5_d512_n500": (5, 8, 64, "bf16", 500),
    "B1_d1024_fp32_n260": (1, 16, 64, "fp32", 260),     # four chunks per lane in fp32
    "B3_d192_fp32_n1100": (3, 3, 64, "fp32", 1100),
}


def weights_of(inp, dtype):
    """The drawn weights with sharper queries and a larger output map, so that
    the cached read moves y by more than its tolerance."""
    w = dict(inp["weights"])
    w["q"] = (w["q"][0] * 4, w["q"][1])
    w["o"] = (w["o"][0] * 16, w["o"][1])
    return w


@pytest.mark.parametrize("name", CASES)
def test_small_batch_steps(gpu, name):
    import torch
    B = gpu
    batch, heads, dh, dt, n0 = CASES[name]
    steps, p = 6, 4
    shape = synth.DecodeShape(batch, heads * dh, heads, dh, (p,), n0=n0, steps=steps, dtype=dt)
    print(f"[case {name}] {shape}", flush=True)
    inp = synth.decode_inputs(shape, 900 + sorted(CASES).index(name))
    w = weights_of(inp, dt)
    cfg = B.decode_config(batch, shape.d_model, heads, dh, (p,), dtype=dt)
    sess = B.DecodeSession(cfg, dev_weights(w, dt), dev(inp["k_cache"], dt), dev(inp["v_cache"], dt), n=n0)
    st = oracle.DecodeState.empty(batch, heads, dh, p, shape.capacity, shape.d_model)
    st.k_cache[:], st.v_cache[:], st.n = inp["k_cache"], inp["v_cache"], n0
    for t in range(steps):
        y = sess.step(dev(inp["x"][t], dt))
        ref = oracle.decode_step(st, w, (p,), inp["x"][t])
        torch.cuda.synchronize()
        x = inp["x"][t].astype(np.float64)
        # y, and the sublayer's share y - x against its own size (bf16 also rounds
        # the x it is added to: half a unit of y)
        err = oracle.max_rel_err(host(y), ref)
        sub = np.abs((host(y) - x) - (ref - x)).max() / np.abs(ref - x).max()
        slack = 2.0 ** -8 * np.abs(ref).max() / np.abs(ref - x).max() if dt == "bf16" else 0.0
        print(f"  step {t}: y {err:.2e}, y - x {sub:.2e}", flush=True)
        assert err <= TOL[dt] and sub <= TOL[dt] + slack
    assert (sess.n, sess.j) == (st.n, st.j)
    rows = slice(n0, st.n)
    assert oracle.max_rel_err(host(sess.k_cache)[:, :, rows], st.k_cache[:, :, rows]) <= TOL[dt]


@pytest.mark.parametrize("batch", [1, 4])
def test_small_batch_ragged_equals_lockstep(gpu, batch):
    """Equal per-sequence positions give the lockstep result bit for bit."""
    import torch
    B = gpu
    shape = synth.DecodeShape(batch, 256, 4, 64, (4,), n0=140, steps=5)
    inp = synth.decode_inputs(shape, 950)
    cfg = B.decode_config(batch, 256, 4, 64, (4,))
    out = []
    for ragged in (False, True):
        sess = B.DecodeSession(cfg, dev_weights(inp["weights"], "bf16"), dev(inp["k_cache"], "bf16"),
                               dev(inp["v_cache"], "bf16"), n=140, ragged=ragged)
        out.append(torch.stack([sess.step(dev(inp["x"][t], "bf16")) for t in range(5)]))
    torch.cuda.synchronize()
    assert torch.equal(*out)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_bits_do_not_depend_on_the_batch(gpu, dtype):
    """Sequences of several lengths, decoded together at their own positions
    and each alone in lockstep: equal bit for bit (slices by a sequence's own
    length, row arithmetic the same for every staged row count, one merge)."""
    import torch
    B = gpu
    lens = [0, 1, 127, 300, 2048, 2049]
    shape = synth.DecodeShape(len(lens), 256, 4, 64, (4,), n0=max(lens), steps=5, dtype=dtype)
    inp = synth.decode_inputs(shape, 960)
    w = dev_weights(inp["weights"], dtype)
    kc, vc = dev(inp["k_cache"], dtype), dev(inp["v_cache"], dtype)
    xs = dev(inp["x"], dtype)
    sess = B.DecodeSession(B.decode_config(len(lens), 256, 4, 64, (4,), dtype=dtype), w, kc.clone(), vc.clone(),
                           ragged=True, n_seq=lens)
    together = torch.stack([sess.step(xs[t]) for t in range(5)])
    for b, n in enumerate(lens):
        one = B.DecodeSession(B.decode_config(1, 256, 4, 64, (4,), dtype=dtype), w, kc[b:b + 1].clone(),
                              vc[b:b + 1].clone(), n=n)
        alone = torch.stack([one.step(xs[t, b:b + 1].clone()) for t in range(5)])
        torch.cuda.synchronize()
        assert torch.equal(alone[:, 0], together[:, b]), n


@pytest.mark.parametrize("dtype,heads,factors", [("bf16", 16, (8, 8)), ("fp32", 8, (4, 16))])
def test_bits_do_not_depend_on_the_batch_across_an_append(gpu, dtype, heads, factors):
    """64 sequences together, 12 of them, and each of a few alone, through a
    step that completes a block and two that read it: cached rows and outputs
    equal bit for bit. The compressions are long enough to be cut along K."""
    import torch
    B = gpu
    d, p, steps = heads * 64, factors[0] * factors[1], 3
    gen = torch.Generator(device="cuda").manual_seed(970)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def rnd(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * std).to(dt)

    shape = synth.DecodeShape(1, d, heads, 64, factors, n0=0, steps=1, dtype=dtype)
    w = dev_weights(synth.decode_inputs(shape, 971)["weights"], dtype)
    lens = [(37 * b) % 200 for b in range(64)]
    kc, vc = rnd(64, heads, 210, 64), rnd(64, heads, 210, 64)
    blk, kl, vl = rnd(64, p, d), rnd(64, heads, p, 64), rnd(64, heads, p, 64)
    xs = rnd(steps, 64, d)

    def decode(rows):
        ragged = len(rows) > 1
        kw = dict(ragged=True, n_seq=[lens[b] for b in rows], j_seq=[p - 1] * len(rows)) if ragged else dict(n=lens[rows[0]])
        s = B.DecodeSession(B.decode_config(len(rows), d, heads, 64, factors, dtype=dtype), w, kc[rows].clone(),
                            vc[rows].clone(), **kw)
        s.x_blk.copy_(blk[rows])
        s.k_loc.copy_(kl[rows])
        s.v_loc.copy_(vl[rows])
        if not ragged:
            s.state.j = p - 1
        y = torch.stack([s.step(xs[t, rows].clone()) for t in range(steps)])
        torch.cuda.synchronize()
        return y, s.k_cache, s.v_cache

    whole = decode(list(range(64)))
    for rows in [list(range(12))] + [[b] for b in (0, 5, 11, 40, 63)]:
        part = decode(rows)
        new = [lens[b] for b in rows]  # the row the block was appended at
        for i, b in enumerate(rows):
            for c in (1, 2):
                assert torch.equal(part[c][i, :, new[i]], whole[c][b, :, new[i]]), (len(rows), b, "cached row")
            assert torch.equal(part[0][:, i], whole[0][:, b]), (len(rows), b)
