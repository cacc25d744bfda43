"""The catch-up attention (head_dim 128) in both its block forms on the GPU, with one and several key ranges: one tile, odd and
even tile counts of a range, rows that fill a wave or leave most of a block idle, one- and two-term queries, one and eight query
heads per kv head, ragged passes.

The last row's logits of a one-layer model with a zero MLP depend on the last query row only, so every row is checked
instead through the K/V rows of the layer above it: a pass of m rows on kv0 cached keys against the same tokens fed one
by one through the decode step, whose attention is another kernel in fp32."""
import pytest
import torch

from paper_2504_12329_amd import binding as B, synth
from tests.gpu_common import print_case

pytestmark = pytest.mark.gpu

# A pass rounds the attention weights to bf16 (2^-9 each, averaged over the keys) and its other inputs to 16 mantissa
# bits; K and V of the second layer then differ from the decode step's by flipped bf16 roundings.  Single bf16 inputs
# (fast) round 2^-9 at every GEMM.  A lost tile or row is off by 0.1 and more.
TOL = {"default": 1e-2, "fast": 3e-2}


# form: waves per block and key ranges; the comment says how many tiles the longest row has, and the last of its ranges
@pytest.mark.parametrize("G,nkv,kv0,m,mode,form", [
    (1, 1, 0, 1, "default", (4, 1)), (1, 1, 0, 64, "default", (4, 1)), (1, 2, 63, 2, "default", (4, 1)),
    (8, 1, 64, 17, "default", (4, 1)), (4, 2, 127, 65, "default", (4, 3)), (5, 8, 700, 40, "default", (4, 12)),
    (7, 4, 1990, 33, "default", (4, 16)), (6, 2, 0, 200, "default", (4, 4)), (5, 8, 10, 300, "default", (8, 1)),
    (6, 2, 0, 200, "fast", (8, 1)), (5, 8, 500, 260, "fast", (8, 1)), (8, 8, 0, 520, "fast", (4, 1)),
    (7, 4, 2050, 126, "default", (8, 6)),   # 34: six tiles, last four
    (5, 8, 3001, 250, "default", (8, 3)),   # 51: seventeen (nine and eight to a half)
    (5, 8, 4096, 86, "default", (8, 7)),    # 66: ten, last six
    (7, 4, 2050, 64, "default", (8, 9)),    # 34: four, last two
    (5, 8, 1900, 150, "fast", (8, 5)),      # 33: seven, last five
    (7, 4, 1200, 200, "fast", (8, 4))])     # 22: six, last four
def test_attention_of_every_row(G, nkv, kv0, m, mode, form):
    print_case(f"2 layers, {G} x {nkv} heads: pass of {m} rows on {kv0} keys ({mode}) against decode steps")
    seq = kv0 + m
    cfg = synth.model_config("tiny_small", max_seq=seq, max_chunk=seq, n_layers=2)
    cfg.update(hidden=256, n_q_heads=G * nkv, n_kv_heads=nkv, head_dim=128, intermediate=128, vocab=512)
    assert B.st_prefill_plan_forms(cfg, m, kv0, mode != "fast")[1:] == form
    g = B.Model(cfg, synth.make_weights(cfg, 31, device="cuda"))
    toks = synth.make_prompt(seq, cfg["vocab"], 32)
    kv = g.kv.view(torch.bfloat16).view(2, 2, nkv, seq, 128)
    if kv0:
        g.prefill(toks[:kv0], want_logits=False)
    g.prefill(toks[kv0:], want_logits=False, fast=mode == "fast")
    one = kv[:, 1, :, kv0:].float().clone()
    g.truncate(kv0)
    for t in toks[kv0:]:
        g.decode_step(int(t), want_logits=False)
    ref = kv[:, 1, :, kv0:].float()
    worst = float(((one - ref).norm(dim=-1) / ref.norm(dim=-1)).max())
    print_case("worst row", worst)
    assert worst <= TOL[mode]
    g.close()


@pytest.mark.parametrize("G,nkv,kv0,m,bad,mode", [
    (6, 2, 30, 512, 448, "default"), (6, 2, 30, 512, 448, "fast"), (7, 4, 2050, 126, 2112, "default"),
    (5, 8, 100, 300, 192, "default"), (4, 1, 40, 40, 64, "default")])
def test_a_non_finite_value_stays_out_of_earlier_key_tiles(G, nkv, kv0, m, bad, mode):
    """The token at position `bad`, the first of a key tile, has a NaN embedding, so its K and V rows are NaN.  Rows whose
    32-row wave ends before that tile begins skip it, also where other waves of their block do not, and must be what they
    are without it, bit for bit."""
    seq = kv0 + m
    print_case(f"2 layers, {G} x {nkv} heads: pass of {m} rows on {kv0} keys ({mode}), NaN at {bad}")
    cfg = synth.model_config("tiny_small", max_seq=seq, max_chunk=seq, n_layers=2)
    cfg.update(hidden=256, n_q_heads=G * nkv, n_kv_heads=nkv, head_dim=128, intermediate=128, vocab=512)
    w = synth.make_weights(cfg, 31, device="cuda")
    w["embed"][511] = float("nan")
    g = B.Model(cfg, w)
    toks = synth.make_prompt(seq, 511, 32)
    kv = g.kv.view(torch.bfloat16).view(2, 2, nkv, seq, 128)
    rows = []
    for poison in (False, True):
        t = toks.copy()
        if poison:
            t[bad] = 511
        g.truncate(0)
        if kv0:
            g.prefill(t[:kv0], want_logits=False)
        g.prefill(t[kv0:], want_logits=False, fast=mode == "fast")
        rows.append(kv[:, 1].float().clone())
    # folded row r of the pass is token r / G; the last wave with a row of token q ends with row r | 31
    last_token = lambda q: min(((q * G + G - 1) | 31) // G, m - 1)  # noqa: E731
    clear = [q for q in range(m) if kv0 + last_token(q) < bad // 64 * 64]
    print_case("rows clear of the tile", len(clear), "of", m)
    assert bool(torch.isnan(rows[1][:, :, bad:]).all())
    if clear:
        at = [kv0 + q for q in clear]
        assert torch.equal(rows[0][:, :, at], rows[1][:, :, at])
    g.close()


@pytest.mark.parametrize("G,nkv,kv0,m", [(6, 2, 0, 480), (7, 4, 0, 480), (5, 8, 0, 1000), (7, 4, 1900, 126), (6, 2, 1300, 21)])
def test_attention_weights_are_rounded_below_their_maximum(G, nkv, kv0, m):
    """The bf16 rounding of the attention weights is a pass's largest error.  Weights rounded at any scale are off by 2^-8 / sqrt 3
    over their mantissa, 1.66e-3 on average, and so is their sum with V.  Taken relative to the running maximum the largest
    weights lie just below 1, where the mantissa is largest, and the maximum itself is exact: with scores spread by 2.5 the
    error is 0.5e-3 to 0.75e-3 however the tiles are dealt out (evaluated in 64 bits); relative to a maximum that
    is raised late it is 1.2e-3 to 1.5e-3.  One layer, so that the last row's logits show it, against the decode step,
    whose weights stay in fp32, over sixteen sequences; the rest of the two paths differs by 16-bit inputs (1e-5)."""
    print_case(f"1 layer, {G} x {nkv} heads: last row of a pass of {m} on {kv0} keys against the decode step")
    seq = kv0 + m
    cfg = synth.model_config("tiny_small", max_seq=seq, max_chunk=seq, n_layers=1)
    cfg.update(hidden=256, n_q_heads=G * nkv, n_kv_heads=nkv, head_dim=128, intermediate=128, vocab=2048)
    w = synth.make_weights(cfg, 33, device="cuda")
    lw = w["layers"][0]
    lw["wqkv"][:(G * nkv + nkv) * 128] *= 5   # q and k of deviation 1.6: scores of deviation 2.5
    lw["wo"] *= 8                             # attention, not the embedding, makes the row
    lw["w_down"].zero_()
    g = B.Model(cfg, w)
    err = 0.0
    for s in range(16):
        toks = synth.make_prompt(seq, cfg["vocab"], 100 + s)
        g.truncate(0)
        if kv0:
            g.prefill(toks[:kv0], want_logits=False)
        a = torch.from_numpy(g.prefill(toks[kv0:])[0]).double()
        g.truncate(seq - 1)
        b = torch.from_numpy(g.decode_step(int(toks[-1]))[0]).double()
        err += float((a - b).norm() / b.norm()) ** 2 / 16
    err **= 0.5
    print_case("worst of the weights: rms error", err)
    assert err <= 1e-3
    g.close()


def test_ragged_segments_shorter_than_the_key_ranges():
    """One pass over segments of very different contexts: the ranges are those of the longest (33 tiles, about nine), so the
    short segments have ranges without a tile and ranges with one.  Against the decode steps of each sequence."""
    G, nkv, ctx, new = 7, 4, [2050, 3, 130, 640], [33, 5, 21, 17]
    print_case(f"2 layers, {G} x {nkv} heads: ragged pass of {new} rows on {ctx} keys against decode steps")
    cfg = synth.model_config("tiny_small", max_seq=2112, max_chunk=2112, n_layers=2)
    cfg.update(hidden=256, n_q_heads=G * nkv, n_kv_heads=nkv, head_dim=128, intermediate=128, vocab=512)
    assert B.st_prefill_plan_forms(cfg, sum(new), 2083 - sum(new))[1:] == (8, 9)  # the same rows as one segment
    w = synth.make_weights(cfg, 31, device="cuda")
    b, g = B.Batch(cfg, w, len(ctx)), B.Model(cfg, w)
    seqs = [synth.make_prompt(c + k, cfg["vocab"], 40 + i) for i, (c, k) in enumerate(zip(ctx, new))]
    bkv = b.kv.view(torch.bfloat16).view(len(ctx), 2, 2, nkv, cfg["max_seq"], 128)
    kv = g.kv.view(torch.bfloat16).view(2, 2, nkv, cfg["max_seq"], 128)
    for i, c in enumerate(ctx):
        b.prefill(i, seqs[i][:c], want_logits=False)
    b.prefill_many(list(range(len(ctx))), [s[c:] for s, c in zip(seqs, ctx)], want_logits=False)
    for i, c in enumerate(ctx):
        g.truncate(0)
        g.prefill(seqs[i][:c], want_logits=False)
        for t in seqs[i][c:]:
            g.decode_step(int(t), want_logits=False)
        ref, one = kv[:, 1, :, c:len(seqs[i])].float(), bkv[i, :, 1, :, c:len(seqs[i])].float()
        worst = float(((one - ref).norm(dim=-1) / ref.norm(dim=-1)).max())
        print_case("segment", i, "worst row", worst)
        assert worst <= TOL["default"]
    b.close()
    g.close()
