"""The trigger scan at the edges of its tiles (4096 positions, four per thread), with results above and below what one
copy brings back (1024 positions), against the rule written out."""
import numpy as np
import pytest
import torch

from paper_2504_12329_amd import binding as B

pytestmark = pytest.mark.gpu


def _rule_written_out(toks, kw, dl, lo, hi, window):
    w = window - 1
    fire = []
    for p in range(lo, hi):
        if w == 0:
            ok = toks[p] in kw
        else:
            ok = p >= w and toks[p - w] in dl and not any(t in dl for t in toks[p - w + 1:p]) and \
                any(t in kw for t in toks[p - w + 1:p + 1])
        if ok:
            fire.append(p)
    return fire


@pytest.mark.parametrize("window", [1, 2, 6, 257])
@pytest.mark.parametrize("lo,hi", [(0, 0), (0, 1), (3, 6), (0, 4095), (1, 4097), (0, 4097), (4095, 4098), (7, 9001)])
def test_scan_tile_edges(window, lo, hi):
    print(f"scan [{lo}, {hi}) window {window}", flush=True)
    vocab = 64
    rng = np.random.Generator(np.random.PCG64(hi * 1000 + window))
    toks = rng.integers(-2, vocab + 2, size=9001, dtype=np.int32)
    if window > 6:                              # long sentences: few delimiters
        toks[(toks == 3) | (toks == 5)] = 7
        toks[::400] = 3
    kw, dl = set(range(8, 40)), {3, 5}
    rule = B.TriggerRule(vocab, B.host_bitmap(vocab, kw), B.host_bitmap(vocab, dl) if window > 1 else None, window)
    dev = torch.from_numpy(toks).cuda()
    want = _rule_written_out(toks.tolist(), kw, dl, lo, hi, window)
    for cap in (0, 5, 1024, 1025, 4096):
        n, pos = B.st_trigger_scan_static(rule, dev, lo, hi, cap)
        assert n == len(want) and pos.tolist() == want[:cap]
    n, pos = B.st_trigger_scan(rule, dev, lo, hi, 9001)
    assert n == len(want) and pos.tolist() == want


@pytest.mark.parametrize("window", [1, 4])
def test_scan_ends_at_the_last_position(window):
    """The last 40 positions of 2^31 - 1 tokens: the tile ends past 2^31."""
    n, first = 2**31 - 1, 2**31 - 1 - 200
    print(f"scan [{n - 40}, {n}) window {window}", flush=True)
    toks = np.random.Generator(np.random.PCG64(5)).integers(0, 16, size=200, dtype=np.int32)
    dev = torch.empty(n, dtype=torch.int32, device="cuda")
    dev[first:] = torch.from_numpy(toks).cuda()
    kw, dl = {1, 2, 3, 4, 5}, {6, 7}
    rule = B.TriggerRule(16, B.host_bitmap(16, kw), B.host_bitmap(16, dl) if window > 1 else None, window)
    want = [first + p for p in _rule_written_out(toks.tolist(), kw, dl, 160, 200, window)]
    assert want
    for scan in (B.st_trigger_scan, B.st_trigger_scan_static):
        found, pos = scan(rule, dev, n - 40, n, 64)
        assert found == len(want) and pos.tolist() == want
    del dev
    torch.cuda.empty_cache()


@pytest.mark.parametrize("vocab,window", [(33, 1), (151936, 2), (245760, 21), (245792, 2), (491520, 1), (600001, 1), (600001, 3)])
def test_scan_tiles_of_8192_with_bitmaps_staged_or_not(vocab, window):
    """Ranges around 8192 and 16384 positions; bitmaps of up to 60 KB together are looked up in LDS, larger ones in global
    memory, also from addresses that are not 16-byte aligned."""
    rng = np.random.Generator(np.random.PCG64(vocab + window))
    toks = rng.integers(-2, vocab + 2, size=16500, dtype=np.int32)
    kw, dl = set(range(0, vocab, 2)), set(range(3, vocab, 7))
    bits = [np.zeros((vocab + 31) // 32, dtype=np.uint32) for _ in range(2)]
    for bm, ids in zip(bits, (kw, dl)):
        np.bitwise_or.at(bm, np.fromiter(ids, np.int64) >> 5, np.uint32(1) << (np.fromiter(ids, np.int64) & 31).astype(np.uint32))
    dev = torch.from_numpy(toks).cuda()
    for shift in (0, 1):
        held = [torch.cat([torch.zeros(shift, dtype=torch.int32), torch.from_numpy(b.view(np.int32))]).cuda() for b in bits]
        rule = B.TriggerRule(vocab, bits[0], bits[1] if window > 1 else None, window)
        rule.kw, rule.delim = held[0][shift:], held[1][shift:]
        rule.c.kw_bitmap, rule.c.delim_bitmap = rule.kw.data_ptr(), rule.delim.data_ptr() if window > 1 else 0
        for lo, hi in ((0, 8191), (0, 8192), (1, 8194), (8190, 16385), (0, 16500)):
            print(f"scan [{lo}, {hi}) vocab {vocab} window {window} shift {shift}", flush=True)
            want = _rule_written_out(toks.tolist(), kw, dl, lo, hi, window)
            n, pos = B.st_trigger_scan(rule, dev, lo, hi, 16500)
            assert n == len(want) and pos.tolist() == want
            n, pos = B.st_trigger_scan_static(rule, dev, lo, hi, 4096)
            assert n == len(want) and pos.tolist() == want[:4096]


@pytest.mark.parametrize("vocab", [64, 151936, 600001])
@pytest.mark.parametrize("window", [1, 3])
def test_scan_lengths_at_which_the_form_changes(vocab, window):
    """Four and eight positions a thread, bitmaps in LDS (not up to 4096 positions, nor for 600 001 ids) or not: the lengths on both
    sides of each change, from the first position and from a later one."""
    rng = np.random.Generator(np.random.PCG64(vocab + window))
    toks = rng.integers(-2, vocab + 2, size=29000, dtype=np.int32)
    kw, dl = set(range(0, vocab, 2)), set(range(3, vocab, 7))
    rule = B.TriggerRule(vocab, B.host_bitmap(vocab, kw), B.host_bitmap(vocab, dl) if window > 1 else None, window)
    dev = torch.from_numpy(toks).cuda()
    for lo in (0, 3001):
        for walked in (4096, 4097, 5632, 5633, 8193, 12288, 12289, 14336, 14337, 24576, 24577):
            hi = lo + walked - (window - 1 if lo else 0)
            print(f"scan [{lo}, {hi}) vocab {vocab} window {window}", flush=True)
            want = _rule_written_out(toks.tolist(), kw, dl, lo, hi, window)
            n, pos = B.st_trigger_scan(rule, dev, lo, hi, 29000)
            assert want and n == len(want) and pos.tolist() == want
            n, pos = B.st_trigger_scan_static(rule, dev, lo, hi, 4096)
            assert n == len(want) and pos.tolist() == want[:4096]
