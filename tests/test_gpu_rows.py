"""The kernel of up to 32 query rows per wave (short prefill chunks; decode at head_dim 64)
where it can go wrong: row counts around its 16-row tiles, COO streams longer than its
staging area, values and thresholds of very different scales, ranges longer than the
wave's table of pages.  The reference is the oracle's fp64 decode attention per query token.

Tolerance, of each row's own 2-norm: a score is a sum of fp32 roundings of terms up to some 30
(2^-24 x 30 = 2e-6, several of them), and its error is the relative error of a probability;
weights and corrections carry 22 bits or more and everything sums in fp32.  2e-5 is ten
such terms."""
import dataclasses
import math

import numpy as np
import pytest
import torch

from paper_2503_18599_amd import synth
from tests.cases import Case, np16

pytestmark = pytest.mark.gpu

DEV = "cuda"
P = 16
REL = 2e-5
INF = float("inf")


def _case(ref, hq, h, d, lens, kind, seed=0):
    w = dataclasses.replace(synth.WORKLOADS[2], n_seqs=len(lens), n_q_heads=hq, n_kv_heads=h, head_dim=d, cid=700 + seed)
    c = Case(w, lens=lens)
    if kind == "all_coo":                      # every value inner: whole records of COO entries
        c.thr = np.tile(np.array([-INF, -INF, INF, INF], np.float32), (h, 2, 1))
        return c
    if kind == "scales":                       # heads and tokens of very different magnitudes
        f = torch.logspace(-3, 3, h).view(1, h, 1)
        t = torch.logspace(-2, 0, c.v.shape[0])[torch.randperm(c.v.shape[0], generator=torch.Generator().manual_seed(1))]
        c.v = (c.v.float() * f * t.view(-1, 1, 1)).clamp(-60000, 60000).half()
        k = np.stack([np16(c.k[:256]), np16(c.v[:256])])
        c.thr = ref.calibrate(k[0][None], k[1][None], 0.04, 0.06)
        return c
    if kind == "small":                        # values whose low fp16 part would be subnormal
        c.v = (c.v.float() * 1e-4).half()
        v = np16(c.v[:256]).reshape(8, -1, h, d)   # (averages of runs: thresholds between fp16 numbers)
        c.calibrate_oracle(ref)
        c.thr[:, 1] = ref.calibrate(v, v, 0.04, 0.06)[:, 1]
        return c
    c.calibrate_oracle(ref)
    if kind == "top":                          # every 29th token of K and V holds fp16's largest value
        g = torch.Generator().manual_seed(2)
        for x in (c.k, c.v):
            at = torch.randint(0, c.d, x.shape[:2], generator=g).unsqueeze(-1)
            sign = 1.0 - 2.0 * torch.randint(0, 2, at.shape, generator=g)
            x[::29] = x[::29].scatter(2, at[::29], (65504.0 * sign[::29]).half())
    return c


def _cache(B, c, paged):
    cache = B.Cache(c.num_blocks, c.H, c.d, torch.from_numpy(c.thr).to(DEV),
                    sparse_pages=8 * c.num_blocks * c.H * 2 if paged else 0)
    bt = c.bt.to(DEV)
    B.quantize_kv(cache, c.k.to(DEV), c.v.to(DEV), bt, torch.zeros(c.n_seqs, dtype=torch.int32, device=DEV), c.cu.to(DEV),
                  int(c.lens.max()))
    return cache, bt


def _check(got, want):
    got, want = got.astype(np.float64), want.astype(np.float64)
    assert np.all(np.isfinite(got))
    rel = np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert rel.max() <= REL, float(rel.max())


@pytest.mark.parametrize("hq,h,d,new,lens,window,paged,kind", [
    (2, 2, 128, 1, [1, 16, 17, 250], 0, False, "t3"),        # one row
    (2, 2, 128, 15, [15, 40, 300], 0, False, "t3"),          # a row short of a tile
    (2, 2, 128, 17, [17, 33, 300], 0, False, "t3"),          # two tiles, the second with one row
    (6, 2, 128, 5, [5, 90, 301], 20, False, "t3"),           # three heads: 15 rows, a window
    (16, 2, 128, 4, [4, 64, 100], 0, False, "t3"),           # eight heads: 32 rows, two tiles full
    (4, 2, 64, 16, [16, 31, 500], 0, False, "t3"),           # head_dim 64, two tiles full
    (8, 2, 64, 3, [3, 100], 33, True, "t3"),                 # head_dim 64 over sparse pages
    (2, 2, 128, 33, [33, 200], 0, False, "t3"),              # two blocks, the second with one row
    (8, 2, 64, 16, [16, 300], 0, False, "t3"),               # 64 rows: two full blocks
    (2, 2, 128, 9, [40, 100], 0, False, "all_coo"),          # 2 KiB of COO per record: read from HBM
    (2, 2, 128, 9, [40, 100], 0, True, "all_coo"),
    (4, 2, 64, 2, [40, 100], 0, False, "all_coo"),
    (8, 8, 128, 4, [200, 37], 0, False, "scales"),
    (8, 8, 64, 4, [200, 37], 0, False, "scales")])
def test_rows_prefill(ref, hq, h, d, new, lens, window, paged, kind):
    from paper_2503_18599_amd import binding as B
    c = _case(ref, hq, h, d, lens, kind)
    cache, bt = _cache(B, c, paged)
    clen = [min(new, n) for n in lens]
    start = np.array([n - m for n, m in zip(lens, clen)], np.int32)
    cu = np.concatenate([[0], np.cumsum(clen)]).astype(np.int32)
    q = torch.randn(int(cu[-1]), hq, d, generator=torch.Generator().manual_seed(3)).half()
    got = B.prefill_attention(cache, q.to(DEV), bt, torch.from_numpy(start).to(DEV), torch.from_numpy(cu).to(DEV),
                              max(lens), 1 / math.sqrt(d), window=window).cpu().numpy()
    seq = np.repeat(np.arange(len(lens)), clen)
    pos = np.concatenate([np.arange(s, n) for s, n in zip(start, lens)])
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, h, d, c.thr, np16(q), c.bt.numpy()[seq],
                                (pos + 1).astype(np.int32), np.float32(1 / math.sqrt(d)), window=window)
    _check(got, want)


@pytest.mark.parametrize("hq,h,lens,window,kind", [
    (4, 4, [1, 15, 16, 17, 128, 700], 0, "t3"), (16, 4, [1, 33, 600], 100, "t3"), (16, 2, [70, 5], 0, "all_coo"),
    (8, 8, [300, 20], 0, "scales")])
def test_rows_decode_d64(ref, hq, h, lens, window, kind):
    from paper_2503_18599_amd import binding as B
    c = _case(ref, hq, h, 64, lens, kind, seed=1)
    cache, bt = _cache(B, c, False)
    q = torch.randn(len(lens), hq, 64, generator=torch.Generator().manual_seed(4)).half()
    got = B.decode_attention(cache, q.to(DEV), bt, c.lens.to(DEV), max(lens), 0.125, window=window).cpu().numpy()
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, h, 64, c.thr, np16(q), c.bt.numpy(),
                                np.array(lens, np.int32), np.float32(0.125), window=window)
    _check(got, want)


@pytest.mark.parametrize("hq,h,lens,dist,bound", [
    (32, 8, [57] * 6, "gauss_outlier_ch", 2.08e-7), (16, 8, [900, 1500, 400], "gauss_outlier_ch", 3.46e-7),
    (32, 8, [57] * 6, "t3_lognormal", 1.71e-7), (16, 8, [900, 1500, 400], "t3_lognormal", 2.82e-7)])
def test_rows_decode_d64_error(ref, hq, h, lens, dist, bound):
    """No further from the 64-bit result than 32-bit products and sums are: a kernel that dequantizes
    to fp32 and sums each score and output in fp32 on the vector units was off by `bound`."""
    from paper_2503_18599_amd import binding as B
    w = dataclasses.replace(synth.WORKLOADS[2], n_seqs=len(lens), n_q_heads=hq, n_kv_heads=h, head_dim=64, cid=720,
                            k_dist=dist, v_dist=dist)
    c = Case(w, lens=lens)
    c.calibrate_oracle(ref)
    cache, bt = _cache(B, c, False)
    q = torch.randn(len(lens), hq, 64, generator=torch.Generator().manual_seed(6)).half()
    got = B.decode_attention(cache, q.to(DEV), bt, c.lens.to(DEV), max(lens), 0.125).cpu().numpy()
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, h, 64, c.thr, np16(q), c.bt.numpy(),
                                np.array(lens, np.int32), np.float32(0.125))
    err = np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want)
    assert err <= bound, float(err)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("big", [65504.0, -65504.0, 600.0])
def test_rows_hidden_key_of_another_size(ref, d, big):
    """Keys that share their page with visible ones but lie before the window, or past the query,
    and score thousands of times as much: no trace of them in the results."""
    from paper_2503_18599_amd import binding as B
    lens, new = [45, 70], 4
    c = _case(ref, 4, 2, d, lens, "t3", seed=9)
    first = c.cu[:-1].long()
    c.k[first + torch.tensor([0, 32])] = big   # the first windows of 30 start at keys 12 and 37
    c.k[first + torch.tensor(lens) - 1] = big  # (the last query sees this one itself)
    cache, bt = _cache(B, c, False)
    q = torch.randn(2 * new, 4, d, generator=torch.Generator().manual_seed(10)).half()
    i32 = dict(dtype=torch.int32, device=DEV)
    got = B.prefill_attention(cache, q.to(DEV), bt, c.lens.to(DEV) - new, torch.tensor([0, new, 2 * new], **i32),
                              max(lens), 0.1, window=30).cpu().numpy()
    pos = np.concatenate([np.arange(n - new, n) for n in lens])
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, 2, d, c.thr, np16(q),
                                c.bt.numpy()[np.repeat([0, 1], new)], (pos + 1).astype(np.int32), np.float32(0.1), window=30)
    seen = np.arange(2 * new) % new != new - 1
    _check(got[seen], want[seen])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale", [-0.05, 0.0])
def test_rows_scale(ref, d, scale):
    from paper_2503_18599_amd import binding as B
    lens, new = [300, 40], 3
    c = _case(ref, 4, 2, d, lens, "t3", seed=4)
    cache, bt = _cache(B, c, False)
    q = torch.randn(2 * new, 4, d, generator=torch.Generator().manual_seed(7)).half()
    i32 = dict(dtype=torch.int32, device=DEV)
    got = B.prefill_attention(cache, q.to(DEV), bt, c.lens.to(DEV) - new, torch.tensor([0, new, 2 * new], **i32),
                              max(lens), scale, window=33).cpu().numpy()
    pos = np.concatenate([np.arange(n - new, n) for n in lens])
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, 2, d, c.thr, np16(q),
                                c.bt.numpy()[np.repeat([0, 1], new)], (pos + 1).astype(np.int32), np.float32(scale), window=33)
    _check(got, want)


def one_range(B, call, n_tokens, hq, h, d, max_len, window=0):
    """The result of call(workspace), after checking that it wrote no split partials: the workspace
    holds the row-block list (at most 16 bytes a token, and its count), then nothing."""
    n = int(B.lib().oaken_prefill_attention_workspace_bytes(n_tokens, hq, h, d, max_len, window))
    ws = torch.full((n + 4096,), 0x5a, dtype=torch.uint8, device=DEV)
    got = call(ws)
    untouched = bool((ws[16 * n_tokens + 1024:] == 0x5a).all())
    assert untouched, "cut into ranges"
    return got


def test_single_tokens_stay_one_range(ref):
    """1600 chunks of one token over 4 heads are 6400 waves: the chip is full, no range is cut."""
    from paper_2503_18599_amd import binding as B
    n, L = 1600, 640
    c = _case(ref, 4, 4, 128, [L], "t3", seed=2)
    cache, bt = _cache(B, c, False)
    q1 = torch.randn(1, 4, 128, generator=torch.Generator().manual_seed(5)).half()
    i32 = dict(dtype=torch.int32, device=DEV)
    got = one_range(B, lambda ws: B.prefill_attention(cache, q1.repeat(n, 1, 1).to(DEV), bt.repeat(n, 1),
                                                      torch.full((n,), L - 1, **i32), torch.arange(n + 1, **i32), L, 0.09,
                                                      workspace=ws), n, 4, 4, 128, L).cpu().numpy()
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, 4, 128, c.thr, np16(q1), c.bt.numpy(),
                                np.array([L], np.int32), np.float32(0.09))
    _check(got[:1], want)
    assert np.array_equal(got, np.broadcast_to(got[:1], got.shape))


@pytest.mark.parametrize("hq,h,d,new", [(16, 2, 128, 2), (16, 2, 128, 4), (16, 2, 64, 2)])
def test_rows_long_range(ref, hq, h, d, new):
    """Many short chunks of one shared 2300-token prefix: the chip is full without cutting ranges, so
    each wave walks all 144 pages, past its 64-page tables twice.  (Physical pages are shuffled: a
    table refilled from another place reads other keys.)"""
    from paper_2503_18599_amd import binding as B
    n, L = 8192 // new, 2300
    c = _case(ref, hq, h, d, [L], "t3", seed=2)
    cache, bt = _cache(B, c, False)
    q1 = torch.randn(new, hq, d, generator=torch.Generator().manual_seed(5)).half()
    i32 = dict(dtype=torch.int32, device=DEV)
    got = one_range(B, lambda ws: B.prefill_attention(cache, q1.repeat(n, 1, 1).to(DEV), bt.repeat(n, 1),
                                                      torch.full((n,), L - new, **i32), torch.arange(n + 1, **i32) * new, L,
                                                      0.09, workspace=ws), n * new, hq, h, d, L)
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, h, d, c.thr, np16(q1), np.repeat(c.bt.numpy(), new, 0),
                                np.arange(L - new + 1, L + 1, dtype=np.int32), np.float32(0.09))
    _check(got[:new].cpu().numpy(), want)
    same = bool((got.view(n, new, hq, d) == got[:new]).all())
    assert same


@pytest.mark.parametrize("hq,h,d,most", [(4, 4, 128, 4), (8, 2, 64, 40), (32, 4, 128, 21)])
def test_row_blocks_of_many_sequences(ref, hq, h, d, most):
    """More sequences than the row-block list takes in one round, empty chunks among them, chunks of
    several blocks: rows at every position of one cached prefix."""
    from paper_2503_18599_amd import binding as B
    n, L = 1500 if most == 4 else 1100, 64
    c = _case(ref, hq, h, d, [L], "t3", seed=5)
    cache, bt = _cache(B, c, False)
    clen = np.array([(i * 5) % most if i % 3 else 0 for i in range(n)])
    start = np.array([(i * 7) % (L - most + 1) for i in range(n)], np.int32)
    cu = np.concatenate([[0], np.cumsum(clen)]).astype(np.int32)
    q = torch.randn(int(cu[-1]), hq, d, generator=torch.Generator().manual_seed(8)).half()
    got = B.prefill_attention(cache, q.to(DEV), bt.repeat(n, 1), torch.from_numpy(start).to(DEV), torch.from_numpy(cu).to(DEV),
                              L, 0.1).cpu().numpy()
    pos = np.concatenate([np.arange(s, s + m) for s, m in zip(start, clen)])
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, h, d, c.thr, np16(q),
                                c.bt.numpy()[np.zeros(len(pos), int)], (pos + 1).astype(np.int32), np.float32(0.1))
    _check(got, want)
