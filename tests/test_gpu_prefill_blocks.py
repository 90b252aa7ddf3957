"""The 128- and 256-row blocks of chunked prefill at the edges of their waves, steps of four
pages and 64-page block tables, over fixed records and on-demand sparse pages, with COO
streams longer than their staging area, negative and zero scales and unaligned queries.  The
reference is the oracle's fp64 decode attention per query token; the tolerance is that of
tests/test_gpu_rows.py."""
import math

import numpy as np
import pytest
import torch

from tests.cases import np16
from tests.test_gpu_rows import _cache, _case, _check, one_range

pytestmark = pytest.mark.gpu

DEV = "cuda"
P = 16


def _run(ref, hq, h, d, new, lens, window=0, paged=False, kind="t3", scale=None, unaligned=False):
    from paper_2503_18599_amd import binding as B
    c = _case(ref, hq, h, d, lens, kind, seed=3)
    cache, bt = _cache(B, c, paged)
    scale = float(np.float32(1 / math.sqrt(d) if scale is None else scale))
    clen = [min(new, n) for n in lens]
    start = np.array([n - m for n, m in zip(lens, clen)], np.int32)
    cu = np.concatenate([[0], np.cumsum(clen)]).astype(np.int32)
    q = torch.randn(int(cu[-1]), hq, d, generator=torch.Generator().manual_seed(3)).half()
    buf = torch.zeros(q.numel() + 8, dtype=torch.float16, device=DEV)
    qd = buf[1 if unaligned else 0:][:q.numel()].view(q.shape)
    qd.copy_(q)
    got = B.prefill_attention(cache, qd, bt, torch.from_numpy(start).to(DEV), torch.from_numpy(cu).to(DEV),
                              max(lens), scale, window=window).cpu().numpy()
    seq = np.repeat(np.arange(len(lens)), clen)
    pos = np.concatenate([np.arange(s, n) for s, n in zip(start, lens)])
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, h, d, c.thr, np16(q), c.bt.numpy()[seq],
                                (pos + 1).astype(np.int32), np.float32(scale), window=window)
    _check(got, want)


@pytest.mark.parametrize("hq,h,d,new,lens,window,paged,kind", [
    (2, 2, 128, 128, [700, 128, 900], 0, False, "t3"),          # 128 rows, whole prompt among them
    (2, 2, 128, 97, [1100, 97], 0, False, "t3"),                # a row into the fourth wave pair
    (8, 2, 128, 64, [400, 64, 577], 0, False, "t3"),            # 256 rows
    (6, 2, 128, 90, [300, 450], 50, False, "t3"),               # three heads, a window inside the chunk
    (16, 2, 128, 33, [1300, 33], 0, True, "t3"),                # eight heads, sparse pages, > 64 pages
    (8, 2, 128, 64, [200, 70], 0, False, "all_coo"),            # 2 KiB of COO per record: read from HBM
    (8, 2, 128, 64, [200, 70], 0, True, "all_coo"),
    (8, 2, 64, 70, [500, 70], 0, False, "all_coo"),
    (8, 2, 64, 64, [1200, 64], 0, True, "t3"),
    (2, 2, 64, 100, [1100, 100], 300, False, "t3"),
    (8, 8, 128, 200, [300, 200], 0, False, "scales"),
    (8, 8, 64, 200, [300, 200], 0, False, "scales")])
def test_prefill_blocks(ref, hq, h, d, new, lens, window, paged, kind):
    _run(ref, hq, h, d, new, lens, window, paged, kind)


@pytest.mark.parametrize("hq,h,d,new,lens", [(2, 2, 64, 128, [300, 128]),    # 128 rows
                                             (2, 2, 128, 70, [950, 900]),    # 70 rows in a 128-row block
                                             (8, 2, 64, 64, [400, 64]),      # 256 rows
                                             (8, 2, 128, 64, [400, 64])])
@pytest.mark.parametrize("paged", [False, True])
def test_prefill_blocks_largest_value(ref, hq, h, d, new, lens, paged):
    """Stored values of +-65504 read back as up to 65536, past fp16's largest finite value.  (Most
    of them are hidden from some rows; the scale keeps the scores of the others comparable.)"""
    c = _case(ref, hq, h, d, lens, "top", seed=3)
    pool = c.oracle_pool(ref)
    for w in (0, 1):                           # (tokens 0 and 29 of the first sequence)
        x = [ref.dequantize_slot(pool, P, h, d, c.thr, int(c.bt[0, t // P]), i, w, t % P) for t in (0, 29) for i in range(h)]
        assert np.abs(x).max() > 65519
    _run(ref, hq, h, d, new, lens, paged=paged, kind="top", scale=1e-5)


@pytest.mark.parametrize("hq,h,d,new,lens", [(2, 2, 64, 128, [300, 128]), (2, 2, 128, 70, [950, 900]),
                                             (8, 2, 128, 64, [400, 64])])
def test_prefill_blocks_small_values(ref, hq, h, d, new, lens):
    _run(ref, hq, h, d, new, lens, kind="small")


@pytest.mark.parametrize("scale", [-0.05, 0.0])
def test_prefill_blocks_scale(ref, scale):
    _run(ref, 8, 2, 128, 64, [500, 64], scale=scale)


@pytest.mark.parametrize("new", [64, 100])
def test_prefill_blocks_unaligned_query(ref, new):
    _run(ref, 4, 2, 128, new, [700, 100], unaligned=True)


@pytest.mark.parametrize("hq,h,d,new", [(4, 4, 128, 65), (4, 2, 128, 65), (4, 4, 64, 65)])
def test_prefill_blocks_long_range(ref, hq, h, d, new):
    """Enough equal chunks of one shared prefix that its 140 pages stay one range: every wave
    refills its 64-page block tables twice.  (Physical pages are shuffled: a table refilled from
    another place reads other keys.)"""
    from paper_2503_18599_amd import binding as B
    n, L = 260, 2240
    c = _case(ref, hq, h, d, [L], "t3", seed=3)
    cache, bt = _cache(B, c, False)
    q1 = torch.randn(new, hq, d, generator=torch.Generator().manual_seed(3)).half()
    i32 = dict(dtype=torch.int32, device=DEV)
    got = one_range(B, lambda ws: B.prefill_attention(cache, q1.repeat(n, 1, 1).to(DEV), bt.repeat(n, 1),
                                                      torch.full((n,), L - new, **i32), torch.arange(n + 1, **i32) * new, L,
                                                      d ** -0.5, workspace=ws), n * new, hq, h, d, L)
    want = ref.decode_attention(c.oracle_pool(ref), c.num_blocks, P, h, d, c.thr, np16(q1), np.repeat(c.bt.numpy(), new, 0),
                                np.arange(L - new + 1, L + 1, dtype=np.int32), np.float32(d ** -0.5))
    _check(got[:new].cpu().numpy(), want)
    same = bool((got.view(n, new, hq, d) == got[:new]).all())
    assert same


def test_prefill_mixed_chunks_cost_little_more_than_apart(ref):
    """Single tokens beside two prompts (a mean chunk of 33 rows) in one call, against the same rows
    in two calls: blocks as wide as the prompts' would leave each token a workgroup of its own."""
    from paper_2503_18599_amd import binding as B
    H, d = 40, 128
    lens, new = [1024] * 30 + [512] * 2, [1] * 30 + [512] * 2
    pages = [n // P for n in lens]
    g = torch.Generator("cuda").manual_seed(3)
    thr = B.calibrate_thresholds(*(torch.randn(1, 64, H, d, generator=g, device=DEV).half() for _ in range(2)))
    cache = B.Cache(sum(pages), H, d, thr)
    first = np.cumsum([0] + pages)
    bt = torch.tensor([[f + min(i, n - 1) for i in range(max(pages))] for f, n in zip(first, pages)], dtype=torch.int32, device=DEV)
    i32 = dict(dtype=torch.int32, device=DEV)
    k, v = (torch.randn(sum(lens), H, d, generator=g, device=DEV).half() for _ in range(2))
    B.quantize_kv(cache, k, v, bt, torch.zeros(len(lens), **i32), torch.tensor(np.concatenate([[0], np.cumsum(lens)]), **i32),
                  max(lens))

    def time(part):
        n = [new[i] for i in part]
        q = torch.randn(sum(n), H, d, generator=g, device=DEV).half()
        args = (bt[list(part)].contiguous(), torch.tensor([lens[i] - new[i] for i in part], **i32),
                torch.tensor(np.concatenate([[0], np.cumsum(n)]), **i32), max(lens[i] for i in part), d ** -0.5)
        best = float("inf")
        for _ in range(15):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(4):
                B.prefill_attention(cache, q, *args)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]) / 4)
        return best

    both, tokens, prompts = time(range(32)), time(range(30)), time(range(30, 32))
    # (312 us against 174 + 91; 474 in workgroups of 128 rows)
    assert both <= 1.5 * (tokens + prompts), (both, tokens, prompts)
