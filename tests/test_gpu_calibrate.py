"""Threshold calibration at the edges of its kernel: rows that are not whole 16-byte chunks,
unaligned sets, rows wider than a workgroup, tiny sets and repeated values, bit for bit
against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# runs, tokens, heads, head_dim, elements that the set starts past an aligned address
SIZES = [(1, 1, 1, 64, 0), (3, 2, 2, 7, 0), (2, 37, 3, 72, 0), (2, 5, 2, 128, 3), (1, 515, 2, 128, 0),
         (2, 3, 1, 8192, 0), (2, 3, 1, 8200, 0), (9, 16, 2, 64, 8)]


@pytest.mark.parametrize("R,T,H,d,shift", SIZES)
@pytest.mark.parametrize("kind", ["normal", "few_values", "wide"])
def test_calibration_sizes(ref, R, T, H, d, shift, kind):
    from paper_2503_18599_amd import binding as B
    g = torch.Generator().manual_seed(R * 1000 + T * 10 + d)
    x = torch.randn(2, R, T, H, d, generator=g)
    if kind == "few_values":
        x = x.round()                      # many ties, both zeros
    elif kind == "wide":
        x = x * torch.exp(4.0 * torch.randn(x.shape, generator=g))
    x = x.clamp(-60000, 60000).half()
    dev = []
    for w in range(2):
        buf = torch.zeros(x[w].numel() + 64, dtype=torch.float16, device="cuda")
        view = buf[shift:shift + x[w].numel()].view(R, T, H, d)
        view.copy_(x[w])
        dev.append(view)
    for outer, inner in ((0.04, 0.06), (0.0, 0.0), (0.3, 0.7)):
        if 2 * round(T * d * outer / 2) > T * d - 1:
            continue
        want = ref.calibrate(x[0].numpy(), x[1].numpy(), outer, inner)
        got = B.calibrate_thresholds(dev[0], dev[1], outer, inner).cpu().numpy()
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), (kind, outer, inner)


@pytest.mark.parametrize("d,shift", [(128, 3), (100, 0), (20, 0)])
def test_calibration_without_whole_chunks_keeps_every_lane_busy(d, shift):
    """Sets that the 16-byte loads do not take: two-byte loads by every lane cost about twice the
    aligned set's time per value; rows walked one at a time, d lanes busy, ten times and more."""
    from paper_2503_18599_amd import binding as B

    def time(dim, off):
        R, T, H = 8, 512, 40
        buf = torch.randn(2, R * T * H * dim + 8, generator=torch.Generator("cuda").manual_seed(1), device="cuda").half()
        k, v = (buf[w][off:off + R * T * H * dim].view(R, T, H, dim) for w in (0, 1))
        best = float("inf")
        for _ in range(20):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            B.calibrate_thresholds(k, v, 0.04, 0.06)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        return best

    assert time(d, shift) / d <= 6.0 * time(128, 0) / 128
