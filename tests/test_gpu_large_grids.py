"""A call of more tiles than one launch holds (400,000 rows: 19.5 million 64 x 64
tiles of 256 threads, where HIP takes fewer than 2^32 work-items)."""
import pytest

import paper_1705_08213_amd as ccc
from gpu_util import say

pytestmark = pytest.mark.gpu


def test_selection_past_one_launch():
    """Random rows, which correlate nowhere near the threshold, with pairs of
    planted rows that do: one entry 0.5 (1 - 1/3)^2 = 0.222 per planted pair's
    (0,0) and (1,1), spread over the triangle from its first to its last tile."""
    import torch
    n_v, n_f = 400000, 1000
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    lo = torch.randint(0, 256, (n_v, 256), dtype=torch.uint8, device="cuda", generator=g) & 0x55
    hi = torch.randint(0, 256, (n_v, 256), dtype=torch.uint8, device="cuda", generator=g) & 0xAA
    v = lo | (hi & (lo << 1))  # codes 00, 01, 11
    pairs = [(0, 1), (0x1F, 399999), (77, 150000), (200000, 200001), (234567, 385400),
             (370688, 370689), (399990, 399998)]
    for k, (i, j) in enumerate(pairs):  # half the fields 11, half 00, another pattern each
        bits = torch.randint(0, 2, (1024,), dtype=torch.uint8, generator=torch.Generator().manual_seed(k))
        row = (bits.view(256, 4) * torch.tensor([3, 12, 48, 192], dtype=torch.uint8)).sum(1)
        v[i] = v[j] = row.to(torch.uint8).cuda()
    want = sorted(i * n_v - i * (i + 1) // 2 + (j - i - 1) for i, j in pairs)
    say("2way select past one launch", n_v, n_f)
    n, index, _, _ = ccc.ccc_2way_select(v, n_f, 0.2, 1000)
    assert n == len(want)
    assert sorted(index.cpu().tolist()) == want
