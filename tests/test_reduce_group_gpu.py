"""Products of eight signatures at a time (sig_reduce_group.hip) inside the chunked scan: counts that leave 2, 4 or 8 for the last launch, words that
fill a workgroup's threads or not, several workgroups to a product, both types.

Against the oracle level by level.  A product rounds as the tree's does and the running sums keep what they round off: the scan's own 2^-24
sqrt(increments) stays the larger part, 5e-6 is ten times that at 300."""
import numpy as np
import pytest

import paper_2001_00706_amd as sig
from oracle import sig_oracle as orc
from paper_2001_00706_amd.inputs import brownian_paths

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("B,chunks,d,N", [(1, 16, 4, 6), (2, 32, 4, 6), (1, 64, 4, 6), (1, 128, 2, 8), (3, 64, 3, 6), (1, 32, 5, 5), (1, 16, 6, 4), (2, 32, 7, 4),
                                          (1, 16, 8, 4), (1, 512, 3, 4), (1, 256, 6, 3)])
def test_chunked_scan(B, chunks, d, N, dtype):
    import torch
    x = brownian_paths(B, 2 * chunks + 1, d, seed=d).astype(dtype)
    out = torch.full((B, orc.channels(d, N)), float("nan"), device="cuda:0", dtype=getattr(torch, np.dtype(dtype).name))
    got = sig.sig_forward_chunked(torch.from_numpy(x).to("cuda:0"), N, chunks, out=out).cpu().numpy()
    want = orc.signature(x.astype(np.float64), N)
    at = 0
    for k in range(1, N + 1):
        a, b = got[:, at:at + d ** k], want[:, at:at + d ** k]
        at += d ** k
        assert np.linalg.norm(a - b) <= (5e-6 if dtype == np.float32 else 1e-13) * np.linalg.norm(b), k
