"""The fused LayerNorm's two-row workgroups (calls of 140000 elements per CU
and more, rows of 6160 to 32768 channels): codes bit for bit those of the
one-row workgroups, which take the same rows in shorter calls, and of the
oracle on a few of them."""
import numpy as np
import pytest
import torch

from oracle import ot_oracle as O
from paper_2406_18832_amd import ot

pytestmark = pytest.mark.gpu


# one width per chunk count and workgroup size, whole and ragged against the
# threads, the narrowest and the widest; an odd number of rows throughout
@pytest.mark.parametrize("K", [6160, 8192, 8208, 12288, 12304, 16384, 16400, 18432, 20480,
                               24560, 28672, 32768])
def test_row_pairs_match_single_rows(K):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    M = -(-140000 * cus // K) | 1
    print(f"[case] ln_quantize row pairs M={M} K={K}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(K)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda")

    h = (normal(M, K) * (normal(K).abs() + 0.1) + normal(K)).half()
    # rows that take the exact sums, next to rows that do not: a mean of 0,
    # constants, and a first value far from the others
    h[0, : K // 2] = 1.5
    h[0, K // 2:] = -1.5
    h[3] = 0.0
    h[4] = 3.0
    h[M - 1, 0] = 60000.0
    gamma, beta, z = normal(K).half(), normal(K).half(), normal(K)
    inv_s = normal(K).abs() * 20 + 0.1
    got = ot.ln_quantize_act(h, gamma, beta, 1e-5, 8, z, inv_s)
    parts = M // 3  # below the line
    ref = torch.cat([ot.ln_quantize_act(h[i: i + parts].contiguous(), gamma, beta, 1e-5, 8, z,
                                        inv_s) for i in range(0, M, parts)])
    torch.cuda.synchronize()
    assert torch.equal(got, ref)
    rows = [0, 1, 2, 3, 4, M - 2, M - 1]
    n = [t.cpu().numpy() for t in (h[rows], gamma, beta, z, inv_s)]
    assert np.array_equal(got[rows].cpu().numpy(), O.ln_quantize_act(n[0], n[1], n[2], 1e-5, n[3],
                                                                    n[4], 8))
