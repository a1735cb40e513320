"""The write intensity 1 - exp(g) of the sequence kernels, read off a memory that one token of ones writes: to one unit in
the last place of the fp64 value, and the same bits as the decode step (a memory is handed from one to the other)."""
import numpy as np
import pytest
import torch

from tests.util import to_np64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [16, 64, 128])
@pytest.mark.parametrize("lo,hi", [(-30.0, 0.0), (-2.0, 0.0), (-0.01, 0.0)])
def test_intensity_of_a_single_write(m, lo, hi):
    import paper_2409_07146_amd as gsa
    B, H, d = 16, 8, 64
    gen = torch.Generator().manual_seed(7)
    g = (lo + (hi - lo) * torch.rand(B, 1, H, m, generator=gen)).float().cuda()
    ones = torch.ones(B, 1, H, d, device="cuda")
    _, _, KT, _ = gsa.gsa_fwd(ones, ones, ones, g, final_state=True)
    want = -np.expm1(to_np64(g)[:, 0])                      # [B, H, m]
    ulp = np.spacing(want.astype(np.float32)).astype(np.float64)
    err = np.abs(to_np64(KT) - want[..., None]) / ulp[..., None]
    assert err.max() <= 1.0, err.max()
    K, V = torch.zeros(B, H, m, d, device="cuda"), torch.zeros(B, H, m, d, device="cuda")
    gsa.gsa_decode_step(ones[:, 0], ones[:, 0], ones[:, 0], g[:, 0].contiguous(), K, V)
    assert torch.equal(K, KT)
