"""Rows of token tensors as long as the launch grid allows (65535 heads): the lanes' 32-bit offsets inside a wave's rows."""
import pytest
import torch

from tests.util import check, to_np64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,T", [("bf16", 64), ("f32", 32)])   # one whole chunk
def test_65535_heads_of_1024_columns(oracle, dtype, T):
    import paper_2409_07146_amd as gsa
    H, d_k, d_v, m = 65535, 1024, 64, 16
    dev = torch.device("cuda")
    if torch.cuda.get_device_properties(dev).total_memory < 120 << 30:
        pytest.skip("needs 100 GB")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=dev).manual_seed(3)
    r = lambda *s: torch.randn(*s, generator=gen, device=dev, dtype=dt)
    q, k, v, dO = (r(1, T, H, d).mul_(d_k ** -0.5) for d in (d_k, d_k, d_v, d_v))
    g = torch.nn.functional.logsigmoid(torch.randn(1, T, H, m, generator=gen, device=dev)) / 8
    o, z, KT, VT = gsa.gsa_fwd(q, k, v, g, final_state=True)
    grads = gsa.gsa_bwd(q, k, v, g, z, dO)
    heads = [0, 1, 4097, 65534]
    own = lambda t: to_np64(t[:, :, heads])
    a = [own(t) for t in (q, k, v, g)]
    f, b = oracle.fwd(*a), oracle.bwd(*a, own(dO))
    check("o", own(o), f["o"], dtype)
    check("KT", to_np64(KT[:, heads]), f["KT"], dtype)
    check("VT", to_np64(VT[:, heads]), f["VT"], dtype)
    for n, t in zip(("dq", "dk", "dv", "dg"), grads):
        check(n, own(t), b[n], dtype)
