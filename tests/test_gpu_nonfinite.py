"""Infinite products: what they reach, and what stays finite."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(m, dtype, T=50, H=2, d=64):
    from paper_2409_07146_amd import synth
    x = synth.make_inputs(synth.GsaConfig("inf", B=2, T=T, H=H, d_k=d, d_v=d, m=m, dtype=dtype, seed=47))
    return [x[n].cuda() for n in ("q", "k", "v", "g")]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m", [16, 64, 128])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_a_score_that_overflows_is_infinite_with_its_sign(m, dtype, sign):
    import paper_2409_07146_amd as gsa
    q, k, v, g = _inputs(m, dtype)
    for t, r in ((20, 7), (40, 39)):      # another row block, the same row block
        q2, k2 = q.clone(), k.clone()
        q2[0, t, 0] = 1e20
        k2[0, r, 0] = sign * 1e20
        _, z, _, _ = gsa.gsa_fwd(q2, k2, v, g)
        assert (z[0, t, 0] == sign * float("inf")).all()
        z[0, t, 0] = 0.0
        assert torch.isfinite(z).all()
