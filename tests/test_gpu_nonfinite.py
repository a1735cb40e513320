"""Infinite products and NaN gates: what they reach, and what stays finite."""
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m", [16, 64, 128])
@pytest.mark.parametrize("logits", [False, True])
@pytest.mark.parametrize("wiped", [False, True])
def test_a_nan_gate_gives_nan_outputs_of_its_head(m, dtype, logits, wiped):
    """From the token on, in its own sequence and head; wiped: in a row block that is evaluated pair by pair."""
    import paper_2409_07146_amd as gsa
    q, k, v, g = _inputs(m, dtype)
    opt = dict(gate_tau=8.0) if logits else {}
    if wiped:
        g[:, 16:32] = -8.0 * (8.0 if logits else 1.0)
    g[0, 20, 1, m // 2] = float("nan")
    o, z, KT, _ = gsa.gsa_fwd(q, k, v, g, final_state=True, **opt)
    assert torch.isnan(o[0, 20:, 1]).all() and torch.isnan(KT[0, 1, m // 2]).all()
    assert torch.isfinite(o[1]).all() and torch.isfinite(o[:, :, 0]).all() and torch.isfinite(KT[1]).all()
    dq, dk, dv, dg, _, _ = gsa.gsa_bwd(q, k, v, g, z, torch.ones_like(v), **opt)
    assert torch.isnan(dq[0, 20:, 1]).all() and torch.isfinite(dq[1]).all() and torch.isfinite(dq[:, :, 0]).all()


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("logits", [False, True])
def test_a_nan_gate_gives_nan_outputs_of_its_head_in_a_decode_step(split, logits):
    import paper_2409_07146_amd as gsa
    m, d = 64, 64
    q, k, v, g = [t[:, 0].contiguous() for t in _inputs(m, "bf16")]
    g[0, 1, 5] = float("nan")
    K, V = torch.zeros(2, 2, m, d, device="cuda"), torch.zeros(2, 2, m, d, device="cuda")
    opt = dict(gate_tau=8.0) if logits else {}
    if split:
        opt["workspace"] = gsa.alloc_decode_workspace(2, 2, d, d, m, q.device)
    o = gsa.gsa_decode_step(q, k, v, g, K, V, **opt)
    assert torch.isnan(o[0, 1]).all() and torch.isfinite(o[1]).all() and torch.isfinite(o[:, 0]).all()
    assert torch.isnan(K[0, 1, 5]).all() and torch.isfinite(K[0, 0]).all() and torch.isfinite(K[1]).all()
