"""Scans of batches that are cut into segments of 8 or 16 chunks, against the fp64 oracle; and the same calls with a
workspace that has no room for the segments' summaries."""
import pytest
import torch

from tests.test_gpu_bwd import DEV, compare_bwd, run_fwd_bwd
from tests.util import rel_l2, to_np64

pytestmark = pytest.mark.gpu

# chunks are 64 tokens (bf16) or 32 (fp32); H*(d_k+d_v)/64 workgroups per sequence
SHAPES = [
    ("bf16", 1, 24 * 64, 2, 64, 128, 32),        # the shortest sequence that is cut: three segments of eight
    ("bf16", 2, 24 * 64 + 1, 1, 128, 64, 16),    # a fourth segment of one token
    ("f32", 1, 31 * 32 + 5, 2, 64, 64, 64),      # a short last segment
    ("bf16", 2, 48 * 64 + 7, 5, 64, 256, 64),   # too many workgroups for segments of eight: sixteen
    ("bf16", 1, 23 * 64 + 63, 2, 64, 64, 128),   # 24 chunks, the last one ragged; 128 slots
]


def _cfg(shape):
    from paper_2409_07146_amd.synth import GsaConfig
    dtype, B, T, H, d_k, d_v, m = shape
    return GsaConfig("segments", B=B, T=T, H=H, d_k=d_k, d_v=d_v, m=m, dtype=dtype, init_state_std=0.1, seed=23)


@pytest.mark.parametrize("shape", SHAPES)
def test_short_segments_against_the_oracle(oracle, shape):
    cfg = _cfg(shape)
    x, got = run_fwd_bwd(cfg, with_state_grads=True)
    compare_bwd(oracle, cfg, x, got, heads=[0, cfg.H - 1], seqs=[cfg.B - 1])


@pytest.mark.parametrize("shape", SHAPES[:3])
def test_workspace_without_room_for_the_summaries(shape):
    """The summaries are the last thing in a workspace: segments * (m * (d_k + d_v) + m * slices) floats per (sequence,
    head).  Without them the scans walk whole sequences; a byte less than that is refused."""
    import paper_2409_07146_amd as gsa
    cfg = _cfg(shape)
    x, got = run_fwd_bwd(cfg)
    d = {n: None if x[n] is None else x[n].to(torch.device(DEV)) for n in ("q", "k", "v", "g", "dO", "K0", "V0")}
    p = gsa.make_problem(d["q"], d["v"], d["g"])
    chunks = -(-cfg.T // (64 if cfg.dtype == "bf16" else 32))
    recs = cfg.B * cfg.H * -(-chunks // 8) * cfg.m
    up = lambda n: -(-n // 256) * 256
    summaries = up(4 * recs * (cfg.d_k + cfg.d_v)) + up(4 * recs * ((cfg.d_k + cfg.d_v) // 64))
    ws = {bwd: torch.empty(gsa.gsa_workspace_bytes(p, bwd) - summaries, dtype=torch.uint8, device=DEV) for bwd in (False, True)}
    o, z, KT, VT = gsa.gsa_fwd(d["q"], d["k"], d["v"], d["g"], K0=d["K0"], V0=d["V0"], final_state=True, workspace=ws[False])
    grads = gsa.gsa_bwd(d["q"], d["k"], d["v"], d["g"], z, d["dO"], K0=d["K0"], V0=d["V0"], initial_state_grad=True, workspace=ws[True])
    # both forms round the same sums to the I/O type once: they differ by its resolution (2^-9) at most, in fp32 by sums in another order
    bar = 4e-3 if cfg.dtype == "bf16" else 1e-5
    for n, t in zip(("o", "KT", "VT", "dq", "dk", "dv", "dg", "dK0", "dV0"), (o, KT, VT) + tuple(grads)):
        assert rel_l2(to_np64(t), to_np64(got[n])) <= bar, n
    with pytest.raises(gsa.GsaError):
        gsa.gsa_fwd(d["q"], d["k"], d["v"], d["g"], workspace=ws[False][:-1])
