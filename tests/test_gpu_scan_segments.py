"""Scans of batches that are cut into segments of 8, 16 or 32 chunks and of packed batches, against the fp64 oracle; and calls with a
workspace that has no room for the segments' summaries."""
import pytest
import torch

from tests.test_gpu_bwd import DEV, compare_bwd, run_fwd_bwd
from tests.util import kernel_launches, rel_l2, to_np64

pytestmark = pytest.mark.gpu

# chunks are 64 tokens (bf16) or 32 (fp32); H*(d_k+d_v)/64 workgroups per sequence
SHAPES = [
    ("bf16", 1, 24 * 64, 2, 64, 128, 32),        # the shortest sequence that is cut: three segments of eight
    ("bf16", 2, 24 * 64 + 1, 1, 128, 64, 16),    # a fourth segment of one token
    ("f32", 1, 31 * 32 + 5, 2, 64, 64, 64),      # a short last segment
    ("bf16", 2, 48 * 64 + 7, 5, 64, 256, 64),   # too many workgroups for segments of eight: sixteen
    ("bf16", 1, 23 * 64 + 63, 2, 64, 64, 128),   # 24 chunks, the last one ragged; 128 slots
]
# too many workgroups for those: segments of 32 chunks
LONG = [
    ("bf16", 1, 75 * 64 + 1, 4, 640, 640, 16),   # 80 workgroups, three segments
    ("bf16", 1, 97 * 64 + 5, 3, 1024, 1024, 64), # 96 in four: 384, more than one per CU
    ("bf16", 3, 70 * 64, 2, 512, 512, 128),
    ("f32", 2, 70 * 32, 2, 512, 640, 16),
    ("f32", 1, 65 * 32 + 3, 4, 512, 640, 32),
    ("f32", 1, 66 * 32 + 3, 4, 640, 640, 64),
    ("f32", 1, 70 * 32, 4, 512, 512, 128),
]
# packed: lengths, then as above
PACKED = [
    ((64 * 78 + 8, 1, 64 * 73, 300), "bf16", 2, 64, 128, 64),
    ((64 * 100,) + tuple(range(1, 10)), "bf16", 3, 320, 320, 32),   # 300 workgroups without segments: two chunks ahead
    ((70, 64 * 65, 0), "bf16", 2, 64, 64, 128),
    ((32 * 69, 0, 32 * 71 + 1, 7), "f32", 2, 64, 64, 16),
    ((32 * 66, 33), "f32", 2, 128, 64, 32),
    ((5, 32 * 67 + 30), "f32", 1, 64, 64, 64),
    ((32 * 65, 32 * 40), "f32", 2, 64, 64, 128),
]


def _cfg(shape, cu=None):
    from paper_2409_07146_amd.synth import GsaConfig
    dtype, B, T, H, d_k, d_v, m = shape
    return GsaConfig("segments", B=B, T=T, H=H, d_k=d_k, d_v=d_v, m=m, dtype=dtype, init_state_std=0.1, cu_seqlens=cu, seed=23)


@pytest.mark.parametrize("shape", SHAPES + LONG)
def test_segments_against_the_oracle(oracle, shape):
    cfg = _cfg(shape)
    (x, got), launches = kernel_launches(lambda: run_fwd_bwd(cfg, with_state_grads=True))
    assert launches["scan_summary_kernel"] == 3   # forward, the backward's recomputation, reverse
    compare_bwd(oracle, cfg, x, got, heads=[0, cfg.H - 1], seqs=[cfg.B - 1])


@pytest.mark.parametrize("case", PACKED)
def test_packed_segments_against_the_oracle(oracle, case):
    lens, dtype, H, d_k, d_v, m = case
    cu = (0,) + tuple(sum(lens[:i + 1]) for i in range(len(lens)))
    cfg = _cfg((dtype, 1, cu[-1], H, d_k, d_v, m), cu)
    (x, got), launches = kernel_launches(lambda: run_fwd_bwd(cfg, with_state_grads=True))
    assert launches["scan_summary_kernel"] == 3
    compare_bwd(oracle, cfg, x, got, heads=[H - 1])


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
