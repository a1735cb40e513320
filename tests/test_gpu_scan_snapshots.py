"""Chunk memories of bf16 scans with 16 and 32 slots, whose snapshots leave by two ways: straight from the registers (up to 256
workgroups, one per 64 columns of a memory, head and sequence or segment) and through LDS (beyond)."""
import pytest

from tests.test_gpu_bwd import compare_bwd, run_fwd_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [16, 32])
@pytest.mark.parametrize("B,T,H,d_k,d_v,cu", [
    (16, 150, 8, 64, 64, None),       # 256 workgroups
    (16, 150, 8, 64, 128, None),      # 384; an odd number of chunks, the last one ragged
    (29, 1, 5, 64, 64, None),         # 290; a single token
    (33, 64, 4, 64, 64, None),        # 264; one whole chunk
    (1, 3300, 4, 640, 640, None),     # 80 walks in two segments of 32 chunks: 160
    (2, 3300, 4, 640, 640, None),     # 320 in segments
    (1, 1000, 4, 576, 576, (0, 0, 1, 65, 300, 300, 1000)),   # packed, with empty sequences: 432
])
def test_both_ways_against_the_oracle(oracle, B, T, H, d_k, d_v, cu, m):
    from paper_2409_07146_amd.synth import GsaConfig
    cfg = GsaConfig("snapshots", B=B, T=T, H=H, d_k=d_k, d_v=d_v, m=m, dtype="bf16", cu_seqlens=cu, init_state_std=0.1, seed=53)
    x, got = run_fwd_bwd(cfg, with_state_grads=True)
    n = len(cu) - 1 if cu else B
    compare_bwd(oracle, cfg, x, got, heads=[0, H - 1], seqs=list(range(n)) if cu else [0, B - 1])
