"""Chunk memories of bf16 scans with 16 and 32 slots, on both sides of the line (256 workgroups, one per 64 columns of a memory, head
and sequence or segment) between loads of four chunks ahead and of two."""
import pytest

from tests.test_gpu_bwd import compare_bwd, run_fwd_bwd
from tests.util import kernel_launches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [16, 32])
@pytest.mark.parametrize("B,T,H,d_k,d_v,cu,segmented", [
    (16, 150, 8, 64, 64, None, False),       # 256 workgroups
    (16, 150, 8, 64, 128, None, False),      # 384; an odd number of chunks, the last one ragged
    (29, 1, 5, 64, 64, None, False),         # 290; a single token
    (33, 64, 4, 64, 64, None, False),        # 264; one whole chunk
    (1, 4801, 4, 640, 640, None, True),   # 80 walks of 76 chunks in three segments: 240
    (1, 6400, 4, 640, 640, None, True),   # in four: 320
    (1, 1000, 4, 576, 576, (0, 0, 1, 65, 300, 300, 1000), False),   # packed, with empty sequences: 432
])
def test_both_ways_against_the_oracle(oracle, B, T, H, d_k, d_v, cu, segmented, m):
    from paper_2409_07146_amd.synth import GsaConfig
    cfg = GsaConfig("snapshots", B=B, T=T, H=H, d_k=d_k, d_v=d_v, m=m, dtype="bf16", cu_seqlens=cu, init_state_std=0.1, seed=53)
    (x, got), launches = kernel_launches(lambda: run_fwd_bwd(cfg, with_state_grads=True))
    assert launches["scan_summary_kernel"] == (3 if segmented else 0)
    n = len(cu) - 1 if cu else B
    compare_bwd(oracle, cfg, x, got, heads=[0, H - 1], seqs=list(range(n)) if cu else [0, B - 1])
