"""Row blocks whose gates are too wide to be factored next to ordinary ones, at every slot count and at ragged lengths,
with the wide contractions inside the chunk kernels (odd and even numbers of 64-column units) and in a kernel of their
own, against the fp64 oracle (forward and backward)."""
import pytest

from tests.test_gpu_bwd import compare_bwd, run_fwd_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,T,H,d_k,d_v", [
    # bf16, inside: at least 4 * (2*d_k + d_v)/64 (chunk, head) pairs
    (16, 65, 4, 64, 128), (32, 96, 4, 64, 64), (64, 129, 4, 128, 64), (64, 47, 8, 64, 128), (128, 80, 4, 64, 128), (64, 350, 4, 192, 320),
    (64, 129, 1, 64, 128),   # too few pairs: the backward's wide contractions run on their own
])
def test_wide_and_ordinary_row_blocks(oracle, m, T, H, d_k, d_v, dtype):
    from paper_2409_07146_amd.synth import GsaConfig
    cfg = GsaConfig("wide", B=2, T=T, H=H, d_k=d_k, d_v=d_v, m=m, dtype=dtype, init_state_std=0.5, seed=29)

    def override(g):
        out = g.clone()
        out[:, 18:44, :, 1::5] = -25.0   # e^-350 across the block that starts at 16, ordinary slots beside it
        out[:, 4:7, :, ::4] = -25.0      # e^-75 and a little: the widest block that is still factored
        out[1, 40:46, :, 2] = -300.0     # below the documented floor of -30
        return out

    x, got = run_fwd_bwd(cfg, with_state_grads=True, g_override=override)
    compare_bwd(oracle, cfg, x, got)
