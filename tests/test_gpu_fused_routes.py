"""The wide contractions inside the chunk kernels and in a kernel of their own, on both sides of the lines between the two,
against the fp64 oracle.  Each case states the route it takes and the kernels' own timing slots tell whether it did."""
import numpy as np
import pytest
import torch

from tests.util import check, to_np64

pytestmark = pytest.mark.gpu


class routes:
    """Names of the kernels launched inside the block."""
    def __enter__(self):
        from paper_2409_07146_amd import api
        torch.cuda.synchronize()
        api.gsa_profile_enable(True)
        api.gsa_profile_reset()
        self.names = set()
        return self.names

    def __exit__(self, *exc):
        from paper_2409_07146_amd import api
        torch.cuda.synchronize()
        self.names.update(n for n, (_, launches) in api.gsa_profile_read().items() if launches)
        api.gsa_profile_enable(False)


@pytest.mark.parametrize("m,H,chunks,d_v,inside", [
    (16, 1, 1, 576, True), (64, 1, 1, 640, False),          # up to 9 units always, more units with few pairs not
    (64, 11, 13, 640, False), (64, 9, 16, 640, True),       # 143 and 144 pairs
    (128, 5, 19, 1024, False), (128, 6, 16, 1024, True),    # 95 and 96 with 128 slots
    (32, 27, 19, 768, True), (32, 27, 19, 832, False),      # 513 pairs: up to 12 units
    (64, 32, 16, 1024, True), (64, 27, 19, 1024, False),    # 512 and 513
])
def test_forward_routes(oracle, m, H, chunks, d_v, inside):
    import paper_2409_07146_amd as gsa
    from paper_2409_07146_amd import synth
    T = 64 * chunks - 23
    x = synth.make_inputs(synth.GsaConfig("routes", B=1, T=T, H=H, d_k=64, d_v=d_v, m=m, dtype="bf16", init_state_std=0.1, seed=94))
    with routes() as names:
        o, _, _, _ = gsa.gsa_fwd(*(x[n].cuda() for n in ("q", "k", "v", "g")), K0=x["K0"].cuda(), V0=x["V0"].cuda())
    assert ("apply_fwd_kernel" not in names) == inside
    for h in {0, H - 1}:
        one = lambda t: np.ascontiguousarray(to_np64(t)[:, :, h:h + 1])
        st = lambda t: np.ascontiguousarray(to_np64(t)[:, h:h + 1])
        ref = oracle.fwd(one(x["q"]), one(x["k"]), one(x["v"]), one(x["g"]), K0=st(x["K0"]), V0=st(x["V0"]))["o"]
        check("o, head %d" % h, one(o), ref, "bf16")
