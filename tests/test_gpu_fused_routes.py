"""The wide contractions inside the chunk kernels and in a kernel of their own, on both sides of the lines between the two,
against the fp64 oracle.  Each case states the route it takes and the kernels' own timing slots tell whether it did."""
import numpy as np
import pytest
import torch

from tests.test_gpu_variants import _inputs, _run_and_compare
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


@pytest.mark.parametrize("readout,given", [("softmax", True), ("swish", False), ("identity", True)])
@pytest.mark.parametrize("m,d_k,d_v", [(16, 64, 64), (32, 64, 128), (64, 128, 64), (128, 64, 64)])
def test_general_form_inside(oracle, m, d_k, d_v, readout, given):
    """Given intensities and element-wise read-outs, 32 (chunk, head) pairs, a ragged last chunk."""
    cfg, x = _inputs(2, 200, 4, d_k, d_v, m, "bf16", seed=91, given=given)
    for n in ("K0", "V0", "dKT", "dVT"):
        x[n] = x[n] * 0.2
    with routes() as names:
        _run_and_compare(oracle, cfg, x, readout)
    assert not names & {"apply_fwd_kernel", "apply_bwd_kernel"}


@pytest.mark.parametrize("m,given", [(32, False), (64, False), (64, True), (128, False)])
def test_gate_logits_inside(oracle, m, given):
    """gate_tau > 0: the gradient goes on to the logit before the wide contractions follow."""
    import paper_2409_07146_amd as gsa
    from scipy.special import expit, log_expit
    tau = 8.0
    cfg, x = _inputs(2, 200, 4, 64, 128, m, "bf16", seed=92, given=given)
    u = (torch.randn(x["g"].shape, generator=torch.Generator().manual_seed(93)) * 2.0).float()
    g64 = log_expit(to_np64(u)) / tau
    put = lambda t: None if t is None else t.cuda()
    d = {n: put(x[n]) for n in ("q", "k", "v", "s", "dO", "K0", "V0", "dKT", "dVT")}
    kw = dict(K0=d["K0"], V0=d["V0"], s=d["s"], gate_tau=tau)
    with routes() as names:
        o, z, _, _ = gsa.gsa_fwd(d["q"], d["k"], d["v"], u.cuda(), **kw)
        res = gsa.gsa_bwd(d["q"], d["k"], d["v"], u.cuda(), z, d["dO"], dKT=d["dKT"], dVT=d["dVT"], initial_state_grad=True, **kw)
    assert not names & {"apply_fwd_kernel", "apply_bwd_kernel"}
    a = {n: None if x[n] is None else to_np64(x[n]) for n in ("q", "k", "v", "s", "dO", "K0", "V0", "dKT", "dVT")}
    kw = dict(K0=a["K0"], V0=a["V0"], s=a["s"])
    check("o", to_np64(o), oracle.fwd(a["q"], a["k"], a["v"], g64, **kw)["o"], "bf16")
    r = oracle.bwd(a["q"], a["k"], a["v"], g64, a["dO"], dKT=a["dKT"], dVT=a["dVT"], **kw)
    r["dg"] = r["dg"] * (1.0 - expit(to_np64(u))) / tau
    for n, t in zip(("dq", "dk", "dv", "dg", "dK0", "dV0", "ds"), res):
        check(n, to_np64(t), r[n], "bf16")


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


@pytest.mark.parametrize("H,inside", [(8, False), (9, True)])     # 24 units: from 96 pairs on
def test_backward_routes(oracle, H, inside):
    from tests.test_gpu_bwd import compare_bwd, run_fwd_bwd
    from paper_2409_07146_amd.synth import GsaConfig
    cfg = GsaConfig("routes", B=1, T=64 * 11 - 5, H=H, d_k=512, d_v=512, m=64, dtype="bf16", init_state_std=0.1, seed=95)
    with routes() as names:
        x, got = run_fwd_bwd(cfg, with_state_grads=True)
    assert ("apply_bwd_kernel" not in names) == inside
    compare_bwd(oracle, cfg, x, got, heads=[0, H - 1])
