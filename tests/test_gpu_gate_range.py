"""Row blocks whose gates decay by close to e^80, the widest that are factored, next to ordinary slots: results are linear in
q (forward, identity read-out) and in dO (backward) over many powers of two, because neither factor of a gate may leave
fp32's range first; and wider blocks, evaluated pair by pair, keep the precision of the factored ones."""
import pytest
import torch

from tests.test_gpu_bwd import compare_bwd
from tests.util import rel_l2, to_np64

pytestmark = pytest.mark.gpu

# Scaling by a power of two changes no rounding; what may change is a term far below the sum it enters that underflows.
# It moves a sum by less than fp32's resolution, and an I/O type's rounding of it rarely.
BAR = {"f32": 1e-6, "bf16": 1e-4}


def _inputs(m, dtype, H, d_k, d_v, T=100):
    from paper_2409_07146_amd import synth
    cfg = synth.GsaConfig("range", B=1, T=T, H=H, d_k=d_k, d_v=d_v, m=m, dtype=dtype, init_state_std=0.3, seed=41)
    x = synth.make_inputs(cfg)
    g = x["g"].clone()
    g[:, 16:32, :, ::2] = -4.95      # e^-79.2 across the block, evenly
    g[:, 70:73, :, 1::4] = -25.0     # e^-75 and a little in three tokens
    x["g"] = g
    x["dKT"] = x["dVT"] = None
    return cfg, x, {n: x[n].cuda() for n in ("q", "k", "v", "g", "dO", "K0", "V0")}


# bf16: 16 (chunk, head) pairs: the wide contractions inside the chunk kernels; 2 pairs: in a kernel of their own
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,H,d_k,d_v", [(16, 8, 64, 64), (64, 8, 64, 64), (64, 1, 128, 64), (128, 8, 64, 64), (32, 1, 64, 128)])
@pytest.mark.parametrize("power", [27, -40])
def test_gradients_are_linear_in_the_output_gradient(oracle, m, H, d_k, d_v, dtype, power):
    import paper_2409_07146_amd as gsa
    cfg, x, d = _inputs(m, dtype, H, d_k, d_v)
    o, z, _, _ = gsa.gsa_fwd(d["q"], d["k"], d["v"], d["g"], K0=d["K0"], V0=d["V0"])
    run = lambda dO: gsa.gsa_bwd(d["q"], d["k"], d["v"], d["g"], z, dO, K0=d["K0"], V0=d["V0"], initial_state_grad=True)
    names = ("dq", "dk", "dv", "dg", "dK0", "dV0")
    base = dict(zip(names, run(d["dO"])))
    if dtype == "f32":   # bf16: test_gpu_wide_gates.py
        compare_bwd(oracle, cfg, x, dict(base, o=o), heads=[0])
    for n, t in zip(names, run(d["dO"] * 2.0 ** power)):
        assert torch.isfinite(t).all(), n
        assert rel_l2(to_np64(t) * 2.0 ** -power, to_np64(base[n])) <= BAR[dtype], n


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m", [16, 32, 64, 128])
@pytest.mark.parametrize("power", [30, -50])
def test_identity_readout_is_linear_in_q(m, dtype, power):
    import paper_2409_07146_amd as gsa
    cfg, x, d = _inputs(m, dtype, 2, 128, 64)
    run = lambda q: gsa.gsa_fwd(q, d["k"], d["v"], d["g"], K0=d["K0"], V0=d["V0"], readout="identity")[:2]
    for n, t, b in zip(("o", "z"), run(d["q"] * 2.0 ** power), run(d["q"])):
        assert torch.isfinite(t).all(), n
        assert rel_l2(to_np64(t) * 2.0 ** -power, to_np64(b)) <= BAR[dtype], n


@pytest.mark.parametrize("m", [16, 32, 64, 128])
def test_pair_by_pair_blocks_keep_the_rest_of_the_products(oracle, m):
    """One block, every slot wiped at every token, no initial memory: z is a sum of products of bf16 numbers, exact in fp32,
    with fp32 weights.  Product and rest together hold 16 bits of it; the product alone would hold 8 (error about 1e-3)."""
    import paper_2409_07146_amd as gsa
    from paper_2409_07146_amd import synth
    x = synth.make_inputs(synth.GsaConfig("wiped", B=1, T=16, H=2, d_k=128, d_v=64, m=m, dtype="bf16", seed=43))
    g = x["g"] * 4.0 - 6.0
    _, z, _, _ = gsa.gsa_fwd(x["q"].cuda(), x["k"].cuda(), x["v"].cuda(), g.cuda())
    ref = oracle.fwd(*(to_np64(t) for t in (x["q"], x["k"], x["v"], g)))["z"]
    assert rel_l2(to_np64(z), ref) <= 2.0 ** -15
