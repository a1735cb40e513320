"""The work whose speed this repository is judged by: decode steps, forward calls and training steps of
Gated Slot Attention, each through the public entry points of paper_2409_07146_amd.

Sizes are the workloads of paper_2409_07146_amd/synth.py and bench.py (H = 4 or 5 heads, head dimensions 64 to
640, 16 to 128 slots, 2K to 16K tokens, decode batches 1 to 64) and generic odd ones between them.  Inputs have
the distributions of synth.make_inputs, drawn on the GPU.
"""
import torch

import paper_2409_07146_amd as gsa

TAU = 8.0   # the layer's gate is alpha = sigmoid(W x)^(1/8)

# kind        decode | forward | train
# layer       the options a GSA layer switches on: gate logits and raw projections (Swish feature map) go in
# workspace   decode: the split form for small batches (gsa_decode_step_ws); 0: gsa_decode_step
# layers      decode: memories of that many layers, one token through all of them replayed from a HIP graph; 0: one call
# final       forward: final memories out and no scores saved, as a prefill does
# keep        train: the forward's memories are kept for the backward (recompute=False)
# lengths     packed sequences of these lengths (then B = 1 and T is their sum); "" = a batch of equal lengths
_DEFAULTS = dict(B=1, T=1, H=4, d_k=512, d_v=512, m=64, dtype="bf16", layer=False, workspace=False, layers=0,
                 final=False, keep=False, lengths="")


def _case(name, kind, **kw):
    c = dict(_DEFAULTS, kind=kind, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # generation at batch 1, one layer's step called from Python: the smallest call there is
        _case("decode_b1", "decode", workspace=True),
        # generation at batch 1 as it is served: one token through the 24 layers of the 1.3B model, HIP graph
        _case("decode_b1_24_layers", "decode", workspace=True, layers=24),
        # a serving batch between the two, five heads, fp32, the layer's element-wise options inside
        _case("decode_b12_h5_layer_f32", "decode", B=12, H=5, dtype="f32", workspace=True, layer=True),
        # the decode workload of bench.py: batch 64, 134 MB of memories read and written
        _case("decode_b64", "decode", B=64),
        # the smallest forward workload: one head, 16 slots, fp32 (latency and launches)
        _case("fwd_tiny_f32", "forward", T=256, H=1, d_k=64, d_v=64, m=16, dtype="f32"),
        # prefill of one 2048-token prompt, final memories out (bench.py --workload prefill_decode)
        _case("prefill_2k", "forward", T=2048, final=True),
        # the forward-only workload: narrow heads, eight sequences
        _case("fwd_d128", "forward", B=8, T=2048, d_k=128, d_v=128),
        # a small odd training step in fp32: ragged tails, d_k != d_v, 32 slots
        _case("train_small_f32", "train", B=3, T=333, H=2, d_k=192, d_v=128, m=32, dtype="f32"),
        # the 1.3B layer's training step (the workload bench.py reports), memories recomputed in the backward
        _case("train_1p3b", "train", B=8, T=2048),
        # the 2.7B layer's training step with the forward's memories kept; the largest
        _case("train_2p7b_keep", "train", B=8, T=2048, d_k=640, d_v=640, keep=True),
        # a packed long-context batch with odd lengths
        _case("train_packed_16k", "train", T=16384, lengths="8191,4097,2050,2046"),
        # the ablation with 128 slots inside a layer: raw projections and gate logits go in, lengths not a multiple of a chunk
        _case("train_m128_layer", "train", B=4, T=1000, m=128, layer=True),
    ]


_LARGEST = 16384 * 4 * 1280   # tokens x heads x (d_k + d_v) of the largest training step


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["decode", "forward", "train"])
    d = [64, 128, 192, 256, 320, 384, 448, 512, 576, 640]
    c = dict(H=rng.choice([1, 2, 3, 4, 4, 5, 8]), d_k=rng.choice(d), d_v=rng.choice(d), m=rng.choice([16, 32, 64, 64, 64, 128]),
             dtype=rng.choice(["bf16", "bf16", "f32"]), layer=rng.random() < 0.3)
    if rng.random() < 0.6:
        c["d_v"] = c["d_k"]
    if kind == "decode":
        per = c["H"] * c["m"] * (c["d_k"] + c["d_v"])
        c["B"] = _log_int(rng, 1, max(1, min(128, 64 * 4 * 64 * 1024 // per)))
        c["workspace"] = rng.random() < 0.6
        return _case("", kind, **c)
    # cost per token and head grows with the slots beyond 64, and four times with fp32
    most = _LARGEST // (c["H"] * (c["d_k"] + c["d_v"])) * 64 // max(64, c["m"])
    most = min(32768, most // 4 if c["dtype"] == "f32" else most)
    tokens = _log_int(rng, 128, most)
    if rng.random() < 0.25:
        n = rng.randint(2, 6)
        cuts = sorted(rng.sample(range(1, tokens), n - 1))
        c["lengths"] = ",".join(str(b - a) for a, b in zip([0] + cuts, cuts + [tokens]))
        c["T"] = tokens
    else:
        c["B"] = min(_log_int(rng, 1, 16), max(1, tokens // 64))
        c["T"] = max(1, tokens // c["B"])
    if kind == "forward":
        c["final"] = rng.random() < 0.5
    else:
        c["keep"] = rng.random() < 0.3
    return _case("", kind, **c)


def _inputs(gen, case, lead):
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[case["dtype"]]
    H, d_k, d_v, m = case["H"], case["d_k"], case["d_v"], case["m"]

    def normal(*shape):
        return torch.randn(*lead, *shape, generator=gen, device="cuda")

    s = 1.0 if case["layer"] else d_k ** -0.5   # raw projections are of order one; phi(q), phi(k) then meet scale 1/sqrt(d_k)
    q, k, v = (normal(H, d_k) * s).to(dt), (normal(H, d_k) * s).to(dt), (normal(H, d_v) * s).to(dt)
    u = normal(H, m)
    g = u if case["layer"] else torch.nn.functional.logsigmoid(u) / TAU
    return dict(q=q, k=k, v=v, g=g.contiguous())


def _options(case):
    if not case["layer"]:
        return {}
    return dict(scale=case["d_k"] ** -0.5, gate_tau=TAU, feature_map="swish")


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    B, T, H, d_k, d_v, m = (case[n] for n in ("B", "T", "H", "d_k", "d_v", "m"))
    opt = _options(case)
    if case["kind"] == "decode":
        n = max(1, case["layers"])
        x = _inputs(gen, case, (B,))
        states = [(torch.randn(B, H, m, d_k, generator=gen, device="cuda") * 0.1,
                   torch.randn(B, H, m, d_v, generator=gen, device="cuda") * 0.1) for _ in range(n)]
        if case["workspace"]:
            opt["workspace"] = gsa.alloc_decode_workspace(B, H, d_k, d_v, m, torch.device("cuda"))
        if not case["layers"]:
            return dict(kind="decode", x=x, K=states[0][0], V=states[0][1], opt=opt)
        outs = [torch.empty_like(x["v"]) for _ in range(n)]

        def token(mem):
            for (K, V), out in zip(mem, outs):
                gsa.gsa_decode_step(x["q"], x["k"], x["v"], x["g"], K, V, out=out, **opt)

        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):   # first use outside the capture
            token([(states[0][0].clone(), states[0][1].clone())])
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            token(states)
        return dict(kind="decode_graph", x=x, opt=opt, graph=graph, outs=outs, states=states)
    x = _inputs(gen, case, (B, T))
    cu = None
    if case["lengths"]:
        ends = [0]
        for n in case["lengths"].split(","):
            ends.append(ends[-1] + int(n))
        cu = torch.tensor(ends, dtype=torch.int32, device="cuda")
    opt["cu_seqlens"] = cu
    if case["kind"] == "forward":
        problem = gsa.make_problem(x["q"], x["v"], x["g"], 1.0, cu)
        opt.update(workspace=gsa.alloc_workspace(problem, False, torch.device("cuda")), final_state=case["final"],
                   save_z=not case["final"])
        return dict(kind="forward", x=x, opt=opt)
    dO = torch.randn(B, T, H, d_v, generator=gen, device="cuda").to(x["v"].dtype)
    for t in x.values():
        t.requires_grad_(True)
    opt["recompute"] = not case["keep"]
    return dict(kind="train", x=x, opt=opt, dO=dO)


def run(state):
    x, opt = state["x"], state["opt"]
    if state["kind"] == "decode_graph":
        state["graph"].replay()
        return state["outs"], [t for pair in state["states"][::8] for t in pair]
    if state["kind"] == "decode":
        o = gsa.gsa_decode_step(x["q"], x["k"], x["v"], x["g"], state["K"], state["V"], **opt)
        return o, state["K"], state["V"]
    if state["kind"] == "forward":
        return gsa.gsa_fwd(x["q"], x["k"], x["v"], x["g"], **opt)
    o = gsa.gsa_attention(x["q"], x["k"], x["v"], x["g"], **opt)
    return (o,) + torch.autograd.grad(o, (x["q"], x["k"], x["v"], x["g"]), state["dO"])


def work(case):
    """Every tensor a call is given read once, every one it returns written once.  FLOPs: the recurrence itself
    (update and read-out of both memories; twice that again for the gradients), whatever the chunk size."""
    esz = 2 if case["dtype"] == "bf16" else 4
    d_k, d_v, m, H = case["d_k"], case["d_v"], case["m"], case["H"]
    heads = case["B"] * case["T"] * H
    mem = m * (d_k + d_v)
    small = (2 * d_k + 2 * d_v) * esz + 4 * m   # q, k, v, g in and o out
    if case["kind"] == "decode":
        n = case["B"] * H * max(1, case["layers"])
        return dict(bytes=n * (2 * 4 * mem + small), flops=n * 4 * mem)
    if case["kind"] == "forward":
        seqs = len(case["lengths"].split(",")) if case["lengths"] else case["B"]
        extra = seqs * H * 4 * mem if case["final"] else heads * 4 * m
        return dict(bytes=heads * small + extra, flops=heads * 4 * mem)
    backward = (4 * d_k + 3 * d_v) * esz + 3 * 4 * m   # q, k, v, dO, g, scores in; dq, dk, dv, dg out
    return dict(bytes=heads * (small + 4 * m + backward), flops=heads * 12 * mem)


def tolerance(case):
    """About four times the distance of these entry points from the fp64 recurrence (oracle/), over the listed cases
    and a few drawn ones.  fp32: 2-norm up to 6e-7, largest difference 1e-5 (decode 1.2e-7 and 6e-7).  bf16: forward
    and decode 2.5e-3 and 2e-2, gradients 5.2e-3 and 6e-2."""
    decode = case["kind"] == "decode"
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 5e-6} if decode else {"rel": 5e-6, "max": 1e-4}
    if decode:
        return {"rel": 7e-3, "max": 2e-2}
    return {"rel": 1e-2, "max": 8e-2} if case["kind"] == "forward" else {"rel": 1.5e-2, "max": 0.2}
