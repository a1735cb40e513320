"""Packed batches on both sides of the rule that decides, on the device, whether the scans walk their sequences whole or in segments:
what it decided, and every sequence against a call of its own."""
import pytest
import torch

from tests.util import kernel_launches, rel_l2, to_np64

pytestmark = pytest.mark.gpu

B16, F32 = torch.bfloat16, torch.float32
CHUNK = {B16: 64, F32: 32}
# lengths in tokens as a function of the chunk, type, slots, heads, d_k, d_v; segments of all sequences and chunks per segment as the device
# has them, or None where the host knows that no sequence is cut
CASES = [
    (lambda C: (72 * C,), B16, 16, 2, 64, 64, None),                            # the longest of the first side, as the host sees it
    (lambda C: (72 * C, 63 * C + 1), B16, 16, 2, 64, 64, (2, 72)),              # the host provides for 136 chunks in one sequence
    (lambda C: (72 * C + 1, 63 * C), B16, 16, 2, 64, 64, (3 + 2, 32)),          # one token more
    (lambda C: (1, 0, 72 * C, 100 * C + 3, 5), B16, 16, 1, 64, 128, (1 + 1 + 3 + 4 + 1, 32)),   # an empty and two tiny sequences
    (lambda C: (0, 75 * C - 7, 75 * C, 70 * C) + (60 * C,) * 4, B16, 16, 4, 256, 256, (8, 75)),   # 459 chunks * 32 workgroups = 133 * 110
    (lambda C: (68 * C, 20 * C), B16, 64, 1, 64, 64, (2, 68)),
    (lambda C: (68 * C + 1, 20 * C), B16, 64, 1, 64, 64, (3 + 1, 32)),
    (lambda C: (64 * C, 30 * C + 1), F32, 128, 1, 64, 64, (2, 64)),
    (lambda C: (64 * C + 1, 30 * C), F32, 128, 1, 64, 64, (3 + 1, 32)),
    # many steps a chunk: up to 96 chunks whole from 110 on, any number from 160 on
    (lambda C: (96 * C, 96 * C), F32, 64, 8, 256, 256, (2, 96)),
    (lambda C: (96 * C + 1, 96 * C), F32, 64, 8, 256, 256, (4 + 3, 32)),
    (lambda C: (100 * C - 5,) * 3, F32, 64, 8, 256, 256, (3, 100)),
]


def _decision(workspace, T, n, C):
    """(segments, chunks per segment) from the tables at the start of the workspace: four ints per chunk and per sequence, then the
    segments before each sequence and in all, and the chunks per segment."""
    up = lambda b: -(-b // 256) * 256
    at = up(16 * (T // C + n)) + up(16 * n)
    return tuple(workspace[at:at + 4 * (n + 2)].view(torch.int32).tolist()[-2:])


@pytest.mark.parametrize("case", range(len(CASES)))
def test_packed_against_single_sequences(case):
    import paper_2409_07146_amd as gsa
    lens, dtype, m, H, d_k, d_v, decided = CASES[case]
    C = CHUNK[dtype]
    lens = lens(C)
    T, dev = sum(lens), torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(5)
    t = lambda *s: torch.randn(*s, generator=gen, device=dev)
    q, k, v, dO = (t(1, T, H, d).mul_(d_k ** -0.5).to(dtype) for d in (d_k, d_k, d_v, d_v))
    g = torch.nn.functional.logsigmoid(t(1, T, H, m)) / 8
    K0, V0 = t(len(lens), H, m, d_k) * 0.1, t(len(lens), H, m, d_v) * 0.1
    ends = [0]
    for n in lens:
        ends.append(ends[-1] + n)
    cu = torch.tensor(ends, dtype=torch.int32, device=dev)
    ws = gsa.alloc_workspace(gsa.make_problem(q, v, g, 1.0, cu), False, dev).fill_(255)
    (o, z, KT, VT), launches = kernel_launches(lambda: gsa.gsa_fwd(q, k, v, g, K0=K0, V0=V0, cu_seqlens=cu, final_state=True, workspace=ws))
    assert launches["scan_summary_kernel"] == (decided is not None)
    assert _decision(ws, T, len(lens), C) == (decided or (-1, -1))
    grads = gsa.gsa_bwd(q, k, v, g, z, dO, K0=K0, V0=V0, cu_seqlens=cu, initial_state_grad=True)
    for i, n in enumerate(lens):
        own, st = slice(ends[i], ends[i + 1]), slice(i, i + 1)
        if n == 0:   # hands its memories through
            assert torch.equal(KT[st], K0[st]) and torch.equal(VT[st], V0[st]) and not grads[4][st].any() and not grads[5][st].any()
            continue
        s = [x[:, own].contiguous() for x in (q, k, v, g, dO)]
        ro, rz, rK, rV = gsa.gsa_fwd(*s[:4], K0=K0[st], V0=V0[st], final_state=True)
        ref = gsa.gsa_bwd(*s[:4], rz, s[4], K0=K0[st], V0=V0[st], initial_state_grad=True)
        got = [o[:, own], KT[st], VT[st]] + [x[:, own] for x in grads[:4]] + [x[st] for x in grads[4:]]
        for name, a, b in zip(("o", "KT", "VT", "dq", "dk", "dv", "dg", "dK0", "dV0"), got, [ro, rK, rV] + list(ref)):
            # two roundings of the same sums to bf16 (2^-9 each) where one side is walked in segments or takes the wide contractions
            # in a kernel of their own; fp32: sums in another order
            assert rel_l2(to_np64(a), to_np64(b)) <= (4e-3 if dtype == B16 else 1e-5), (name, i)
