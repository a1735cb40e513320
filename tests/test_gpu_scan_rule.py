"""Packed batches on both sides of the rule that decides, on the device, whether the scans walk their sequences whole or in segments:
every sequence against a call of its own."""
import pytest
import torch

from tests.util import rel_l2, to_np64

pytestmark = pytest.mark.gpu

C = 64   # tokens per chunk (bf16)
# lengths, heads, d_k, d_v; True: walked whole.  More than 72 chunks in the longest sequence are walked whole only where
# chunks * heads * (d_k + d_v)/64 is at least 110 times as many.
CASES = [
    ((72 * C,), 2, 64, 64, True),                        # the longest of the first side, as the host sees it
    ((72 * C, 63 * C + 1), 2, 64, 64, True),             # the host provides for 136 chunks in one sequence; here the device decides
    ((72 * C + 1, 63 * C), 2, 64, 64, False),            # one token more
    ((1, 0, 72 * C, 100 * C + 3, 5), 1, 64, 128, False),  # three segments and a last one of five chunks; an empty and two tiny sequences
    ((0, 75 * C - 7, 75 * C, 70 * C) + (60 * C,) * 4, 4, 256, 256, True),   # 459 chunks * 32 workgroups = 133 * 110
]


@pytest.mark.parametrize("lens,H,d_k,d_v,whole", CASES)
def test_packed_against_single_sequences(lens, H, d_k, d_v, whole):
    import paper_2409_07146_amd as gsa
    m, T, dev = 16, sum(lens), torch.device("cuda")
    longest = max(-(-n // C) for n in lens)
    steps = sum(-(-n // C) for n in lens) * H * (d_k + d_v) // 64
    assert whole == (longest <= max(72, steps // 110))
    gen = torch.Generator(device=dev).manual_seed(5)
    t = lambda *s: torch.randn(*s, generator=gen, device=dev)
    q, k, v, dO = (t(1, T, H, d).mul_(d_k ** -0.5).bfloat16() for d in (d_k, d_k, d_v, d_v))
    g = torch.nn.functional.logsigmoid(t(1, T, H, m)) / 8
    K0, V0 = t(len(lens), H, m, d_k) * 0.1, t(len(lens), H, m, d_v) * 0.1
    ends = [0]
    for n in lens:
        ends.append(ends[-1] + n)
    cu = torch.tensor(ends, dtype=torch.int32, device=dev)
    o, z, KT, VT = gsa.gsa_fwd(q, k, v, g, K0=K0, V0=V0, cu_seqlens=cu, final_state=True)
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
            # in a kernel of their own
            assert rel_l2(to_np64(a), to_np64(b)) <= 4e-3, (name, i)
