"""Waves that take several tasks of a pair one after the other and leave one partial (more tasks than the chip's 4096 wave slots
have room for at a time): few turns of even tasks, many turns of the longest ones, a pair count that needs several turns
of the slots themselves, every layout of the heads, and a value that is no number in a later task."""
import pytest
import torch

import paper_2605_03884_amd as qkv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dense_attention(q, k, v, H, rep, D):
    """float64 on the dequantized values of one layer"""
    s = (q.double().view(H, rep, D) @ k.double().transpose(1, 2).contiguous()) * D ** -0.5
    return torch.softmax(s, dim=-1) @ v.double(), torch.logsumexp(s, dim=-1)


@pytest.mark.parametrize("L,H,T,D,rep", [(35, 8, 4200, 128, 4), (35, 8, 6100, 64, 3), (40, 8, 9000, 64, 4), (35, 8, 3001, 128, 6), (35, 8, 1700, 128, 13),
                                         (35, 8, 2100, 64, 16), (30, 8, 2300, 256, 2), (30, 8, 1300, 256, 9), (625, 8, 700, 64, 2), (560, 8, 500, 128, 5)])
@pytest.mark.parametrize("budget", [2.4, 6.0])
def test_several_tasks_a_wave(L, H, T, D, rep, budget):
    print("[case] L=%d H=%d T=%d D=%d rep=%d budget %g" % (L, H, T, D, rep, budget), flush=True)
    desc = qkv.Desc.make(L, H, T, D, 64)
    gen = torch.Generator(device=DEV).manual_seed(T + rep)
    bits, counts = qkv.assign_bits(torch.rand((T,), device=DEV, generator=gen), budget)
    k, v = (torch.randn((L, H, T, D), dtype=torch.float16, device=DEV, generator=gen) for _ in range(2))
    raw = int((bits == 16).nonzero()[-1])                 # the last raw row: infinite in one dimension of one pair
    v[L - 1, H - 1, raw, D // 2 + 1] = float("inf")
    card = torch.empty(qkv.card_bytes(desc, counts), dtype=torch.uint8, device=DEV)
    qkv.quantize_pack(desc, k, v, bits, counts, card)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    qkv.unpack_dequant(card, desc, k, v, status=status)
    q = torch.randn((L, H * rep, D), dtype=torch.float16, device=DEV, generator=gen)
    size = qkv.card_attend_workspace(desc, H * rep)
    ws = torch.full((size + 256,), 0x7F, dtype=torch.uint8, device=DEV)
    out, lse = torch.full((L, H * rep, D), float("nan"), device=DEV), torch.full((L, H * rep), float("nan"), device=DEV)
    qkv.card_attend(card, desc, q, D ** -0.5, out, lse=lse, status=status, workspace=ws[:size])
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and (ws[size:] == 0x7F).all()
    at = out[L - 1].view(H, rep, D)[H - 1, :, D // 2 + 1]
    assert not torch.isfinite(at).any()
    at.zero_()
    v[L - 1, H - 1, :, D // 2 + 1] = 0
    for l in sorted({0, 1, L // 2, L - 1}):
        want, want_lse = dense_attention(q[l], k[l], v[l], H, rep, D)
        # a score is off by at most D 2^-24 scale sum |q k|, and out by twice that times max |v| (and its own fp32 sums)
        e = D * 2.0 ** -24 * D ** -0.5 * float((q[l].double().abs().view(H, rep, D) @ k[l].double().abs().transpose(1, 2).contiguous()).max())
        assert float((out[l].view(H, rep, D).double() - want).abs().max()) <= (2 * e + 1e-5) * float(v[l].abs().max())
        assert float((lse[l].view(H, rep).double() - want_lse).abs().max()) <= e + 1e-5


@pytest.mark.parametrize("L,H,T,D,rep", [(35, 8, 6100, 64, 3), (40, 8, 9000, 64, 8), (35, 8, 2100, 64, 16), (35, 8, 4200, 128, 4)])
def test_an_infinite_key_in_a_later_task(L, H, T, D, rep):
    """Scores of -inf in rows of every raw task of one pair: a weight of zero, and nothing else of the wave's tasks is lost."""
    print("[case] L=%d H=%d T=%d D=%d rep=%d" % (L, H, T, D, rep), flush=True)
    desc = qkv.Desc.make(L, H, T, D, 64)
    gen = torch.Generator(device=DEV).manual_seed(T + rep)
    bits, counts = qkv.assign_bits(torch.rand((T,), device=DEV, generator=gen), 7.0)
    k, v = (torch.randn((L, H, T, D), dtype=torch.float16, device=DEV, generator=gen) for _ in range(2))
    q = torch.randn((L, H * rep, D), dtype=torch.float16, device=DEV, generator=gen)
    raw = (bits == 16).nonzero().flatten()[7::50]
    k[L - 1, H - 1, raw, 3] = float("inf")
    q[L - 1, (H - 1) * rep:, 3] = -q[L - 1, (H - 1) * rep:, 3].abs() - 0.01
    card = torch.empty(qkv.card_bytes(desc, counts), dtype=torch.uint8, device=DEV)
    qkv.quantize_pack(desc, k, v, bits, counts, card)
    qkv.unpack_dequant(card, desc, k, v)
    out, lse = torch.full((L, H * rep, D), float("nan"), device=DEV), torch.full((L, H * rep), float("nan"), device=DEV)
    qkv.card_attend(card, desc, q, D ** -0.5, out, lse=lse)
    torch.cuda.synchronize()
    keep = torch.ones(T, dtype=torch.bool, device=DEV)
    keep[raw] = False                                     # tokens whose weight is zero, in that pair only
    for l, h, rows in ((0, 0, keep | True), (L - 1, H - 2, keep | True), (L - 1, H - 1, keep)):
        kk, vv, qq = k[l, h:h + 1, rows], v[l, h:h + 1, rows], q[l, h * rep:(h + 1) * rep]
        want, want_lse = dense_attention(qq, kk, vv, 1, rep, D)
        e = D * 2.0 ** -24 * D ** -0.5 * float((qq.double().abs() @ kk[0].double().abs().T.contiguous()).max())
        assert float((out[l, h * rep:(h + 1) * rep].double() - want[0]).abs().max()) <= (2 * e + 1e-5) * float(vv.abs().max())
        assert float((lse[l, h * rep:(h + 1) * rep].double() - want_lse[0]).abs().max()) <= e + 1e-5
