"""How attention over a short card cuts its tasks: every class alone and mixed, token counts at the edges of the units (64, 48,
32 and 16 tokens by width), with the workspace the library asks for and with the least it accepts, and the merge over
more tasks than its threads hold at a time.  Tolerances: the bounds of test_gpu_attend.py."""
import numpy as np
import pytest
import torch

import paper_2605_03884_amd as qkv
from oracle import attend_ref
from test_gpu_attend import bounds, build_card

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def least_workspace(L, H, T, rep, D):
    """Bytes for tasks of as many tokens as the scores' LDS holds (192 where those would leave wave slots empty)."""
    room = 1536 // ((rep + 3) // 4 * 4)
    c = room // 192 * 192 if room >= 192 else 64
    while c > 192 and L * H * ((T + c - 1) // c + 2) < 4096:
        c -= 192
    return (L * H * ((T + c - 1) // c + 3) * rep * (D + 2) + 4) * 4


@pytest.mark.parametrize("T", [1, 16, 17, 48, 65, 193, 500, 1537])
@pytest.mark.parametrize("mix", ["even", "low", "2", "4", "8", "16"])
def test_short_cards(T, mix):
    L, H, rep, D, G = 1, 2, 4, 128, 32
    print("[case] T=%d widths %s" % (T, mix), flush=True)
    rng = np.random.default_rng(T)
    if mix in ("even", "low"):
        bits = rng.choice(np.array([2, 4, 8, 16], np.uint8), size=T, p=[0.25] * 4 if mix == "even" else [0.8, 0.1, 0.08, 0.02])
    else:
        bits = np.full(T, int(mix), np.uint8)
    rd, card = build_card(L, H, T, D, G, bits, T)
    q = rng.standard_normal((L, H * rep, D)).astype(np.float16)
    want_o, want_lse = attend_ref.card_attend(card, rd, q, D ** -0.5)
    tol_o, tol_lse = bounds(card, rd, q, D ** -0.5)
    desc = qkv.Desc.make(L, H, T, D, G)
    card_dev, q_dev = torch.from_numpy(card).to(DEV), torch.from_numpy(q).to(DEV)
    best, least = qkv.card_attend_workspace(desc, H * rep), least_workspace(L, H, T, rep, D)
    assert best >= least
    for size in (best, least, (best + least) // 2):
        ws = torch.full((size + 256,), 0x7F, dtype=torch.uint8, device=DEV)
        out = torch.full((L, H * rep, D), float("nan"), device=DEV)
        lse = torch.full((L, H * rep), float("nan"), device=DEV)
        qkv.card_attend(card_dev, desc, q_dev, D ** -0.5, out, lse=lse, workspace=ws[:size])
        torch.cuda.synchronize()
        assert float(np.abs(out.cpu().numpy() - want_o).max()) <= tol_o
        assert float(np.abs(lse.cpu().numpy() - want_lse).max()) <= tol_lse
        assert (ws[size:] == 0x7F).all()
    with pytest.raises(qkv.QkvError):
        qkv.card_attend(card_dev, desc, q_dev, D ** -0.5, out, lse=lse, workspace=ws[:least - 4])


@pytest.mark.parametrize("L,H,T,D,rep", [(32, 8, 300, 128, 4), (32, 8, 1000, 64, 2), (1, 8, 2000, 128, 4)])
def test_results_depend_on_the_workspace_size_only_below_the_queried_one(L, H, T, D, rep):
    """A finer cut than the least: the queried workspace, a larger one and the library's own scratch give the same bits, the
    smallest workspace accepted gives them to the bound."""
    print("[case] L=%d H=%d T=%d D=%d rep=%d" % (L, H, T, D, rep), flush=True)
    rng = np.random.default_rng(T)
    bits = rng.choice(np.array([2, 4, 8, 16], np.uint8), size=T, p=[0.5, 0.3, 0.15, 0.05])
    rd, card = build_card(L, H, T, D, 32, bits, T)
    q = rng.standard_normal((L, H * rep, D)).astype(np.float16)
    want_o, want_lse = attend_ref.card_attend(card, rd, q, D ** -0.5)
    tol_o, tol_lse = bounds(card, rd, q, D ** -0.5)
    desc = qkv.Desc.make(L, H, T, D, 32)
    card_dev, q_dev = torch.from_numpy(card).to(DEV), torch.from_numpy(q).to(DEV)
    best, least = qkv.card_attend_workspace(desc, H * rep), least_workspace(L, H, T, rep, D)
    assert best > least
    results = []
    for size in (best, best + 4096, least, None):
        out = torch.full((L, H * rep, D), float("nan"), device=DEV)
        lse = torch.full((L, H * rep), float("nan"), device=DEV)
        if size is None:
            qkv.card_attend_static(card_dev, desc, q_dev, D ** -0.5, out, lse=lse)
        else:
            qkv.card_attend(card_dev, desc, q_dev, D ** -0.5, out, lse=lse, workspace=torch.empty(size, dtype=torch.uint8, device=DEV))
        torch.cuda.synchronize()
        assert float(np.abs(out.cpu().numpy() - want_o).max()) <= tol_o
        assert float(np.abs(lse.cpu().numpy() - want_lse).max()) <= tol_lse
        results.append((out, lse))
    for out, lse in (results[1], results[3]):
        assert torch.equal(out, results[0][0]) and torch.equal(lse, results[0][1])


@pytest.mark.parametrize("D,rep,T", [(64, 1, 49000), (128, 3, 49000), (256, 16, 17000), (128, 16, 20000)])
def test_merge_over_many_tasks(D, rep, T):
    assert (qkv.card_attend_workspace(qkv.Desc.make(1, 1, T, D, 32), rep) // 4 - 4) // (rep * (D + 2)) > 256
    print("[case] D=%d rep=%d T=%d" % (D, rep, T), flush=True)
    rng = np.random.default_rng(D + rep)
    bits = rng.choice(np.array([2, 4, 8, 16], np.uint8), size=T, p=[0.5, 0.3, 0.15, 0.05])
    rd, card = build_card(1, 1, T, D, 32, bits, T)
    q = rng.standard_normal((1, rep, D)).astype(np.float16)
    want_o, want_lse = attend_ref.card_attend(card, rd, q, D ** -0.5)
    tol_o, tol_lse = bounds(card, rd, q, D ** -0.5)
    out = torch.empty((1, rep, D), device=DEV)
    lse = torch.empty((1, rep), device=DEV)
    qkv.card_attend(torch.from_numpy(card).to(DEV), qkv.Desc.make(1, 1, T, D, 32), torch.from_numpy(q).to(DEV), D ** -0.5, out, lse=lse)
    torch.cuda.synchronize()
    assert float(np.abs(out.cpu().numpy() - want_o).max()) <= tol_o
    assert float(np.abs(lse.cpu().numpy() - want_lse).max()) <= tol_lse


@pytest.mark.parametrize("T,rep", [(512, 4), (513, 4), (512, 16), (513, 16), (1023, 16), (1025, 16)])
@pytest.mark.parametrize("mix", ["16", "low"])
def test_around_the_limit_of_the_even_cut(T, rep, mix):
    """256 pairs: full tasks that fit the wave slots (1024 tokens at 16 heads), where even ones may not be more than the slots."""
    L, H, D = 32, 8, 64
    print("[case] T=%d rep=%d widths %s" % (T, rep, mix), flush=True)
    rng = np.random.default_rng(T + rep)
    bits = np.full(T, 16, np.uint8) if mix == "16" else rng.choice(np.array([2, 4, 8, 16], np.uint8), size=T, p=[0.2, 0.1, 0.1, 0.6])
    rd, card = build_card(L, H, T, D, 64, bits, T)
    q = rng.standard_normal((L, H * rep, D)).astype(np.float16)
    want_o, want_lse = attend_ref.card_attend(card, rd, q, D ** -0.5)
    tol_o, tol_lse = bounds(card, rd, q, D ** -0.5)
    out = torch.empty((L, H * rep, D), device=DEV)
    lse = torch.empty((L, H * rep), device=DEV)
    qkv.card_attend(torch.from_numpy(card).to(DEV), qkv.Desc.make(L, H, T, D, 64), torch.from_numpy(q).to(DEV), D ** -0.5, out, lse=lse)
    torch.cuda.synchronize()
    assert float(np.abs(out.cpu().numpy() - want_o).max()) <= tol_o
    assert float(np.abs(lse.cpu().numpy() - want_lse).max()) <= tol_lse


@pytest.mark.parametrize("L,H,T,D,rep,tasks", [(8, 16, 300, 64, 16, 8), (8, 16, 300, 256, 16, 8), (17, 8, 300, 128, 9, 8), (5, 26, 8300, 64, 16, 133),
                                               (30, 16, 130, 64, 5, 4), (16, 16, 70, 128, 16, 5), (16, 16, 60, 256, 16, 4)])
def test_merge_with_fewer_threads(L, H, T, D, rep, tasks):
    """More than 1024 and 2048 workgroups of the merge: 128 threads (also with more tasks than that), and 64 where a task's rows are few."""
    print("[case] L=%d H=%d T=%d D=%d rep=%d" % (L, H, T, D, rep), flush=True)
    assert L * H * rep > 1024
    desc = qkv.Desc.make(L, H, T, D, 64)
    assert (qkv.card_attend_workspace(desc, H * rep) // 4 - 4) // (L * H * rep * (D + 2)) == tasks
    rng = np.random.default_rng(D + rep)
    bits = rng.choice(np.array([2, 4, 8, 16], np.uint8), size=T, p=[0.5, 0.3, 0.15, 0.05])
    rd, card = build_card(L, H, T, D, 64, bits, T)
    q = rng.standard_normal((L, H * rep, D)).astype(np.float16)
    want_o, want_lse = attend_ref.card_attend(card, rd, q, D ** -0.5)
    tol_o, tol_lse = bounds(card, rd, q, D ** -0.5)
    out = torch.empty((L, H * rep, D), device=DEV)
    lse = torch.empty((L, H * rep), device=DEV)
    qkv.card_attend(torch.from_numpy(card).to(DEV), desc, torch.from_numpy(q).to(DEV), D ** -0.5, out, lse=lse)
    torch.cuda.synchronize()
    assert float(np.abs(out.cpu().numpy() - want_o).max()) <= tol_o
    assert float(np.abs(lse.cpu().numpy() - want_lse).max()) <= tol_lse


@pytest.mark.parametrize("L,H,T,D,rep,tasks", [(5, 26, 3328, 64, 16, 55), (5, 26, 3392, 64, 16, 56), (5, 26, 8350, 64, 16, 134),
                                               (5, 26, 2496, 256, 16, 42), (5, 26, 2560, 256, 16, 43)])
@pytest.mark.parametrize("mix", ["low", "4"])
def test_order_of_waves(L, H, T, D, rep, tasks, mix):
    """Pairs first up to 1.75 waves per slot of 4096 (1.33 at head_dim 256), tasks first beyond, an idle wave a pair where the tasks
    are even: every (layer, kv head) has its own query, so a wave at another place shows."""
    print("[case] L=%d H=%d T=%d D=%d rep=%d widths %s" % (L, H, T, D, rep, mix), flush=True)
    desc = qkv.Desc.make(L, H, T, D, 64)
    size = qkv.card_attend_workspace(desc, H * rep)
    assert (size // 4 - 4) // (L * H * rep * (D + 2)) == tasks
    bits, counts = torch.full((T,), 4, dtype=torch.uint8, device=DEV), [0, T, 0, 0]
    if mix == "low":
        bits, counts = qkv.assign_bits(torch.rand((T,), device=DEV), 3.0)
    gen = torch.Generator(device=DEV).manual_seed(T)
    k, v = (torch.randn((L, H, T, D), dtype=torch.float16, device=DEV, generator=gen) for _ in range(2))
    card = torch.empty(qkv.card_bytes(desc, counts), dtype=torch.uint8, device=DEV)
    qkv.quantize_pack(desc, k, v, bits, counts, card)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    qkv.unpack_dequant(card, desc, k, v, status=status)
    q = torch.randn((L, H * rep, D), dtype=torch.float16, device=DEV, generator=gen)
    ws = torch.full((size + 256,), 0x7F, dtype=torch.uint8, device=DEV)
    out, lse = torch.full((L, H * rep, D), float("nan"), device=DEV), torch.full((L, H * rep), float("nan"), device=DEV)
    qkv.card_attend(card, desc, q, D ** -0.5, out, lse=lse, workspace=ws[:size])
    torch.cuda.synchronize()
    assert (ws[size:] == 0x7F).all()
    for l in range(L):                           # float64 on the dequantized values, a layer at a time
        s = (q[l].double().view(H, rep, D) @ k[l].double().transpose(1, 2).contiguous()) * D ** -0.5
        want_lse = torch.logsumexp(s, dim=-1)
        want = torch.softmax(s, dim=-1) @ v[l].double()
        # a score is off by at most D 2^-24 scale sum |q k|, and out by twice that times max |v| (and its own fp32 sums)
        e = D * 2.0 ** -24 * D ** -0.5 * float((q[l].double().abs().view(H, rep, D) @ k[l].double().abs().transpose(1, 2).contiguous()).max())
        assert float((out[l].view(H, rep, D).double() - want).abs().max()) <= (2 * e + 1e-5) * float(v[l].abs().max())
        assert float((lse[l].view(H, rep).double() - want_lse).abs().max()) <= e + 1e-5
