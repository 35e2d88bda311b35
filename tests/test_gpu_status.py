"""The status word where the grid reports by itself and where a kernel in front of it does: both sides of the rule (2048
tokens; 64 planes of 128 values), a damaged entry at every edge of the check's four-entry loads and 1024-entry sweeps."""
import pytest
import torch

import paper_2605_03884_amd as qkv
import qkv_synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def make(L, H, T, D, G, seed):
    K, V = qkv_synth.make_kv(L, H, T, D, seed, "llama", device=DEV)
    bits, counts = qkv.assign_bits(qkv_synth.make_scores(T, seed + 1, DEV), 4.0)
    desc = qkv.Desc.make(L, H, T, D, G)
    card = torch.zeros(qkv.card_bytes(desc, counts), dtype=torch.uint8, device=DEV)
    qkv.quantize_pack(desc, K, V, bits, counts, card)
    return desc, card, counts


def read(desc, card, how):
    """(status, rows written per token) of one call into outputs that start as all-ones bit patterns."""
    status = torch.full((1,), 0x7777, dtype=torch.int32, device=DEV)
    k = torch.full((desc.layers, desc.kv_heads, desc.tokens, desc.head_dim), -1, dtype=torch.int16, device=DEV).view(torch.float16)
    v = k.clone()
    if how == "dense":
        qkv.unpack_dequant(card, desc, k, v, status=status)
    else:
        qkv.inject_layers(card, desc, [k[l] for l in range(desc.layers)], [v[l] for l in range(desc.layers)], status=status)
    torch.cuda.synchronize()
    untouched = (k.view(torch.int16) == -1).all(dim=3) & (v.view(torch.int16) == -1).all(dim=3)
    return int(status.item()), untouched


@pytest.mark.parametrize("L,H,T,D", [(1, 1, 1, 128), (1, 2, 5, 64), (1, 1, 1023, 128), (1, 1, 2048, 64), (1, 1, 2049, 64),
                                     (4, 7, 2053, 128), (4, 8, 2053, 128), (4, 4, 4100, 256), (8, 8, 1500, 64)])
def test_status_on_both_sides_of_the_rule(L, H, T, D):
    print("[case] L=%d H=%d T=%d D=%d" % (L, H, T, D), flush=True)
    desc, card, counts = make(L, H, T, D, 32, 100 + T)
    al = lambda x: (x + 255) // 256 * 256
    off_bits, off_slot = 256, 256 + al(T)
    off_order = off_slot + al(4 * T)
    for how in ("dense", "layers"):
        st, untouched = read(desc, card, how)
        assert st == 0 and not untouched.any()
        other = qkv.Desc.make(L, H, T, D, 64)
        st, untouched = read(other, card, how)
        assert st == qkv.STATUS_BAD_HEADER and untouched.all()
    order = card[off_order:off_order + 4 * T].view(torch.int32)
    for j in sorted({0, min(3, T - 1), min(1023, T - 1), min(1024, T - 1), min(2047, T - 1), T - 1}):
        t = int(order[j])
        for damage in ("order", "slot", "bits"):
            bad = card.clone()
            if damage == "order":
                bad[off_order + 4 * j:off_order + 4 * j + 4] = torch.tensor([255, 255, 255, 127], dtype=torch.uint8, device=DEV)
            elif damage == "slot":
                bad[off_slot + 4 * t] += 1
            else:
                bad[off_bits + t] = 3
            st, untouched = read(desc, bad, "dense" if j % 2 else "layers")
            assert st == qkv.STATUS_BAD_ORDER, (j, damage)
            assert untouched[:, :, t].all() and int(untouched.any(dim=1).any(dim=0).sum()) == 1, (j, damage)
