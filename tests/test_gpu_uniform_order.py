"""Cards whose tiles look their row addresses up before or after they load: uniform ones injected into more and into fewer layers than
the line between them, raw rows beyond 512 MiB, of any share of the tokens, keys per channel beyond 512 MiB of cache.  Unpacking at small
sizes is compared with the oracle elsewhere; here the calls must agree with it, or with the raw rows themselves."""
import numpy as np
import pytest
import torch

import paper_2605_03884_amd as qkv
import qkv_synth
from oracle import ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def make(L, H, T, D, width, kc=False):
    g = torch.Generator(device=DEV)
    g.manual_seed(T + width)
    k = torch.randn((L, H, T, D), dtype=torch.float16, device=DEV, generator=g)
    v = torch.randn((L, H, T, D), dtype=torch.float16, device=DEV, generator=g)
    bits = torch.full((T,), width, dtype=torch.uint8, device=DEV)
    counts = [T * (width == w) for w in (2, 4, 8, 16)]
    desc = qkv.Desc.make(L, H, T, D, 32)
    card = torch.empty(qkv.card_bytes(desc, counts), dtype=torch.uint8, device=DEV)
    (qkv.quantize_pack_kc if kc else qkv.quantize_pack)(desc, k, v, bits, counts, card)
    return desc, card, k, v


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("width,kc", [(2, False), (4, False), (8, False), (16, False), (2, True), (4, True), (8, True)])
def test_injection_agrees_with_unpacking(D, width, kc):
    L, H, T, P = 7, 2, 448, 5
    print("[case] inject D=%d width %d %s" % (D, width, "keys per channel" if kc else ""), flush=True)
    desc, card, k, v = make(L, H, T, D, width, kc)
    status = torch.ones(1, dtype=torch.int32, device=DEV)
    (qkv.unpack_dequant_kc if kc else qkv.unpack_dequant)(card, desc, k, v, status=status)
    for rope in (0, 64):
        base = 10000.0 if rope else 0.0
        one, some = [[torch.full((L, H, T + P, D), 7.0, dtype=torch.float16, device=DEV) for _ in range(2)] for _ in range(2)]
        qkv.inject_layers(card, desc, [x[:, P:] for x in one[0]], [x[:, P:] for x in one[1]], rope_base=base, rope_delta=rope,
                          status=status, keys_per_channel=kc)
        for begin in (0, 3, 6):
            end = min(begin + 3, L)
            qkv.inject_layers(card, desc, [x[:, P:] for x in some[0][begin:end]], [x[:, P:] for x in some[1][begin:end]], begin,
                              rope_base=base, rope_delta=rope, status=status, keys_per_channel=kc)
        assert int(status.item()) == 0
        assert torch.equal(one[1][:, :, P:], v)
        if rope == 0:
            assert torch.equal(one[0][:, :, P:], k)
        for a, b in zip(one, some):
            assert torch.equal(a, b) and (a[:, :, :P] == 7.0).all()


def test_raw_rows_of_a_large_card():
    L, H, T, D = 32, 8, 4224, 128
    print("[case] 16-bit card beyond 512 MiB", flush=True)
    desc, card, k, v = make(L, H, T, D, 16)
    assert card.numel() > 512 << 20
    k2, v2 = torch.empty_like(k), torch.empty_like(v)
    status = torch.ones(1, dtype=torch.int32, device=DEV)
    qkv.unpack_dequant(card, desc, k2, v2, status=status)
    assert int(status.item()) == 0 and torch.equal(k, k2) and torch.equal(v, v2)
    k2.zero_(), v2.zero_()
    qkv.inject_layers(card, desc, list(k2), list(v2), status=status)
    assert int(status.item()) == 0 and torch.equal(k, k2) and torch.equal(v, v2)


@pytest.mark.parametrize("raw", [0, 1, 32, 33, 34, 132, 133])
@pytest.mark.parametrize("D,G", [(64, 32), (128, 64), (256, 128)])
def test_streamed_cards_of_mixed_widths(D, G, raw):
    """A buffer beyond 512 MiB makes the card in it one that is streamed.  Raw tokens below, at and above a quarter, where their loads go out in halves."""
    L, H, T = 6, 2, 133
    print("[case] streamed D=%d, %d raw tokens of %d" % (D, raw, T), flush=True)
    rng = np.random.default_rng(D + raw)
    bits = np.concatenate([np.full(raw, 16, np.uint8), rng.choice(np.array([2, 4, 8], np.uint8), T - raw)])
    rng.shuffle(bits)
    K, V = qkv_synth.make_kv(L, H, T, D, 7 + raw, "llama")
    rd = ref.make_desc(L, H, T, D, G)
    card = ref.quantize_pack(rd, K.numpy().view(np.uint16), V.numpy().view(np.uint16), bits, ref.count_bits(bits).tolist())
    want = [torch.from_numpy(x.reshape(L, H, T, D).view(np.int16)).to(DEV) for x in ref.unpack_dequant(card, rd)]
    buffer = torch.empty((512 << 20) + 4096, dtype=torch.uint8, device=DEV)
    buffer[:card.size] = torch.from_numpy(card).to(DEV)
    desc = qkv.Desc.make(L, H, T, D, G)
    status = torch.ones(1, dtype=torch.int32, device=DEV)
    k, v = [torch.full((L, H, T, D), 7.0, dtype=torch.float16, device=DEV) for _ in range(2)]
    qkv.unpack_dequant(buffer, desc, k, v, status=status)
    assert int(status.item()) == 0
    assert torch.equal(k.view(torch.int16), want[0]) and torch.equal(v.view(torch.int16), want[1])
    for many in (L, 3):
        k.fill_(7.0), v.fill_(7.0)
        for begin in range(0, L, many):
            qkv.inject_layers(buffer, desc, list(k[begin:begin + many]), list(v[begin:begin + many]), begin, status=status)
        assert int(status.item()) == 0
        assert torch.equal(k.view(torch.int16), want[0]) and torch.equal(v.view(torch.int16), want[1])


@pytest.mark.parametrize("width", [2, 4, 8])
def test_keys_per_channel_on_both_sides_of_512_mib(width):
    """The same planes in one large card and in two of half its layers."""
    L, H, T, D = 32, 8, 4096, 128
    print("[case] keys per channel, width %d" % width, flush=True)
    desc, card, k, v = make(L, H, T, D, width, True)
    k2, v2 = torch.empty_like(k), torch.empty_like(v)
    qkv.unpack_dequant_kc(card, desc, k2, v2)
    half = qkv.Desc.make(L // 2, H, T, D, 32)
    bits = torch.full((T,), width, dtype=torch.uint8, device=DEV)
    counts = [T * (width == w) for w in (2, 4, 8, 16)]
    card = torch.empty(qkv.card_bytes(half, counts), dtype=torch.uint8, device=DEV)
    for part in (slice(0, L // 2), slice(L // 2, L)):
        ks, vs = torch.empty_like(k[part]), torch.empty_like(v[part])
        qkv.quantize_pack_kc(half, k[part], v[part], bits, counts, card)
        qkv.unpack_dequant_kc(card, half, ks, vs)
        assert torch.equal(ks, k2[part]) and torch.equal(vs, v2[part])
