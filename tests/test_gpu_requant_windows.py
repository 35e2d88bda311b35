"""Requantization at the edges of its windows (256 rows of an outgoing segment) and of its rounds, and the relabelling of
2-bit groups against the chain through the dense cache for pairs that card creation would never write."""
import numpy as np
import pytest
import torch

import paper_2605_03884_amd as qkv
import qkv_synth
from oracle import ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def hop(card, rd, bits_new, label):
    """The call's card against the oracle's unpack + pack, byte for byte."""
    print("[case] " + label, flush=True)
    counts = ref.count_bits(bits_new).tolist()
    k, v = ref.unpack_dequant(card, rd)
    want = ref.quantize_pack(rd, k, v, bits_new, counts)
    desc = qkv.Desc.make(rd.layers, rd.kv_heads, rd.tokens, rd.head_dim, rd.group_size)
    out = torch.full((want.size,), 0xA5, dtype=torch.uint8, device=DEV)
    status = torch.full((1,), 0x7777, dtype=torch.int32, device=DEV)
    qkv.requantize(torch.from_numpy(card).to(DEV), desc, torch.from_numpy(bits_new).to(DEV), counts, out, status=status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    diff = np.flatnonzero(out.cpu().numpy() != want)
    assert diff.size == 0, (label, "differs at %d bytes, first %d" % (diff.size, int(diff[0])))


def draw_bits(T, rng, shares):
    return rng.choice(np.array([2, 4, 8, 16], np.uint8), size=T, p=shares)


@pytest.mark.parametrize("T,D,G", [(255, 128, 32), (256, 64, 32), (257, 256, 128), (513, 128, 64), (1, 64, 64), (700, 128, 128)])
def test_window_edges(T, D, G):
    rng = np.random.default_rng(T)
    K, V = qkv_synth.make_kv(1, 3, T, D, T, "llama")
    rd = ref.make_desc(1, 3, T, D, G)
    mixes = {"even": [0.25] * 4, "low": [0.9, 0.06, 0.03, 0.01], "high": [0.0, 0.1, 0.3, 0.6]}
    for na, a in mixes.items():
        bits = draw_bits(T, rng, a)
        card = ref.quantize_pack(rd, K.numpy().view(np.uint16), V.numpy().view(np.uint16), bits, ref.count_bits(bits).tolist())
        for nb, b in mixes.items():
            hop(card, rd, draw_bits(T, rng, b), "T=%d D=%d G=%d %s to %s" % (T, D, G, na, nb))


@pytest.mark.parametrize("T,D,G", [(250, 64, 64), (300, 64, 32), (1030, 64, 64), (1535, 128, 128), (3100, 64, 32), (3200, 64, 64)])
def test_windows_across_planes_and_inside_them(T, D, G):
    """128 planes: windows of 64, 128 and 256 rows that run across planes up to 393215 rows, then windows of a plane (3100 and
    3200 tokens: an even and an odd number of them)."""
    rng = np.random.default_rng(T)
    K, V = qkv_synth.make_kv(8, 8, T, D, T, "llama")
    rd = ref.make_desc(8, 8, T, D, G)
    a, b = draw_bits(T, rng, [0.4, 0.3, 0.2, 0.1]), draw_bits(T, rng, [0.62, 0.26, 0.08, 0.04])
    if T > 3000:
        assert sum((n + 255) // 256 for n in ref.count_bits(b).tolist()) % 2 == (T == 3200)
    card = ref.quantize_pack(rd, K.numpy().view(np.uint16), V.numpy().view(np.uint16), a, ref.count_bits(a).tolist())
    hop(card, rd, b, "128 planes, T=%d D=%d G=%d" % (T, D, G))


def chain_on_the_gpu(L, H, T, a, b, group_size=64):
    """Cards too large for the oracle: the call's card against injection and creation on the GPU, byte for byte."""
    ca, cb = ref.count_bits(a).tolist(), ref.count_bits(b).tolist()
    a, b = torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV)
    desc = qkv.Desc.make(L, H, T, 64, group_size)
    g = torch.Generator(device=DEV)
    g.manual_seed(T)
    k = torch.randn((L, H, T, 64), dtype=torch.float16, device=DEV, generator=g)
    v = torch.randn((L, H, T, 64), dtype=torch.float16, device=DEV, generator=g)
    card = torch.empty(qkv.card_bytes(desc, ca), dtype=torch.uint8, device=DEV)
    qkv.quantize_pack(desc, k, v, a, ca, card)
    qkv.unpack_dequant(card, desc, k, v)
    want = torch.empty(qkv.card_bytes(desc, cb), dtype=torch.uint8, device=DEV)
    qkv.quantize_pack(desc, k, v, b, cb, want)
    del k, v
    out = torch.full((want.numel(),), 0xA5, dtype=torch.uint8, device=DEV)
    status = torch.full((1,), 0x7777, dtype=torch.int32, device=DEV)
    qkv.requantize(card, desc, b, cb, out, status=status)
    assert int(status.item()) == 0
    assert torch.equal(out, want)


def test_two_planes_per_workgroup():
    """2176 planes in pairs that share their look-ups: at least 8192 workgroups, both cards below 512 MiB."""
    L, H, T = 64, 17, 1600
    print("[case] requant L=%d H=%d T=%d, two planes a workgroup" % (L, H, T), flush=True)
    rng = np.random.default_rng(1)
    a, b = draw_bits(T, rng, [0.4, 0.3, 0.2, 0.1]), draw_bits(T, rng, [0.5, 0.3, 0.15, 0.05])
    windows = sum((n + 255) // 256 for n in ref.count_bits(b).tolist())
    assert windows * L * H >= 8192 and 2 * L * H * T >= 1536 * 256
    assert max(qkv.card_bytes(qkv.Desc.make(L, H, T, 64, 64), ref.count_bits(x).tolist()) for x in (a, b)) <= 512 << 20
    chain_on_the_gpu(L, H, T, a, b)


def test_more_planes_than_a_grid_is_wide():
    """2^21 layers times heads of five tokens: a workgroup per plane and width would be a launch of more than 2^32 threads, and windows across
    planes are more workgroups than stand side by side."""
    print("[case] requant L=2048 H=1024 T=5", flush=True)
    chain_on_the_gpu(2048, 1024, 5, np.array([16, 2, 8, 4, 2], np.uint8), np.array([2, 8, 16, 2, 4], np.uint8))


@pytest.mark.parametrize("G", [32, 64, 128])
@pytest.mark.parametrize("kind", ["normal", "subnormal scale", "zero scale", "negative scale", "one code", "two codes", "mixed"])
def test_two_bit_groups_of_any_content(kind, G):
    """2-bit cards with drawn pairs and codes; every decoded value stays finite."""
    T, D, P = 96, 128, 2
    rng = np.random.default_rng(len(kind) + G)
    rd = ref.make_desc(1, 1, T, D, G)
    zero = np.zeros((1, 1, T, D), np.uint16)
    card = ref.quantize_pack(rd, zero, zero, np.full(T, 2, np.uint8), [T, 0, 0, 0])
    off = ref.card_offsets(rd, [T, 0, 0, 0])
    n_codes, n_pairs = P * T * D // 4, P * T * D // G
    codes = rng.integers(0, 256, n_codes).astype(np.uint8)
    scale = np.abs(rng.standard_normal(n_pairs) * 10.0 ** rng.integers(-3, 3, n_pairs)).astype(np.float16)
    low = (rng.integers(1, 1024, n_pairs) * 2.0 ** -24).astype(np.float16)
    zeros = (rng.standard_normal(n_pairs) * 10.0 ** rng.integers(-6, 4, n_pairs)).astype(np.float16)
    pick = rng.integers(0, 4, n_pairs)
    if kind == "subnormal scale":
        scale = low
        zeros = np.where(rng.random(n_pairs) < 0.5, zeros, (rng.integers(-3000, 3000, n_pairs) * 2.0 ** -24).astype(np.float16))
    if kind == "zero scale":
        scale[:] = 0
        zeros[::3] = np.float16(-0.0)
    if kind == "negative scale":
        scale[::2] = -scale[::2]
    if kind == "one code":
        codes = np.repeat(pick * 0x55, n_codes // n_pairs).astype(np.uint8)
    if kind == "two codes":
        codes = np.where(rng.random(n_codes) < 0.9, np.repeat(pick * 0x55, n_codes // n_pairs), rng.integers(0, 4, n_codes) * 0x55).astype(np.uint8)
    if kind == "mixed":
        scale = np.choose(pick, [scale, low, np.zeros_like(scale), -scale])
    card[off["codes2"]:off["codes2"] + n_codes] = codes
    card[off["meta2"]:off["meta2"] + 4 * n_pairs] = np.stack([scale, zeros], axis=1).reshape(-1).view(np.uint8)
    for width in (2, 4, 8, 16):
        hop(card, rd, np.full(T, width, np.uint8), "2-bit, %s, G=%d to %d bits" % (kind, G, width))


@pytest.mark.parametrize("G", [32, 64, 128])
@pytest.mark.parametrize("old", [4, 8])
def test_wider_groups_of_any_content(old, G):
    """4- and 8-bit cards with drawn pairs and codes; every decoded value stays finite."""
    T, D, P = 96, 128, 2
    rng = np.random.default_rng(old + G)
    rd = ref.make_desc(1, 1, T, D, G)
    zero = np.zeros((1, 1, T, D), np.uint16)
    counts = [T * (w == old) for w in (2, 4, 8, 16)]
    card = ref.quantize_pack(rd, zero, zero, np.full(T, old, np.uint8), counts)
    off = ref.card_offsets(rd, counts)
    n_codes, n_pairs = P * T * D * old // 8, P * T * D // G
    card[off["codes%d" % old]:off["codes%d" % old] + n_codes] = rng.integers(0, 256, n_codes).astype(np.uint8)
    scale, zeros = drawn_pairs(rng, n_pairs)
    card[off["meta%d" % old]:off["meta%d" % old] + 4 * n_pairs] = np.stack([scale, zeros], axis=1).reshape(-1).view(np.uint8)
    for width in (2, 4, 8, 16):
        hop(card, rd, np.full(T, width, np.uint8), "%d-bit, any pairs, G=%d to %d bits" % (old, G, width))


def drawn_pairs(rng, n):
    """Scales of every kind - ordinary, subnormal, zero, negative - and zeros of any size; 255 steps from any zero stay finite."""
    scale = np.abs(rng.standard_normal(n) * 10.0 ** rng.integers(-3, 2, n)).astype(np.float16)
    low = (rng.integers(1, 1024, n) * 2.0 ** -24).astype(np.float16)
    zeros = (rng.standard_normal(n) * 10.0 ** rng.integers(-6, 4, n)).astype(np.float16)
    return np.choose(rng.integers(0, 4, n), [scale, low, np.zeros_like(scale), -scale]), zeros


def planes_at_a_time(desc, total_in, counts_out):
    """How many planes a workgroup of the windows of tokens does with one look-up and sort; 0: the call goes through windows of a width."""
    total_out = qkv.card_bytes(desc, counts_out)
    rows = 2 * desc.layers * desc.kv_heads * desc.tokens
    values, both = rows * desc.head_dim, total_in + total_out
    if desc.head_dim < 128 or values < 131072000 or 2 * total_in > 3 * values or total_out > values or both > 2 * values:
        return 0
    if desc.head_dim > 128:
        return 2 if 16 * both <= 15 * values and rows >= 2 * 1024 * 512 else 1
    one_width = desc.tokens in counts_out
    return 2 if 16 * both <= 19 * values or (one_width and total_in <= total_out) or (16 * both <= 21 * values and both <= 256 << 20) else 1


MIXES = {"wide": [0.4, 0.3, 0.2, 0.1], "middle": [0.62, 0.26, 0.08, 0.04], "narrow": [0.85, 0.1, 0.04, 0.01], "of 2": [1, 0, 0, 0], "of 4": [0, 1, 0, 0]}


class LongCard:
    """A card long enough for the windows of tokens, made on the GPU, and what creation makes of it after injection."""

    def __init__(self, L, H, T, D, G, old, new, order="drawn", planes=None):
        print("[case] windows of tokens L=%d H=%d T=%d D=%d G=%d %s to %s %s" % (L, H, T, D, G, old, new, order), flush=True)
        self.shape, rng = (L, H, T, D, G), np.random.default_rng(T)
        a, b = draw_bits(T, rng, MIXES[old]), draw_bits(T, rng, MIXES[new])
        if order == "sorted":
            a = np.sort(a)
        self.ca, self.cb = ref.count_bits(a).tolist(), ref.count_bits(b).tolist()
        self.desc = qkv.Desc.make(L, H, T, D, G)
        self.off = ref.card_offsets(ref.make_desc(L, H, T, D, G), self.ca)
        self.a, self.b = torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV)
        g = torch.Generator(device=DEV)
        g.manual_seed(T)
        self.k = torch.randn((L, H, T, D), dtype=torch.float16, device=DEV, generator=g)
        self.v = torch.randn((L, H, T, D), dtype=torch.float16, device=DEV, generator=g)
        self.card = torch.empty(qkv.card_bytes(self.desc, self.ca), dtype=torch.uint8, device=DEV)
        taken = planes_at_a_time(self.desc, self.card.numel(), self.cb)
        assert taken == planes if planes else taken > 0
        qkv.quantize_pack(self.desc, self.k, self.v, self.a, self.ca, self.card)
        qkv.unpack_dequant(self.card, self.desc, self.k, self.v)
        self.status = torch.full((1,), 0x7777, dtype=torch.int32, device=DEV)

    def requantize(self, counts):
        out = torch.full((qkv.card_bytes(self.desc, counts),), 0xA5, dtype=torch.uint8, device=DEV)
        qkv.requantize(self.card, self.desc, self.b, counts, out, status=self.status)
        return out

    def compare(self, counts, want_status):
        want = torch.full((qkv.card_bytes(self.desc, counts),), 0xA5, dtype=torch.uint8, device=DEV)
        qkv.quantize_pack(self.desc, self.k, self.v, self.b, counts, want)
        out = self.requantize(counts)
        assert int(self.status.item()) == want_status
        assert torch.equal(out, want)


@pytest.mark.parametrize("L,H,T,D,G,old,new,order,planes", [
    (32, 8, 2001, 128, 32, "wide", "middle", "drawn", 1), (32, 8, 2048, 128, 64, "wide", "middle", "sorted", 2),
    (16, 8, 2049, 256, 128, "wide", "middle", "drawn", 1), (16, 8, 2100, 256, 32, "wide", "middle", "sorted", 1),
    (1, 1, 512003, 128, 128, "wide", "middle", "drawn", 2), (1024, 5, 101, 128, 32, "wide", "middle", "drawn", 1),
    (64, 1, 8191, 128, 32, "of 4", "middle", "drawn", 2), (32, 8, 7001, 128, 32, "wide", "middle", "drawn", 1),
    (32, 8, 8191, 128, 32, "middle", "narrow", "drawn", 2), (32, 8, 8193, 128, 32, "of 4", "of 4", "drawn", 2),
    (16, 8, 4101, 256, 128, "middle", "narrow", "sorted", 2), (4, 2, 65537, 128, 64, "of 2", "wide", "drawn", 2)])
def test_windows_of_tokens(L, H, T, D, G, old, new, order, planes):
    """At least 131072000 values of 128 or 256 dimensions in narrow rows: windows of 512 rows inside a plane, across the ends of planes and over
    many short ones, one and two planes at a time, below and above 512 MiB, against injection and creation on the GPU; with an entry
    of the incoming tables out of range, or a width that is none, the token's rows are those of zeros, and with counts that are not those of
    the widths the card is what creation makes of the same counts."""
    c = LongCard(L, H, T, D, G, old, new, order, planes)
    c.compare(c.cb, 0)
    wrong = list(c.cb)
    at = 0 if wrong[0] >= 3 else 1
    wrong[at], wrong[at + 1] = wrong[at] - 3, wrong[at + 1] + 3
    c.compare(wrong, 0)
    slots = c.card[c.off["slot"]:c.off["slot"] + 4 * T].view(torch.int32)
    for lost, spoil in ((T // 2, lambda t: slots[t:t + 1].fill_(1 << 30)), (T // 3, lambda t: c.card[c.off["bits"] + t:c.off["bits"] + t + 1].fill_(7))):
        spoil(lost)
        c.k[:, :, lost], c.v[:, :, lost] = 0, 0
        c.compare(c.cb, qkv.STATUS_BAD_ORDER)


@pytest.mark.parametrize("G,new", [(32, "wide"), (64, "middle"), (128, "of 4"), (32, "of 2")])
def test_windows_of_tokens_any_pairs(G, new):
    """Pairs that creation would never write, ordinary ones among them, at every width: 2-bit rows that can't be relabelled, and the wider decoders."""
    c = LongCard(32, 8, 2003, 128, G, "wide", new)
    rng = np.random.default_rng(G)
    for i, width in enumerate((2, 4, 8)):
        n = 2 * 32 * 8 * c.ca[i] * (128 // G)
        scale, zeros = drawn_pairs(rng, n)
        at = c.off["meta%d" % width]
        mine = torch.from_numpy(np.stack([scale, zeros], axis=1).reshape(-1).view(np.int32)).to(DEV)
        pairs = c.card[at:at + 4 * n].view(torch.int32)
        pairs.copy_(torch.where(torch.arange(n, device=DEV) % 5 == 0, pairs, mine))
    qkv.unpack_dequant(c.card, c.desc, c.k, c.v)
    assert torch.isfinite(c.k).all() and torch.isfinite(c.v).all()
    c.compare(c.cb, 0)


def test_windows_of_tokens_refused_card():
    """A header that is none, and a card with keys per channel: nothing is written but the front matter."""
    c = LongCard(32, 8, 2001, 128, 32, "wide", "middle")
    out = ref.card_offsets(ref.make_desc(*c.shape), c.cb)
    per_plane = [c.cb[0] * 32, c.cb[0] * 16, c.cb[1] * 64, c.cb[1] * 16, c.cb[2] * 128, c.cb[2] * 16, c.cb[3] * 256]
    for byte, value in ((3, 0), (188, qkv.FLAG_KEYS_PER_CHANNEL)):
        was = int(c.card[byte].item())
        c.card[byte] = value
        got = c.requantize(c.cb)
        assert int(c.status.item()) == qkv.STATUS_BAD_HEADER
        for name, n in zip(("codes2", "meta2", "codes4", "meta4", "codes8", "meta8", "fp16"), per_plane):
            assert (got[out[name]:out[name] + 512 * n] == 0xA5).all(), name
        c.card[byte] = was
    c.compare(c.cb, 0)
