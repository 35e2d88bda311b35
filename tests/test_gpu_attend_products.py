"""The products of attention over a card where their packing could show: a value that is no number, or an infinity, reaches its own
output dimension and no other (the value product pairs neighbouring dimensions), such a key its own token's score and no other (with 64
dimensions the score product pairs tokens), scales of either sign and zero (the sign is
taken into q), scores far apart, rows that end inside a round at every width, and head counts at the edges of the three row layouts.
Tolerances: the bounds of test_gpu_attend.py."""
import numpy as np
import pytest
import torch

import qkv_synth
from oracle import attend_ref, ref
from test_gpu_attend import bounds, build_card, check, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,G", [(64, 32), (128, 32), (256, 64)])
@pytest.mark.parametrize("rep", [1, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_no_number_stays_in_its_dimension(D, G, rep, value):
    L, H, T, t, d = 1, 2, 70, 37, D // 2 + 5
    print("[case] D=%d rep=%d value %s" % (D, rep, value), flush=True)
    bits = qkv_synth.make_bits_uniform_choice(T, D + rep).numpy()
    bits[t] = 16                                          # a raw row
    K, V = qkv_synth.make_kv(L, H, T, D, 31 + rep, "llama")
    counts = [int((bits == w).sum()) for w in (2, 4, 8, 16)]
    rd = ref.make_desc(L, H, T, D, G)
    clean = ref.quantize_pack(rd, K.numpy(), V.numpy(), bits, counts)
    V[0, 1, t, d] = value
    card = ref.quantize_pack(rd, K.numpy(), V.numpy(), bits, counts)
    q = np.random.default_rng(D + rep).standard_normal((L, H * rep, D)).astype(np.float16)
    scale = D ** -0.5
    out, lse, st = run_gpu(card, L, H, T, D, G, q, scale)
    assert st == 0
    want_o, want_lse = attend_ref.card_attend(clean, rd, q, scale)
    tol_o, tol_lse = bounds(clean, rd, q, scale)
    assert not np.isfinite(out[0, rep:, d]).any()         # every head of the second kv head
    out[0, rep:, d] = want_o[0, rep:, d]
    assert float(np.abs(out - want_o).max()) <= tol_o and float(np.abs(lse - want_lse).max()) <= tol_lse


def check_keys(card, rd, q, scale, exact):
    """`exact`: the query heads whose result the definition gives, a weight of zero for a score of -inf."""
    out, lse, st = run_gpu(card, rd.layers, rd.kv_heads, rd.tokens, rd.head_dim, rd.group_size, q, scale)
    with np.errstate(invalid="ignore"):
        want_o, want_lse = attend_ref.card_attend(card, rd, q, scale)
    kq, vq = ref.unpack_dequant(card, rd)
    k = np.abs(kq.view(np.float16).astype(np.float64))
    k[~np.isfinite(k)] = 0.0                              # such a token's weight is exactly zero: it has no part in the error
    ds = max(float((k[l, hq // (q.shape[1] // rd.kv_heads)] @ np.abs(q[l, hq].astype(np.float64))).max()) for l in range(rd.layers) for hq in exact)
    ds *= rd.head_dim * 2.0 ** -24 * scale
    base, vmax = (rd.tokens + 8) * 2.0 ** -24 + 2.0 ** -21, float(np.abs(vq.view(np.float16).astype(np.float64)).max())
    assert st == 0 and np.isfinite(want_o[:, exact]).all()
    assert float(np.abs(out[:, exact] - want_o[:, exact]).max()) <= (2 * ds + base) * vmax
    assert float(np.abs(lse[:, exact] - want_lse[:, exact]).max()) <= ds + base


@pytest.mark.parametrize("D,G", [(64, 32), (64, 64), (128, 32), (256, 64)])
@pytest.mark.parametrize("rep", [1, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_no_number_in_a_key_stays_with_its_token(D, G, rep, value):
    """Raw rows in either half of a round of 32 tokens, alone and several, at the ends of the card and of the segment."""
    H, T, scale = 2, 301, D ** -0.5
    for tokens in ([5], [21], [0, 31, 300], [96, 120, 150, 151]):
        print("[case] D=%d G=%d rep=%d key %s at %s" % (D, G, rep, value, tokens), flush=True)
        bits = np.full(T, 16, np.uint8)
        bits[100:150] = qkv_synth.make_bits_uniform_choice(50, D + rep).numpy()
        bits[tokens] = 16
        K, V = qkv_synth.make_kv(1, H, T, D, 41 + rep, "llama")
        q = np.random.default_rng(D + rep + tokens[0]).standard_normal((1, H * rep, D)).astype(np.float16)
        exact = list(range(rep))                          # all of the first kv head, whose keys are numbers
        for i, t in enumerate(tokens):
            d = (17 * i + 3 + D // 2) % D
            K[0, 1, t, d] = value
            if not np.isnan(value):                       # every other head of the second: a score of -inf
                q[0, rep::2, d] = -np.abs(q[0, rep::2, d]) * np.sign(value) - np.float16(0.01 * np.sign(value))
        if not np.isnan(value):
            exact += list(range(rep, 2 * rep, 2))
        rd = ref.make_desc(1, H, T, D, G)
        card = ref.quantize_pack(rd, K.numpy(), V.numpy(), bits, [int((bits == w).sum()) for w in (2, 4, 8, 16)])
        check_keys(card, rd, q, scale, exact)


@pytest.mark.parametrize("width", [2, 4, 8])
@pytest.mark.parametrize("D,rep", [(64, 3), (64, 8), (64, 12), (128, 4), (256, 2)])
def test_a_decoded_infinity_in_a_key_stays_with_its_token(width, D, rep):
    """A group whose zero point is -inf, against heads that are positive there: scores of -inf at 2, 4 and 8 bits too."""
    H, T, G, group = 2, 200, 32, 1
    for t in (3, 19, 64 + 16, 199):
        print("[case] D=%d rep=%d width %d token %d" % (D, rep, width, t), flush=True)
        rd, card = build_card(1, H, T, D, G, np.full(T, width, np.uint8), 50 + rep + width)
        card = card.copy()
        at = int(card[128:152].view(np.uint64)[{2: 0, 4: 1, 8: 2}[width]]) + ((1 * T + t) * (D // G) + group) * 4
        card[at:at + 4] = np.array([0x0000, 0xFC00], np.uint16).view(np.uint8)             # (scale, zero) = (0, -inf)
        q = np.random.default_rng(D + rep + t).standard_normal((1, H * rep, D)).astype(np.float16)
        q[..., group * G:(group + 1) * G] = np.abs(q[..., group * G:(group + 1) * G]) + np.float16(0.01)
        check_keys(card, rd, q, D ** -0.5, list(range(H * rep)))


@pytest.mark.parametrize("scale", [-0.09, 0.0, -0.0])
@pytest.mark.parametrize("D,rep", [(64, 8), (128, 4), (128, 16), (256, 5)])
def test_scales_that_are_not_positive(scale, D, rep):
    T = 300
    bits = qkv_synth.make_bits_uniform_choice(T, 7 + D + rep).numpy()
    rd, card = build_card(1, 2, T, D, 32, bits, 70 + rep)
    q = np.random.default_rng(rep).standard_normal((1, 2 * rep, D)).astype(np.float16)
    print("[case] scale %g D=%d rep=%d" % (scale, D, rep), flush=True)
    out, lse, st = run_gpu(card, 1, 2, T, D, 32, q, scale)
    want_o, want_lse = attend_ref.card_attend(card, rd, q, scale)
    tol_o, tol_lse = bounds(card, rd, q, abs(scale))
    assert st == 0 and float(np.abs(out - want_o).max()) <= tol_o and float(np.abs(lse - want_lse).max()) <= tol_lse


@pytest.mark.parametrize("width", [2, 4, 8, 16])
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("T", [1, 31, 33, 97, 193])
def test_rows_that_end_inside_a_round(width, D, T):
    check(1, 2, 3, T, 32, np.full(T, width, np.uint8), 3 * T + D + width, "attend %d-bit D=%d T=%d" % (width, D, T), D=D)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rep", [4, 5, 8, 9, 13, 16])
def test_head_counts_at_the_edges_of_the_layouts(D, rep):
    T = 257
    bits = qkv_synth.make_bits_uniform_choice(T, D + 3 * rep).numpy()
    check(1, 2, rep, T, 64, bits, D + 5 * rep, "attend D=%d rep=%d" % (D, rep), D=D)


@pytest.mark.parametrize("size", ["scale 1e7", "scale -3e8", "scale 1e12", "scale 1e30", "scale 1e35", "values"])
@pytest.mark.parametrize("D,rep,T", [(64, 1, 500), (64, 9, 90), (128, 4, 1100), (128, 6, 33), (256, 5, 300)])
def test_scores_far_apart(size, D, rep, T):
    """Scores whose fp32 spacing is larger than 1: one token decides, or two alike do, whatever the maximum rounds to."""
    H = 2
    rng = np.random.default_rng(D + rep + T)
    bits = qkv_synth.make_bits_uniform_choice(T, 5 + D + rep).numpy() if size.startswith("scale") else np.full(T, 16, np.uint8)
    bits[[2, T - 2]] = 16
    K, V = qkv_synth.make_kv(1, H, T, D, 80 + rep, "llama")
    q = rng.standard_normal((1, H * rep, D)).astype(np.float16)
    scale = float(size.split()[1]) if size.startswith("scale") else D ** -0.5
    if size == "values":
        K, q = (K.float() * 900).clamp(-60000, 60000).half(), (q.astype(np.float32) * 9000).astype(np.float16)
    K[0, 1, 2] = torch.from_numpy(q[0, rep] * np.float16(np.sign(scale) * (8 if size.startswith("scale") else 1)))
    K[0, 1, T - 2] = K[0, 1, 2]                           # two raw rows alike, the largest score of the second kv head's first head
    rd = ref.make_desc(1, H, T, D, 32)
    card = ref.quantize_pack(rd, K.numpy(), V.numpy(), bits, [int((bits == w).sum()) for w in (2, 4, 8, 16)])
    out, lse, st = run_gpu(card, 1, H, T, D, 32, q, scale)
    assert st == 0
    want_o, want_lse = attend_ref.card_attend(card, rd, q, scale)
    kq, vq = (x.view(np.float16).astype(np.float64)[0] for x in ref.unpack_dequant(card, rd))
    clear = 0
    for hq in range(H * rep):
        s = scale * (kq[hq // rep] @ q[0, hq].astype(np.float64))
        ds = D * 2.0 ** -24 * abs(scale) * float((np.abs(kq[hq // rep]) @ np.abs(q[0, hq].astype(np.float64))).max())
        s = np.sort(np.delete(s, 2)) if hq == rep else np.sort(s)
        if s[-1] - s[-2] < 2 * ds + 64:                   # the definition itself decides closer than fp32 sums can
            continue
        clear += 1
        print("[case] %s D=%d rep=%d head %d: largest score %.3g" % (size, D, rep, hq, s[-1]), flush=True)
        assert np.abs(out[0, hq] - want_o[0, hq]).max() <= ((T + 8) * 2.0 ** -24 + 2.0 ** -21) * np.abs(vq).max()
        assert abs(lse[0, hq] - want_lse[0, hq]) <= ds + 2.0 ** -22 * abs(want_lse[0, hq])
    assert clear > rep
