"""The products of attention over a card where their packing could show: a value that is no number, or an infinity, reaches its own
output dimension and no other (the value product pairs neighbouring dimensions), scales of either sign and zero (the sign is
taken into q), rows that end inside a round at every width, and head counts at the edges of the three row layouts.
Tolerances: the bounds of test_gpu_attend.py."""
import numpy as np
import pytest

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
