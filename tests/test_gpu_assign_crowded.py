"""Widths, card tables and greedy widths of scores that crowd together - one value, two, a narrow range, one histogram bucket, one value
among others, all in one stretch - at the lengths where the number of keys per thread changes: waves whose lanes share a bucket,
cuts that share a prefix until the last pass, cuts that no token lies behind."""
import numpy as np
import pytest
import torch

import paper_2605_03884_amd as qkv
from oracle import ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

KINDS = {
    "one value": lambda u: np.full(u.size, np.float32(0.37)),
    "two values": lambda u: np.where(u < 0.5, np.float32(0.0), np.float32(1.0)),
    "narrow": lambda u: np.float32(0.5) + u * np.float32(1e-4),
    "one bucket": lambda u: np.float32(0.5) + u * np.float32(0.06),
    "half zeros": lambda u: np.where(u < 0.5, np.float32(0.0), u),
    "half in one stretch": lambda u: np.where(np.arange(u.size) < u.size // 2, np.float32(0.6), u),
}


@pytest.mark.parametrize("T", [4096, 4097, 8192, 8193, 16384, 16385, 32768])
@pytest.mark.parametrize("kind", list(KINDS))
def test_crowded_scores(T, kind):
    print("[case] T=%d %s" % (T, kind), flush=True)
    scores = KINDS[kind](np.random.default_rng(T).random(T, dtype=np.float32)).astype(np.float32)
    s = torch.from_numpy(scores).to(DEV)
    for budget in (2.0, 2.6, 4.0, 9.0, 16.0):
        want, counts = ref.assign_bits(scores, budget)
        bits, got = qkv.assign_bits(s, budget)
        assert got == counts.tolist()
        want_dev = torch.from_numpy(want).to(DEV)
        assert torch.equal(bits, want_dev), budget
        desc = qkv.Desc.make(1, 1, T, 64, 32)
        card = torch.full((qkv.card_bytes(desc, got),), 0x5A, dtype=torch.uint8, device=DEV)
        same = card.clone()
        qkv.assign_plan(desc, s, budget, card)
        qkv.card_plan(desc, want_dev, got, same)
        assert torch.equal(card, same), budget
        want, counts = ref.assign_bits_greedy(scores, budget)
        bits, got = qkv.assign_bits_greedy(s, budget)
        assert torch.equal(bits, torch.from_numpy(want).to(DEV)), budget
        assert got.cpu().tolist() == counts.tolist(), budget
