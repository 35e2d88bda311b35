"""Widths and card tables of sequences beyond one workgroup's registers (several launches, scratch inside the results):
lengths at the edges of its parts, ties of every kind at the cuts, pointers off their alignment, counts beyond 16 bits."""
import numpy as np
import pytest
import torch

import paper_2605_03884_amd as qkv
from oracle import ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def scores_of(kind, T, rng):
    if kind == "uniform":
        return rng.random(T, dtype=np.float32)
    if kind == "normal":
        return rng.standard_normal(T).astype(np.float32)
    if kind == "constant":
        return np.full(T, 0.25, np.float32)
    if kind == "few":                                    # ties at every cut, in every part
        return rng.integers(0, 5, T).astype(np.float32)
    s = rng.standard_normal(T).astype(np.float32)        # the ends of the total order
    s[:: 7] = np.float32(0.0); s[1:: 7] = np.float32(-0.0); s[2:: 7] = np.inf; s[3:: 7] = -np.inf; s[4:: 7] = np.nan
    return s


def check(T, kind, budget, shift=0):
    print("[case] T=%d %s budget %g shift %d" % (T, kind, budget, shift), flush=True)
    scores = scores_of(kind, T, np.random.default_rng(T + 1))
    want, counts = ref.assign_bits(scores, budget)
    s_buf = torch.empty(T + 4, device=DEV)
    s_dev = s_buf[shift:shift + T]
    s_dev.copy_(torch.from_numpy(scores))
    buf = torch.full((T + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    bits, got = qkv.assign_bits(s_dev, budget, bits=buf[16 + shift:16 + shift + T])
    assert got == counts.tolist()
    want_dev = torch.from_numpy(want).to(DEV)
    assert torch.equal(bits, want_dev)
    assert (buf[:16 + shift] == 0x5A).all() and (buf[16 + shift + T:] == 0x5A).all()

    desc = qkv.Desc.make(1, 1, T, 64, 32)
    n = qkv.card_bytes(desc, got)
    card = torch.full((n,), 0x5A, dtype=torch.uint8, device=DEV)
    buf.fill_(0x5A)
    bits = buf[16 + shift:16 + shift + T]
    assert qkv.assign_plan(desc, s_dev, budget, card, bits=bits) == got
    assert torch.equal(bits, want_dev)
    same = torch.full((n,), 0x5A, dtype=torch.uint8, device=DEV)       # the widths classified by the other kernel
    qkv.card_plan(desc, want_dev, got, same)
    assert torch.equal(card, same)                                     # header, tables and pads; nothing else touched
    card.fill_(0x5A)
    qkv.assign_plan(desc, s_dev, budget, card)                         # no widths wanted
    assert torch.equal(card, same)


@pytest.mark.parametrize("T", [16384, 16385, 20003, 32769, 32781, 40960, 40961, 57347, 131072, 131073, 524289, 4194245])
def test_lengths(T):
    check(T, "uniform", 4.0)


@pytest.mark.parametrize("kind", ["normal", "constant", "few", "ends"])
@pytest.mark.parametrize("budget", [2.0, 3.0, 5.0, 9.5, 16.0])
def test_ties_and_budgets(kind, budget):
    check(50003, kind, budget, shift=1)
    check(98304, kind, budget)


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_pointers_off_their_alignment(shift):
    check(70001, "few", 4.0, shift)
