"""How many tasks attention over a card is cut into, read off the workspace the library asks for (host arithmetic, no GPU)."""
import pytest

import paper_2605_03884_amd as qkv


def tasks(L, H, T, D, rep):
    floats = qkv.card_attend_workspace(qkv.Desc.make(L, H, T, D, 32), H * rep) // 4 - 4
    per_task = L * H * rep * (D + 2)
    assert floats % per_task == 0
    return floats // per_task


def base_tasks(L, H, T, rep):
    """Tasks of as many tokens as the scores' LDS holds, smaller where those would leave wave slots empty, and 3 to spare."""
    room = 1536 // ((rep + 3) // 4 * 4)
    c = room // 192 * 192 if room >= 192 else 64
    while c > 192 and L * H * ((T + c - 1) // c + 2) < 4096:
        c -= 192
    return (T + c - 1) // c + 3


@pytest.mark.parametrize("L,H", [(32, 8), (48, 8), (64, 8), (32, 1), (1, 8), (1, 1)])
@pytest.mark.parametrize("D", [64, 128, 256])
def test_a_finer_cut_fits_the_wave_slots_and_the_fixed_scratch(L, H, D):
    """A cut beyond the least number of tasks fills the chip's 4096 wave slots once at most, leaves the merge no more than 96 partials
    a head, and qkv_card_attend_static has the room for it (16 MiB), so that it cuts - and rounds - like the call with a workspace."""
    finer = 0
    for rep in (1, 2, 3, 4, 5, 16):
        for T in list(range(1, 4000, 37)) + [5000, 8192, 20000, 32768]:
            n, base = tasks(L, H, T, D, rep), base_tasks(L, H, T, rep)
            assert n >= base
            if n > base:
                finer += 1
                assert L * H * n <= 4096 and n <= min(96, T // 48 + 3), (L, H, T, D, rep, n)
                assert qkv.card_attend_workspace(qkv.Desc.make(L, H, T, D, 32), H * rep) <= 16 << 20
                assert rep <= 4 and D <= 128
    assert (finer > 0) == (D <= 128)
