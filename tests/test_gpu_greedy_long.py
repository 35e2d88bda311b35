"""The greedy allocator where its kernels change over: tokens per thread, one workgroup against several, parts of the scratch,
pointers off their alignment, and budgets that end inside equal keys or cover everything."""
import numpy as np
import pytest
import torch

import paper_2605_03884_amd as qkv
from oracle import ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T", [2048, 2049, 16384, 16385, 32769, 41759, 41760, 62001, 131072, 1400003])
@pytest.mark.parametrize("kind", ["uniform", "few", "zeros"])
def test_lengths(T, kind):
    print("[case] T=%d %s" % (T, kind), flush=True)
    rng = np.random.default_rng(T)
    scores = {"uniform": lambda: rng.random(T, dtype=np.float32),
              "few": lambda: rng.integers(0, 4, T).astype(np.float32),
              "zeros": lambda: np.where(rng.random(T) < 0.001, rng.standard_normal(T), 0.0).astype(np.float32)}[kind]()
    for shift, budget in ((0, 4.0), (1, 2.7), (3, 11.3), (2, 16.0), (0, 2.0)):
        if T > 200000 and budget not in (4.0, 2.7):
            continue
        want, counts = ref.assign_bits_greedy(scores, budget)
        s = torch.empty(T + 4, device=DEV)[shift:shift + T]
        s.copy_(torch.from_numpy(scores))
        buf = torch.full((T + 32,), 0x5A, dtype=torch.uint8, device=DEV)
        bits, got = qkv.assign_bits_greedy(s, budget, bits=buf[8 + shift:8 + shift + T])
        torch.cuda.synchronize()
        assert torch.equal(bits, torch.from_numpy(want).to(DEV)), (budget, shift)
        assert got.cpu().tolist() == counts.tolist(), (budget, shift)
        assert (buf[:8 + shift] == 0x5A).all() and (buf[8 + shift + T:] == 0x5A).all()


@pytest.mark.parametrize("T", [600, 5000, 9000, 30000, 40000])
def test_last_key_shared_by_many(T):
    """The budget ends among equal keys: in a wave's first, last or middle tokens, on and off the four of a thread, at every level."""
    scores = np.where(np.arange(T) % 5 == 3, 0.5, 1.0).astype(np.float32)
    s = torch.from_numpy(scores).to(DEV)
    for budget in (2.001, 2.002, 2.057, 2.114, 2.228, 2.3, 2.456, 2.911, 3.59, 3.6, 4.3, 5.501, 5.6, 6.777, 9.119, 12.003, 15.999):
        print("[case] T=%d budget %g" % (T, budget), flush=True)
        want, counts = ref.assign_bits_greedy(scores, budget)
        bits, got = qkv.assign_bits_greedy(s, budget)
        torch.cuda.synchronize()
        assert torch.equal(bits, torch.from_numpy(want).to(DEV)), budget
        assert got.cpu().tolist() == counts.tolist(), budget
