"""The k chunks of batch members that leave them open (kc = 0): the length the
work list is built with (host), and the states of batches that mix open and
chosen lengths against single cavities (GPU; the same per-cell code: bit for
bit, the norms to the rounding of their grouping, 64 eps for sums of positive
terms).
"""
import numpy as np
import pytest

import paper_2006_02602_amd as C
from paper_2006_02602_amd import _lib

HEAD, ITEM = 64, 8


def member(n, dtype=0, kc=0, ti=0):
    m = _lib.CavBatchMember(C.Grid(*n, dtype=dtype).c(), C.Params().c(), 0x1000, 0x2000, 0x3000, 1 << 30, kc)
    m.ti = ti
    return m


def items(members):
    """Work items of a list of the members, from its table's size."""
    one = C.cavity_batch_table_bytes(members)
    base = C.cavity_batch_table_bytes([member((2, 2, 2))] * len(members)) - ITEM * len(members)
    return (one - base) // ITEM


def tiles(n, dtype, ti):
    w, h = C.batch_tile(dtype, ti)
    return -(-n[0] // w) * -(-n[1] // h)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("shapes", [
    [((2, 2, 2), 0, 0)], [((20, 20, 3), 0, 0)], [((64, 64, 64), 0, 0)], [((24, 40, 96), 0, 0), ((50, 61, 37), 0, 0)],
    [((96, 96, 96), 0, 0)] * 40, [((30, 20, 200), 5, 0), ((33, 17, 9), 0, 0), ((20, 20, 20), 0, 1)],
    [((40, 40, 40), 7, 0), ((21, 9, 12), 12, 1)]])
def test_open_length_balances_the_items(shapes, dtype):
    """The length is one that no other even cut of the deepest open member
    beats in sum(k + 3) / 256 + K (256 compute units, as on the CPU)."""
    narrow = {0: 32, 1: 16}[dtype]
    ms = [member(n, dtype, kc, narrow if t else 0) for n, kc, t in shapes]
    deepest = max([n[2] for n, kc, _ in shapes if kc == 0], default=0)

    def count(k):
        return sum(tiles(n, dtype, narrow if t else 0) * -(-n[2] // min(kc or k, n[2])) for n, kc, t in shapes)

    def cost(k):
        s = sum(tiles(n, dtype, narrow if t else 0) * (n[2] + 3 * -(-n[2] // min(kc or k, n[2]))) for n, kc, t in shapes)
        return s / 256 + k

    lengths = {max(2, -(-deepest // c)) for c in range(1, deepest + 1)} or {1}
    best = min(cost(k) for k in lengths)
    import torch
    if not torch.cuda.is_available():
        assert items(ms) in {count(k) for k in lengths if cost(k) <= best * (1 + 1e-12)}
    assert items(ms) in {count(k) for k in lengths}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [0, 1])
def test_open_and_chosen_lengths_in_one_batch(dtype):
    import torch
    narrow = {0: 32, 1: 16}[dtype]
    mix = [((66, 9, 97), 0, 0), ((17, 17, 2), 0, 0), ((40, 33, 31), 4, narrow), ((5, 6, 50), 0, narrow),
           ((31, 64, 3), 100, 0)]
    print("open chunks", dtype, flush=True)
    b = C.Batch([(C.Grid(*n, dtype=dtype), C.Params(Ra=2e4), kc, ti) for n, kc, ti in mix]).init(range(len(mix)), 0.3)
    b.step(3)
    for m, (n, _, _) in enumerate(mix):
        a = C.Cavity(C.Grid(*n, dtype=dtype), C.Params(Ra=2e4)).init(m, 0.3)
        a.step(3)
        torch.cuda.synchronize()
        inner = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
        assert torch.equal(a.fields()[inner], b.fields(m)[inner])
        na, nb = np.array(a.norms()), np.array(b.norms(m))
        assert (np.abs(na - nb) <= 64 * np.finfo(np.float64).eps * na).all()
