"""Batch's check that the offsets fit the queries judges every offsets tensor by
its own contents, also one that takes the memory of a tensor freed before."""
import pytest
import torch

idx = pytest.importorskip("paper_2506_01576_amd")


def _batch():
    bt = idx.Batch.__new__(idx.Batch)
    bt.key_bits, bt.count, bt._total_seen = 64, 1, {}
    return bt


def test_offsets_in_reused_memory():
    bt, memory = _batch(), bytearray(16)
    for total in (5, 11, 6, 12):
        memory[8:16] = total.to_bytes(8, "little")
        offsets = torch.frombuffer(memory, dtype=torch.int64)
        if total <= 10:
            bt._check_total(offsets, 10, exact=False)
        else:
            with pytest.raises(ValueError):
                bt._check_total(offsets, 10, exact=False)
        del offsets


def test_offsets_changed_in_place():
    bt = _batch()
    offsets = torch.tensor([0, 5])
    for t in (offsets, offsets[:], offsets):
        bt._check_total(t, 10, exact=False)
    offsets[1] = 11
    with pytest.raises(ValueError):
        bt._check_total(offsets, 10, exact=False)
