"""How a chunk of several workgroups ends: their shares of its tag are added up by atomics, in one step up to
32 workgroups and in sets of 32 above that.  Both sides of either edge, by themselves and several chunks at
a time, pass after pass over the same slots, with tags wrong in each of their words; against the CPU
oracle, bit for bit."""
import numpy as np
import pytest
import torch

from device_batch import DeviceBatch, expand
from test_gpu_bursts import _workload
from test_gpu_parity import _oracle_encrypt

pytestmark = pytest.mark.gpu

PASS = 4096   # bytes of a workgroup of one pass; "block -1" begins the chunk


def _of(groups):
    return groups * PASS - 16


@pytest.mark.parametrize("groups", [[2], [31], [32], [33], [64], [65], [255], [2, 33, 64, 1, 32], [96, 97]])
def test_groups_of_a_chunk(groups):
    w = _workload("ends", [_of(g) for g in groups], [0])
    host = w.payload_host()
    key = expand(w)
    cts, tags = _oracle_encrypt(w, host)
    b = DeviceBatch(w, torch.from_numpy(host).cuda())
    for turn in range(6):
        b.cipher.zero_()
        b.tags.zero_()
        b.encrypt(key)
        torch.cuda.synchronize()
        assert np.array_equal(b.tags.cpu().numpy().reshape(-1, 16), tags), turn
        cipher = b.cipher.cpu().numpy()
        for i in range(w.n):
            assert np.array_equal(w.chunk(cipher, i), cts[i]), (turn, i)
        # one chunk of them with a bit of its tag wrong, in another word each turn; twice it is right
        wrong = turn % w.n if turn < 4 else -1
        received = b.tags.clone()
        if wrong >= 0:
            received[16 * wrong + 4 * turn + 1] ^= 1 << turn
        b.back.fill_(0xDD)
        b.decrypt(key, tags=received)
        torch.cuda.synchronize()
        assert b.ok.cpu().numpy().tolist() == [int(i != wrong) for i in range(w.n)], turn
        back = b.back.cpu().numpy()
        for i in range(w.n):
            plain = w.chunk(back, i)
            assert np.array_equal(plain, w.chunk(host, i)) if i != wrong else not plain.any(), (turn, i)
    key.free()
