"""Batches that go to burst_kernel, at the edges of its shapes: the blocks of a wavefront, of a workgroup of
four, eight and sixteen wavefronts and of two to four passes, with "block -1" in a pass, in one of its
own and beside the first; chunks in one workgroup and in several; more chunks than compute units; AAD of
every kind and IVs of other lengths — against the CPU oracle, bit for bit.  (Which kind of burst_kernel
and how many passes a shape takes: tests/test_routes.py.)"""
import numpy as np
import pytest
import torch

import oracle
import workloads
from device_batch import DeviceBatch
from test_gpu_parity import _full_parity

import paper_2411_03357_amd as pgcm

pytestmark = pytest.mark.gpu

KIB = 1024


def _workload(name, lens, alens, key_bytes=32, iv_bytes=12):
    rng = np.random.default_rng([workloads.BASE_SEED, 577, len(name), len(lens)])
    n = len(lens)
    lens = np.array(lens, np.uint64)
    alens = np.resize(np.array(alens, np.int64), n)
    offsets, total = workloads._layout(lens)
    aad_off = np.zeros(n + 1, np.uint64)
    aad_off[1:] = np.cumsum(alens)
    ivs = (workloads.iv_sequence((1 << 61) + 5, n) if iv_bytes == 12 else
           rng.integers(0, 256, (n, iv_bytes), dtype=np.uint8))
    return workloads.Workload(name, 960, rng.integers(0, 256, key_bytes, dtype=np.uint8), ivs, lens,
                              offsets, total, "u8",
                              rng.integers(0, 256, int(alens.sum()), dtype=np.uint8), aad_off)


# bytes around the blocks of 16, 64, 128, 256, 512, 768 blocks
_EDGES = [16 * b + d for b in (16, 64, 128, 256) for d in (-17, -16, -1, 0, 1, 16)]
_MORE = [16 * b + d for b in (256, 512, 768, 1024) for d in (-16, 0, 1)]

SHAPES = {
    # one chunk a call is by far the usual case: every edge by itself
    **{"one_%d" % v: ([v], [0]) for v in (1, 16, 255, 256, 257, 1024, 2048, 4096, 8192)},
    **{"one_aad_%d" % v: ([v], [16]) for v in (16, 1008, 1024, 2048, 4080, 4096)},
    # the workgroup of the AAD's first blocks ends before "block -1", and with it
    "aad_before": ([1023 * 16 - 12], [33]),
    "aad_with_last": ([1024 * 16], [33]),
    "short": ([0, 1] + _EDGES, [0]),
    "short_aad": ([0, 1] + _EDGES, [16, 0, 5, 64, 17, 1, 48]),
    # the AAD fills lanes, a pass, and is longer than goes in lanes
    "long_aad": ([0, 5, 1024, 4096, 4097, 8192], [1008, 1024, 1025, 16, 3000, 1024]),
    # workgroups of one pass of 64 blocks or of 128: as many as there are compute units, a set of shares and one
    # more, both in one launch, and payload, AAD and "block -1" at the edges of a pass
    "apart_64_most": ([256 * 1024], [0]),
    "apart_64_set": ([32 * 1024, 16 * 1024 + 1], [0]),
    "apart_128_set": ([32 * 1024 + 1], [0]),
    "apart_64_sets": ([64 * 1024 + 1], [0]),
    "apart_128_most": ([512 * 1024 - 16], [16]),
    "apart_128_over": ([256 * 1024], [7]),
    "apart_64_edges": ([9000, 0, 1] + [16 * b + d for b in (64, 128, 576) for d in (-1, 0, 1)],
                       [0, 1008, 16, 1024, 3000, 1025, 33]),
    "apart_128_edges": ([290 * KIB, 0, 1] + [16 * b + d for b in (128, 256, 640) for d in (-1, 0, 1)],
                        [1024, 1008, 16, 0, 3000, 1025, 33]),
    # short chunks, some of them in several workgroups of one pass of 64 blocks or of 128; and too many for that
    "spread_64_most": ([8192] * 32, [0]),
    "spread_64_edges": ([0, 1, 8192] + _EDGES[12:], [1008, 0, 16, 1025, 3000, 33]),
    "spread_128_most": ([8192 - 16 * (i % 3) for i in range(56)] + [4096] * 8, [0]),
    "whole": ([8192] * 65 + _EDGES, [0]),
    # ... with AAD of every kind: a workgroup of one to three passes for each of more than 64 chunks
    "whole_aad": ([0, 1] + _EDGES + [8192, 4096] + [16 * b + d for b in (257, 448, 500) for d in (-1, 0, 1)] + [20] * 34,
                  [16, 0, 5, 64, 17, 1, 48]),
    "whole_long_aad": ([0, 5, 1024, 4096, 4097, 8192, 8177] * 10, [1008, 1024, 1025, 16, 3000]),
    # workgroups of sixteen wavefronts and one pass, the first ones of chunks short: AAD in lanes, at the edges of a
    # row and longer, "block -1" in the first workgroup and in the second
    "fold_1": ([v + 16 * 4096 for v in _MORE], [0, 16, 33, 1008, 1024, 1025, 3000]),
    "fold_1_most": ([1 << 20], [0]),
    "fold_1_aad_most": ([(1 << 20) - 64 * 16], [1024]),
    "fold_1_aad_before": ([(150 * 256 - 1) * 16 - 12], [33]),
    "fold_1_aad_with_last": ([150 * 4096], [33]),
    "fold_1_long_aad": ([513 * KIB], [3000]),
    # workgroups of one to four passes, some of them short; in 2 and 4 a chunk's first may make one more
    "two": ([300 * KIB, 8 * KIB + 16, 9000, 1], [0, 16, 70]),
    "passes_1": (_MORE + [200 * KIB], [0, 16]),
    "passes_2": ([v + 40 * 4096 for v in _MORE], [16, 0, 33]),
    "passes_4": ([v + 60 * 4096 for v in _MORE], [0, 0, 20]),
    "even_2": ([512 * 4096 - 16], [0]),
    "even_4": ([1024 * 4096 - 16 * 64], [1008]),
    "even_4_some": ([v + 70 * 4096 for v in _MORE], [0, 0, 20]),
    # three passes, and chunks whose first workgroup makes one more than the others: of AAD alone, with
    # payload, and of a short last chunk
    "passes_3": ([600 * 4096 - 5], [0]),
    "spare_1": ([256 * 4096], [16]),
    "spare_1_payload": ([256 * 4096 + 100], [0]),
    "spare_1_long_aad": ([256 * 4096], [3000]),
    "spare_2": ([512 * 4096 - 48 * 16], [1008]),
    "spare_3": ([768 * 4096 + 4095], [0]),
    "spare_of_some": ([64 * 4096] * 7 + [63 * 4096 + 1, 5], [16, 0, 40]),
    # sweeps of four passes, the first of them whole or not; with block -1, AAD or the chunk's start in the
    # spare one, in a missing one; rows further from the end than KeyTables::row_hop reaches
    "sweeps_2": ([256 * 5 * 4096 - 5], [0]),
    "sweeps_2_whole": ([256 * 8 * 4096 - 16], [3000]),
    "sweeps_2_spare": ([256 * 8 * 4096], [16]),
    "sweeps_2_missing": ([2 << 20] * 3, [0]),
    "sweeps_2_missing_2": ([85 * 6 * 4096] * 3, [0]),
    "sweeps_3": ([100 * 9 * 4096 + 1, 150 * 9 * 4096 - 16, 70000, 8200], [0, 1008, 40, 16]),
    "sweeps_4": ([256 * 14 * 4096 + 33], [20]),
    "sweeps_of_each": ([14 * 4096 + 13 * i for i in range(200)], [16, 0, 3000, 7]),
    # more chunks than compute units: mixed, and all of much the same length
    "many_mixed": ([(37 * i * i) % 8192 + 1 for i in range(40)] + [20] * 260, [0, 9]),
    "many_even": ([4096 + 16 * (i % 3) for i in range(300)], [0, 16]),
    # ... so many passes of sixteen wavefronts that chunks of more than one have a workgroup for each
    "many_apart": ([1600 + (97 * i * i) % 6593 for i in range(300)], [0, 16, 40, 1008, 0, 3000]),
    "many_apart_512": ([4096, 8192, 4096, 4097, 8177] * 30 + [4096] * 160 + [4097] * 56, [0]),
    "many_apart_513": ([4096, 8192, 4096, 4097, 8177] * 30 + [4096] * 159 + [4097] * 57, [0]),
    "many_long": ([8192 - i % 20 for i in range(270)], [0, 64]),
}


@pytest.mark.parametrize("shape", SHAPES)
def test_shapes(shape):
    lens, alens = SHAPES[shape]
    w = _workload(shape, lens, alens)
    flips = [(i, 3, 1, "tag") for i in {0, w.n // 2}] if w.n > 1 else []
    _full_parity(w, flip=flips)


@pytest.mark.parametrize("key_bytes,iv_bytes", [(16, 12), (24, 16), (32, 8), (16, 40), (32, 1040)])
@pytest.mark.parametrize("shape", ["short_aad", "passes_1", "apart_64_edges", "apart_128_edges", "spread_64_edges",
                                   "whole_aad", "whole_long_aad", "fold_1", "passes_4", "sweeps_2_missing",
                                   "many_even", "many_mixed", "many_apart"])
def test_other_keys_and_ivs(shape, key_bytes, iv_bytes):
    lens, alens = SHAPES[shape]
    _full_parity(_workload(shape, lens[:40] if shape == "short_aad" else lens, alens, key_bytes, iv_bytes))


@pytest.mark.parametrize("iv_bytes", (12, 40))
@pytest.mark.parametrize("longest", (1024, 2048))
@pytest.mark.parametrize("n", (255, 256, 257, 512))
def test_workgroups_with_and_without_a_wavefront_more(n, longest, iv_bytes):
    """up to a workgroup of four or of eight wavefronts for each compute unit has one more, beyond that none: chunks
    that are empty, of AAD alone and of a whole pass, some rejected"""
    lens = [0, longest, 1, longest - 16, 777] * 103
    w = _workload("more_%d" % longest, lens[:n], [0, 0, 16, 5, 1025, 33, 1024], iv_bytes=iv_bytes)
    _full_parity(w, flip=[(0, 3, 1, "tag"), (1, 0, 5, "tag"), (n - 1, 9, 2, "tag")])


# chunks of at most 64 blocks, AAD included, and of at most 128: (longest, AAD lengths, wavefronts with blocks)
MORE = {"four": (1024 - 48, [0, 16, 5, 33], 4), "four_aad": (0, [1008], 4), "eight": (2048 - 48, [0, 16, 5, 33], 8),
        "eight_aad": (1040, [1008, 0, 1000], 8)}


def more(n, shape):
    """n such chunks, each in one workgroup: the longest among them, if there is payload at all"""
    longest, alens, waves = MORE[shape]
    lens = [longest, 0, min(longest, 1), max(longest - 16, 0), longest // 2 + 5 if longest else 0]
    return np.resize(lens, n), np.resize(alens, n), waves


@pytest.mark.parametrize("iv_bytes", (12, 40))
@pytest.mark.parametrize("shape", MORE)
@pytest.mark.parametrize("n", (65, 255, 256, 257, 512))
def test_workgroups_of_four_and_of_eight(n, shape, iv_bytes):
    """up to a workgroup for each compute unit has a wavefront more than its blocks need, beyond that none, whose blocks
    make E_K(J0) as well"""
    lens, alens, _ = more(n, shape)
    _full_parity(_workload("of_%s" % shape, lens, alens, iv_bytes=iv_bytes),
                 flip=[(0, 3, 1, "tag"), (2, 0, 5, "tag"), (n - 1, 9, 2, "tag")])


# workgroups of sixteen wavefronts, some of two passes in rows, which others hash meanwhile when decrypting, and some of one,
# in quads; "spare": chunks' first workgroups make up to three and hash behind the cipher.  65 chunks and more have their
# descriptors in pinned memory.
APART = {
    "halves": ([400 * 4096 + 17, 4096, 100 * 4096 - 15, 1], [16, 0, 33]),
    "halves_long_aad": ([400 * 4096 - 50 * 16], [3000]),
    "spare": ([512 * 4096 - 48 * 16], [1008]),
    "spare_some": ([100 * 4096 + 1, 103 * 4096 - 16, 150 * 4096, 155 * 4096 - 5, 4096], [0, 16, 1008]),
    "staged": ([6 * 4096 - 16 * (i % 3) - i % 2 for i in range(80)], [0, 16, 5]),
    "staged_spare": ([5 * 4096 - 16 * (i % 3) - i % 2 for i in range(100)], [0, 16, 5]),
}


@pytest.mark.parametrize("in_place", (False, True))
@pytest.mark.parametrize("key_bytes,iv_bytes", [(32, 12), (24, 40)])
@pytest.mark.parametrize("shape", APART)
def test_some_rows_hashed_apart(shape, key_bytes, iv_bytes, in_place):
    """with nothing changed, and with a bit of the first, a middle and the last chunk: in the first workgroup, which may
    be the one of fewer or more passes, half way and in the last block"""
    lens, alens = APART[shape]
    w = _workload("some_%s" % shape, lens, alens, key_bytes, iv_bytes)
    host = w.payload_host()
    srcs = [w.chunk(host, i) for i in range(w.n)]
    aads = [np.frombuffer(w.aad_of(i), np.uint8) for i in range(w.n)]
    cts, tags, _ = oracle.encrypt_batch(w.key, w.ivs, aads, srcs, nthreads=8)
    wire = np.zeros_like(host)
    for i in range(w.n):
        w.chunk(wire, i)[:] = cts[i]
    key = pgcm.expand_key_bytes(w.key.tobytes())
    b = DeviceBatch(w, torch.from_numpy(host).cuda())
    b.tags.copy_(torch.from_numpy(np.ascontiguousarray(tags).reshape(-1)))
    for at in (None, 0.0, 0.5, 1.0):
        flipped = set() if at is None else {0, w.n // 2, w.n - 1}
        sent = wire.copy()
        for i in flipped:
            w.chunk(sent, i)[int(at * (lens[i] - 1))] ^= 32
        b.cipher.copy_(torch.from_numpy(sent))
        out = b.cipher if in_place else b.back
        b.decrypt(key, dst=out)
        torch.cuda.synchronize()
        got, ok = out.cpu().numpy(), b.ok.cpu().tolist()
        for i in range(w.n):
            assert ok[i] == (i not in flipped), (at, i)
            assert np.array_equal(w.chunk(got, i), np.zeros_like(srcs[i]) if i in flipped else srcs[i]), (at, i)
    key.free()


# one pass of 256 blocks a workgroup, and two, whose rows are hashed by wavefronts of their own when decrypting: whole,
# short, ragged, with AAD in lanes of the first row, of a pass of its own, and too long for lanes
_HASHED_APART = {
    "one": ([1 << 20], [0]), "one_short": ([(1 << 20) - 65 * 16 - 3], [33]),
    "two": ([2 << 20], [0]), "two_ragged": ([(2 << 20) - 5], [0]), "two_aad": ([(2 << 20) - 64 * 16], [1008]),
    "two_long_aad": ([(2 << 20) - 48 * 16], [3000]), "two_half": ([400 * 4096 + 17], [16]),
    "some": ([700 * KIB, 300 * KIB + 1, 64 * KIB - 16, 5000, 1, 0], [0, 16, 1024, 5]),
}


@pytest.mark.parametrize("in_place", (False, True))
@pytest.mark.parametrize("key_bytes,iv_bytes", [(32, 12), (16, 40)])
@pytest.mark.parametrize("shape", _HASHED_APART)
def test_rows_hashed_apart(shape, key_bytes, iv_bytes, in_place):
    lens, alens = _HASHED_APART[shape]
    w = _workload("apart_%s" % shape, lens, alens, key_bytes, iv_bytes)
    host = w.payload_host()
    srcs = [w.chunk(host, i) for i in range(w.n)]
    aads = [np.frombuffer(w.aad_of(i), np.uint8) for i in range(w.n)]
    cts, tags, _ = oracle.encrypt_batch(w.key, w.ivs, aads, srcs, nthreads=8)
    key = pgcm.expand_key_bytes(w.key.tobytes())
    for flipped in (None, 0, w.n // 2):
        b = DeviceBatch(w, torch.from_numpy(host).cuda())
        wire = np.zeros_like(host)
        for i in range(w.n):
            w.chunk(wire, i)[:] = cts[i]
        if flipped is not None and lens[flipped]:
            w.chunk(wire, flipped)[lens[flipped] * 2 // 3] ^= 16
        b.cipher.copy_(torch.from_numpy(wire))
        b.tags.copy_(torch.from_numpy(np.ascontiguousarray(tags).reshape(-1)))
        out = b.cipher if in_place else b.back
        b.decrypt(key, dst=out)
        torch.cuda.synchronize()
        got, ok = out.cpu().numpy(), b.ok.cpu().tolist()
        for i in range(w.n):
            rejected = i == flipped and lens[i] != 0
            assert ok[i] == (0 if rejected else 1), (flipped, i)
            assert np.array_equal(w.chunk(got, i), np.zeros_like(srcs[i]) if rejected else srcs[i]), (flipped, i)
    key.free()


@pytest.mark.parametrize("iv_bytes", (12, 16, 40))
@pytest.mark.parametrize("length", (1, 1024, 8192))
def test_one_chunk_somewhere_in_the_callers_arrays(length, iv_bytes):
    """a key that shares no launch has one chunk of several: IV, tag and verdict are at its place, and what other
    chunks have there stays as it is"""
    w = _workload("one_of_three", [5000, 100, length], [16], iv_bytes=iv_bytes)
    host = w.payload_host()
    other = np.arange(16, dtype=np.uint8)
    raw = [w.key, w.key, other]
    keys = [pgcm.expand_key_bytes(w.key.tobytes()), pgcm.expand_key_bytes(other.tobytes())]
    pgcm.set_one_launch(keys[1], False)
    b = DeviceBatch(w, torch.from_numpy(host).cuda())
    index = np.array([0, 0, 1], np.uint32)
    pgcm.encrypt_batch_keys(keys, index, b.ivs, iv_bytes, b.aad_ptrs, b.aad_lens, b.ptrs(b.plain), b.lens,
                            b.ptrs(b.cipher), b.tags)
    b.tags.view(-1, 16)[1, 3] ^= 4
    pgcm.decrypt_verify_batch_keys(keys, index, b.ivs, iv_bytes, b.aad_ptrs, b.aad_lens, b.ptrs(b.cipher), b.lens,
                                   b.ptrs(b.back), b.tags, b.ok)
    b.tags.view(-1, 16)[1, 3] ^= 4
    torch.cuda.synchronize()
    cipher, tags = b.cipher.cpu().numpy(), b.tags.cpu().numpy().reshape(-1, 16)
    for i in range(w.n):
        ct, tag = oracle.encrypt(raw[i], w.ivs[i], np.frombuffer(w.aad_of(i), np.uint8), w.chunk(host, i))
        assert w.chunk(cipher, i).tobytes() == ct and tags[i].tobytes() == tag, i
    assert b.ok.cpu().tolist() == [1, 0, 1]
    assert np.array_equal(w.chunk(b.back.cpu().numpy(), 2), w.chunk(host, 2))
    for key in keys:
        key.free()
