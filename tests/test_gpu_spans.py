"""Batches cut into spans of rows: chunks that a wavefront, a workgroup or several share, that end at
and next to the edges of a row, keys with fewer rows than a workgroup has wavefronts, lists of
chunks longer than a workgroup keeps in LDS, and IVs of many blocks — against the CPU oracle, bit for
bit."""
import numpy as np
import pytest
import torch

import iv_craft
import openssl_ref
import oracle
import workloads
from device_batch import DeviceBatch

import paper_2411_03357_amd as pgcm

pytestmark = pytest.mark.gpu

KIB, MIB = 1024, 1 << 20


def _even(rng, n, lo, hi):
    return [int(v) for v in np.exp(rng.uniform(np.log(lo), np.log(hi), n))]


# name: (chunk lengths, bytes of each key, how the keys go round the chunks, bytes of an IV)
SHAPES = {
    # next to nothing: a key with one row, one with a few, and empty chunks
    "least": lambda r: ([1, 0, 4 * KIB, 16, 0, 1041], (32, 16), 2, 12),
    # the edges of rows, with a row in front for the blocks before block 0 and without
    "edges": lambda r: ([k * KIB + d for k in (1, 2, 3, 15, 16, 17) for d in (-16, -1, 0, 1, 16)],
                        (16, 24, 32), 3, 16),
    # a few long chunks: shares of few rows, every chunk in many workgroups
    "long": lambda r: (_even(r, 17, 700 * KIB, 2 * MIB), (32, 24), 2, 12),
    # as many chunks as wavefronts, one key with nearly all of them
    "dealt": lambda r: (_even(r, 700, 30 * KIB, 90 * KIB), (32, 16, 32), 40, 12),
    # more chunks than shares: cut in equal parts, lists longer than LDS has room for
    "many": lambda r: (_even(r, 9000, 40, 3 * KIB), (32,), 1, 12),
    # shares of many rows
    "big": lambda r: (_even(r, 60, 500 * KIB, 2 * MIB) + [9 * MIB + 5], (16,), 1, 12),
    # IVs of several blocks, up to the edges of a row of 64 and beyond, hashed by the wavefronts that
    # need them: chunks cut into spans, and one-launch batches of one pass and of four
    "iv_17": lambda r: (_even(r, 90, 4 * KIB, 500 * KIB), (32, 16), 2, 17),
    "iv_1000": lambda r: (_even(r, 900, 40, 30 * KIB), (24,), 1, 1000),
    "iv_1024": lambda r: ([1, 5000, 0, 8 * KIB], (32,), 1, 1024),
    "iv_1025": lambda r: ([300 * KIB + 5], (32,), 1, 1025),
    "iv_2064": lambda r: (_even(r, 12, 300 * KIB, 350 * KIB), (16,), 1, 2064),
    "iv_3089": lambda r: (_even(r, 20, KIB, 90 * KIB), (24, 32), 2, 3089),
}


@pytest.mark.parametrize("shape", SHAPES)
def test_spans(shape):
    rng = np.random.default_rng([workloads.BASE_SEED, 1618, len(shape)])
    lens, key_bytes, cycle, iv_bytes = SHAPES[shape](rng)
    n = len(lens)
    lens = np.array(lens, np.uint64)
    alens = rng.integers(0, 70, n)
    offsets, total = workloads._layout(lens)
    aad_off = np.zeros(n + 1, np.uint64)
    aad_off[1:] = np.cumsum(alens)
    ivs = rng.integers(0, 256, (n, iv_bytes), dtype=np.uint8)
    raw_keys = [rng.integers(0, 256, b, dtype=np.uint8) for b in key_bytes]
    w = workloads.Workload("spans_" + shape, 900, raw_keys[0], ivs, lens, offsets, total, "u8",
                           rng.integers(0, 256, int(alens.sum()), dtype=np.uint8), aad_off)
    index = np.minimum(np.arange(n) % cycle, len(raw_keys) - 1).astype(np.uint32)
    keys = [pgcm.expand_key_bytes(k) for k in raw_keys]
    host = w.payload_host()
    expect = np.full(total, 0xEE, np.uint8)
    expect_tags = np.zeros((n, 16), np.uint8)
    for q, raw in enumerate(raw_keys):
        mine = np.flatnonzero(index == q)
        cts, tags, _ = oracle.encrypt_batch(
            raw, ivs[mine], [np.frombuffer(w.aad_of(i), np.uint8) for i in mine],
            [w.chunk(host, i) for i in mine], nthreads=16)
        expect_tags[mine] = tags
        for i, ct in zip(mine, cts):
            expect[int(offsets[i]):int(offsets[i]) + ct.size] = ct

    b = DeviceBatch(w, torch.from_numpy(host).cuda())
    b.cipher.fill_(0xEE)
    for _ in range(2):                   # twice: the arrival words must be left clean
        b.tags.zero_()
        pgcm.encrypt_batch_keys(keys, index, b.ivs, iv_bytes, b.aad_ptrs, b.aad_lens,
                                b.ptrs(b.plain), b.lens, b.ptrs(b.cipher), b.tags)
    torch.cuda.synchronize()
    bad = np.flatnonzero(b.cipher.cpu().numpy() != expect)
    assert bad.size == 0, "ciphertext byte %d" % bad[0]
    bad = np.flatnonzero((b.tags.cpu().numpy().reshape(n, 16) != expect_tags).any(1))
    assert bad.size == 0, "tag of chunk %d (length %d)" % (bad[0], lens[bad[0]])

    tampered = set(rng.integers(0, n, 2).tolist())
    for i in tampered:
        b.tags[16 * i + 5] ^= 0x10
    b.back.fill_(0xDD)
    pgcm.decrypt_verify_batch_keys(keys, index, b.ivs, iv_bytes, b.aad_ptrs, b.aad_lens,
                                   b.ptrs(b.cipher), b.lens, b.ptrs(b.back), b.tags, b.ok)
    torch.cuda.synchronize()
    assert np.array_equal(np.flatnonzero(b.ok.cpu().numpy() == 0), sorted(tampered))
    expect = np.full(total, 0xDD, np.uint8)
    for i in range(n):
        end = int(offsets[i] + lens[i])
        expect[int(offsets[i]):end] = 0 if i in tampered else host[int(offsets[i]):end]
    bad = np.flatnonzero(b.back.cpu().numpy() != expect)
    assert bad.size == 0, "plaintext byte %d" % bad[0]
    for k in keys:
        k.free()


def test_a_key_listed_twice_is_timed_once():
    w = workloads.mini(2)
    key = pgcm.expand_key(w.key)
    b = DeviceBatch(w, torch.from_numpy(w.payload_host()).cuda())
    index = (np.arange(w.n) % 2).astype(np.uint32)
    pgcm.set_timing(key, True)
    for calls in (1, 2, 3):
        pgcm.encrypt_batch_keys([key, key], index, b.ivs, 12, b.aad_ptrs, b.aad_lens,
                                b.ptrs(b.plain), b.lens, b.ptrs(b.cipher), b.tags)
        times = pgcm.bulk_kernel_ms_history(key)
        assert len(times) == calls and all(t > 0 for t in times), times
    tags = b.tags.clone()
    b.encrypt(key)
    torch.cuda.synchronize()
    assert torch.equal(tags, b.tags)
    key.free()


@pytest.mark.parametrize("key_bytes", (16, 24, 32))
def test_pieces_of_more_rows_than_a_segment(key_bytes):
    """Shares of some 140 rows, more than the second-round constants of a piece are formed for at once,
    with counters that wrap in the first chunk: against libcrypto, every byte."""
    rng = np.random.default_rng([workloads.BASE_SEED, 2718, key_bytes])
    raw = rng.integers(0, 256, key_bytes, dtype=np.uint8)
    h = openssl_ref.aes_ecb_block(raw.tobytes(), bytes(16))
    lens = np.array([300 * MIB + 7, 250 * MIB - 48, 9 * KIB], np.uint64)
    n = len(lens)
    wrap = (0xFFFFFFFF - 5_000_001).to_bytes(4, "big")
    ivs = np.stack([np.frombuffer(iv_craft.iv_for_j0(h, rng.bytes(12) + wrap), np.uint8),
                    *rng.integers(0, 256, (n - 1, 16), dtype=np.uint8)])
    offsets, total = workloads._layout(lens)
    aad_off = np.array([0, 20, 20, 60], np.uint64)
    w = workloads.Workload("long_pieces", 901, raw, ivs, lens, offsets, total, "u8",
                           rng.integers(0, 256, 60, dtype=np.uint8), aad_off)
    host = rng.integers(0, 256, total, dtype=np.uint8)
    key = pgcm.expand_key_bytes(raw)
    b = DeviceBatch(w, torch.from_numpy(host).cuda())
    b.encrypt(key)
    b.decrypt(key)
    torch.cuda.synchronize()
    cipher, tags = b.cipher.cpu().numpy(), b.tags.cpu().numpy().reshape(n, 16)
    for i in range(n):
        ref = openssl_ref.GcmEncryptStream(raw.tobytes(), ivs[i].tobytes(), w.aad_of(i))
        assert np.array_equal(ref.update(w.chunk(host, i)), w.chunk(cipher, i)), i
        assert ref.tag() == tags[i].tobytes(), i
    assert bool((b.ok == 1).all())
    assert torch.equal(b.back, b.plain)
    key.free()
