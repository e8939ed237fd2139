"""pgcm_reserve: after it, batches within the reserved sizes get no memory of any kind, whichever way
they go (one launch, spans read from host memory or uploaded, a wavefront per chunk), and their
results are the CPU oracle's, bit for bit; batches under several keys, each reserved for its share, and
what they leave in a workspace."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from device_batch import DeviceBatch

import paper_2411_03357_amd as pgcm

pytestmark = pytest.mark.gpu

KIB, MIB = 1024, 1 << 20

# chunk lengths
SHAPES = {
    "one_launch": lambda r: [2 * MIB] * 3,
    "spans_few": lambda r: [int(v) for v in r.integers(200 * KIB, 450 * KIB, 60)],
    "spans_host": lambda r: [int(v) for v in r.integers(30 * KIB, 90 * KIB, 700)],
    "spans_uploaded": lambda r: [int(v) for v in r.integers(1, 3 * KIB, 9000)],
    "one_row": lambda r: [int(v) for v in r.integers(0, 1009, 2000)],
}


def workload(name, rng, lens, key, ivs):
    lens = np.array(lens, np.uint64)
    alens = rng.integers(0, 40, lens.size)
    aad_off = np.zeros(lens.size + 1, np.uint64)
    aad_off[1:] = np.cumsum(alens)
    offsets, total = workloads._layout(lens)
    return workloads.Workload(name, 950, key, ivs, lens, offsets, total, "u8",
                              rng.integers(0, 256, int(alens.sum()), dtype=np.uint8), aad_off)


def expected(w, host):
    """whole ciphertext buffer (zero between chunks) and tags by the oracle"""
    cts, tags, _ = oracle.encrypt_batch(w.key, w.ivs,
                                        [np.frombuffer(w.aad_of(i), np.uint8) for i in range(w.n)],
                                        [w.chunk(host, i) for i in range(w.n)], nthreads=16)
    out = np.zeros(w.total_bytes, np.uint8)
    for i, ct in enumerate(cts):
        out[int(w.offsets[i]):int(w.offsets[i]) + ct.size] = ct
    return out, tags


@pytest.mark.parametrize("shape", SHAPES)
def test_reserved_batches_allocate_nothing(shape):
    rng = np.random.default_rng([workloads.BASE_SEED, 8128, len(shape)])
    lens = SHAPES[shape](rng)
    w = workload("reserved_" + shape, rng, lens, rng.integers(0, 256, 32, dtype=np.uint8),
                 rng.integers(0, 256, (len(lens), 12), dtype=np.uint8))
    host = w.payload_host()
    cipher, tags = expected(w, host)
    key = pgcm.expand_key(w.key)
    b = DeviceBatch(w, torch.from_numpy(host).cuda())
    stream = torch.cuda.Stream()
    with pytest.raises(pgcm.PgcmError):
        pgcm.describe_context(key, stream)             # nothing has used the stream
    pgcm.reserve(key, w.n, w.payload_bytes, stream)
    reserved = pgcm.describe_context(key, stream)
    torch.cuda.synchronize()
    for _ in range(6):                                 # more than there are staging buffers
        b.encrypt(key, stream=stream)
        b.decrypt(key, stream=stream)
    after = pgcm.describe_context(key, stream)
    torch.cuda.synchronize()
    for field in ("allocations", "workspace_bytes", "stage_bytes"):
        assert after[field] == reserved[field], field
    assert np.array_equal(b.cipher.cpu().numpy(), cipher)
    assert np.array_equal(b.tags.cpu().numpy().reshape(-1, 16), tags)
    assert bool((b.ok == 1).all()) and torch.equal(b.back, b.plain)
    key.free()


def _keys_batch(rng, lens, key_bytes):
    """chunks of several keys in turn: the device batch, the keys, whose chunk is whose, and the
    oracle's ciphertext buffer and tags"""
    n = len(lens)
    raw = [rng.integers(0, 256, k, dtype=np.uint8) for k in key_bytes]
    ivs = rng.integers(0, 256, (n, 12), dtype=np.uint8)
    index = (np.arange(n) % len(raw)).astype(np.uint32)
    w = workload("reserved_keys", rng, lens, raw[0], ivs)
    host = w.payload_host()
    cipher, tags = np.zeros(w.total_bytes, np.uint8), np.zeros((n, 16), np.uint8)
    for q, k in enumerate(raw):
        mine = np.flatnonzero(index == q)
        cts, tags[mine], _ = oracle.encrypt_batch(
            k, ivs[mine], [np.frombuffer(w.aad_of(i), np.uint8) for i in mine],
            [w.chunk(host, i) for i in mine], nthreads=16)
        for i, ct in zip(mine, cts):
            cipher[int(w.offsets[i]):int(w.offsets[i]) + ct.size] = ct
    b = DeviceBatch(w, torch.from_numpy(host).cuda())
    return b, [pgcm.expand_key_bytes(k) for k in raw], index, cipher, tags


def _encrypt_keys(b, keys, index, stream=None):
    pgcm.encrypt_batch_keys(keys, index, b.ivs, 12, b.aad_ptrs, b.aad_lens, b.ptrs(b.plain),
                            b.lens, b.ptrs(b.cipher), b.tags, stream)


# chunk lengths of batches under several keys: all in one launch; more chunks than share one (in
# several launches of some keys each); one key's too many for a launch with others
KEYS_SHAPES = {
    "one_launch": (lambda r: [int(v) for v in r.integers(4 * KIB, 500 * KIB, 120)], (16, 24, 32)),
    "launches": (lambda r: [int(v) for v in r.integers(1, 5 * KIB, 5600)], (32, 16) * 4),
    "apart": (lambda r: [int(v) for v in r.integers(1, 3 * KIB, 8100)], (32, 24)),
}


@pytest.mark.parametrize("shape", KEYS_SHAPES)
def test_every_key_reserved_for_its_share(shape):
    rng = np.random.default_rng([workloads.BASE_SEED, 8129, len(shape)])
    lens, key_bytes = KEYS_SHAPES[shape]
    b, keys, index, cipher, tags = _keys_batch(rng, lens(rng), key_bytes)
    stream = torch.cuda.Stream()
    for q, key in enumerate(keys):
        mine = np.flatnonzero(index == q)
        pgcm.reserve(key, mine.size, int(b.lens[mine].sum()), stream)
    reserved = [pgcm.describe_context(key, stream) for key in keys]
    torch.cuda.synchronize()
    for _ in range(6):
        _encrypt_keys(b, keys, index, stream)
    after = [pgcm.describe_context(key, stream) for key in keys]
    torch.cuda.synchronize()
    for r, a in zip(reserved, after):
        assert a["allocations"] == r["allocations"]
    assert np.array_equal(b.cipher.cpu().numpy(), cipher)
    assert np.array_equal(b.tags.cpu().numpy().reshape(-1, 16), tags)
    for key in keys:
        key.free()


def test_no_keys_partial_hashes_stay_in_anothers_workspace():
    rng = np.random.default_rng([workloads.BASE_SEED, 8130])
    # every chunk in several workgroups, so that partial hashes go through the workspace
    b, keys, index, cipher, tags = _keys_batch(rng, [2 * MIB + 5] * 12, (32, 16))
    _encrypt_keys(b, keys, index)
    groups = torch.cuda.get_device_properties(0).multi_processor_count
    # a slot of 64 bytes for every part, and every workgroup has one at least
    work = pgcm.describe_context(keys[0], None, 64 * groups)["workspace"]
    assert not work.any()
    keys[1].free()
    assert np.array_equal(b.cipher.cpu().numpy(), cipher)
    assert np.array_equal(b.tags.cpu().numpy().reshape(-1, 16), tags)
    keys[0].free()
