"""Calls of at most 64 chunks of up to 8 KiB, one of them longer than 256 blocks, on more streams than the key has
areas of slots for, from several threads, between replays of a graph and while another thread captures one: they
get no context and no memory, and their results are the CPU oracle's, bit for bit."""
import threading

import numpy as np
import pytest
import torch

import workloads
from device_batch import DeviceBatch
from test_gpu_bursts import _workload
from test_gpu_graphs import _Checked
from test_gpu_reservations import expected

import paper_2411_03357_amd as pgcm

pytestmark = pytest.mark.gpu

KIB, MIB = 1024, 1 << 20
# in two to nine workgroups a chunk, of 64 blocks or of 128
SHORT = [[8 * KIB], [8 * KIB] * 32, [4 * KIB] * 64, [1, 8191, 300, 4097, 8176]]
MANY = [1 + (97 * i * i) % 8192 for i in range(300)]


def _batches(rng, raw_key):
    return [_Checked("short_%d" % i, rng, lens, raw_key) for i, lens in enumerate(SHORT)]


def _rng_and_key(number):
    rng = np.random.default_rng([workloads.BASE_SEED, 6060, number])
    return rng, rng.integers(0, 256, 32, dtype=np.uint8)


def _no_context(key, stream):
    with pytest.raises(pgcm.PgcmError):
        pgcm.describe_context(key, stream)


def test_long_aad_captured_and_in_fixed_buffers():
    """a workgroup of sixteen wavefronts a chunk, whose AAD fills a row, or more"""
    w = _workload("captured_long_aad", [0, 5, 1024, 4096, 4097, 8192], [1008, 1024, 1025, 16, 3000])
    host = w.payload_host()
    cipher, tags = expected(w, host)
    b = DeviceBatch(w, torch.from_numpy(host).cuda())
    key = pgcm.expand_key(w.key)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()

    def check(what):
        torch.cuda.synchronize()
        assert np.array_equal(b.cipher.cpu().numpy(), cipher), what
        assert np.array_equal(b.tags.cpu().numpy().reshape(-1, 16), tags), what
        b.cipher.zero_()
        b.tags.zero_()
        torch.cuda.synchronize()

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        b.encrypt(key)
        b.decrypt(key)
    for r in range(3):
        b.back.zero_()
        b.ok.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        assert bool((b.ok == 1).all()) and torch.equal(b.back, b.plain), r
        check(r)
    pgcm.encrypt_batch_static(key, b.ivs, b.aad_ptrs, b.aad_lens, b.ptrs(b.plain), b.lens, b.ptrs(b.cipher), b.tags)
    check("static")
    # more chunks than compute units, that have several workgroups where no launch is needed to clear their slots
    rng, raw_key = _rng_and_key(5)
    m = _Checked("static_many", rng, MANY, raw_key)
    other = pgcm.expand_key(raw_key)
    for turn in range(2):
        pgcm.encrypt_batch_static(other, m.b.ivs, m.b.aad_ptrs, m.b.aad_lens, m.b.ptrs(m.b.plain), m.b.lens,
                                  m.b.ptrs(m.b.cipher), m.b.tags)
        m.b.decrypt(other)
        m.check(turn)
        m.clear()
    other.free()
    key.free()


def test_on_many_streams():
    rng, raw_key = _rng_and_key(1)
    key = pgcm.expand_key(raw_key)
    batches = _batches(rng, raw_key)
    streams = [None] + [torch.cuda.Stream() for _ in range(24)]
    for turn in range(2):
        for k, stream in enumerate(streams):
            for b in batches:
                b.clear()
            torch.cuda.synchronize()
            for b in batches:
                b.b.encrypt(key, stream=stream)
                b.b.decrypt(key, stream=stream)
            for b in batches:
                b.check((turn, k))
    for stream in streams:
        _no_context(key, stream)
    key.free()


def test_from_several_threads():
    """every thread on a stream of its own and, for every other batch, on one that all share"""
    rng, raw_key = _rng_and_key(2)
    key = pgcm.expand_key(raw_key)
    shared = torch.cuda.Stream()
    own = [(torch.cuda.Stream(), _batches(rng, raw_key)) for _ in range(4)]
    failed = []
    torch.cuda.synchronize()

    def work(stream, batches):
        try:
            torch.cuda.set_device(0)
            for _ in range(20):
                for k, b in enumerate(batches):
                    on = shared if k % 2 else stream
                    b.b.encrypt(key, stream=on)
                    b.b.decrypt(key, stream=on)
        except Exception as e:  # pylint: disable=broad-except
            failed.append(e)

    threads = [threading.Thread(target=work, args=a) for a in own]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
    for _, batches in own:
        for b in batches:
            b.check("threads")
    key.free()


def test_between_replays():
    rng, raw_key = _rng_and_key(3)
    key = pgcm.expand_key(raw_key)
    graphed = [_Checked("captured", rng, [2 * MIB, 300 * KIB + 1], raw_key),
               _Checked("captured_short", rng, [8 * KIB] * 20, raw_key)]
    many = _Checked("many", rng, MANY, raw_key)
    batches = _batches(rng, raw_key) + [many]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    pgcm.reserve(key, 300, 4 * MIB, stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for g in graphed:
            g.b.encrypt(key)
            g.b.decrypt(key)
    for r in range(4):
        for b in graphed + batches:
            b.clear()
        torch.cuda.synchronize()
        for b in batches:
            b.b.encrypt(key, stream=stream)
        with torch.cuda.stream(stream):
            graph.replay()
        for b in batches:
            b.b.decrypt(key, stream=stream)
        for b in graphed + batches:
            b.check(r)
    torch.cuda.synchronize()
    key.free()


def test_while_another_thread_captures():
    """the calls allocate nothing, so that a capture in the global mode, under which no thread may, goes on"""
    rng, raw_key = _rng_and_key(4)
    key = pgcm.expand_key(raw_key)
    graphed = _Checked("captured", rng, [2 * MIB, 300 * KIB + 1], raw_key)
    batches = _batches(rng, raw_key)
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    for b in batches:
        b.clear()
    pgcm.reserve(key, 2, 3 * MIB, stream)
    torch.cuda.synchronize()
    failed = []

    def work():
        try:
            torch.cuda.set_device(0)
            for b in batches:
                b.b.encrypt(key, stream=other)
                b.b.decrypt(key, stream=other)
        except Exception as e:  # pylint: disable=broad-except
            failed.append(e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="global"):
        graphed.b.encrypt(key)
        thread = threading.Thread(target=work)
        thread.start()
        thread.join()
        graphed.b.decrypt(key)
    assert not failed, failed
    for b in batches:
        b.check("while capturing")
    for r in range(2):
        graphed.clear()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        graphed.check(r)
    _no_context(key, other)
    torch.cuda.synchronize()
    key.free()
