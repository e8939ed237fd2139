"""The work a user of this library has it do, as cases that can be timed and compared.

The library encrypts, and decrypts with verification, what crosses the host-GPU boundary: swapped
KV-cache blocks, offloaded weight layers, adapters, and the small transfers in between.  A case is
one batch through the public calls, as a runtime makes them between two synchronisation points
(payload, IVs, tags and verdicts on the device, descriptor arrays on the host, all of them kept by
the runtime from call to call), or a short swap trace through the speculative pipe.

Fields of a case
  path        "batch": one key; "keys": a key per chunk; "pipe": the pipe and its receiver
  direction   "enc", "dec", or "both": encrypt, then decrypt and verify what came out
  chunks, lo, hi, ragged
              chunk lengths: log-uniform in [lo, hi], this share of them no multiple of 16 bytes,
              the others rounded down to one (equal chunks: lo == hi, ragged 0)
  mix         picks the lengths, so that every seed gives the same ones with other contents
  payload     "bytes" (uniform) or "half" (16-bit floats, normal: cache blocks and weights)
  key_bytes, iv_bytes, aad (longest AAD, 0 for none; "aad_fixed": every chunk has that much)
  bounce      ciphertext in pinned host memory instead of device memory
  tampered    share of the chunks with one bit flipped before decryption
"""
import numpy as np
import torch

import paper_2411_03357_amd as pgcm

KIB, MIB = 1 << 10, 1 << 20
ALIGN = 256          # chunks start at multiples of this in their packed buffer


def _batch(name=None, **fields):
    case = dict(path="batch", direction="enc", chunks=1, lo=1, hi=1, ragged=0.0, mix=0,
                payload="bytes", key_bytes=32, iv_bytes=12, aad=0, aad_fixed=False, bounce=False,
                tampered=0.0)
    case.update(fields)
    if name is not None:
        case["name"] = name
    return case


def listed():
    kv = 2 * 16 * 5120 * 2   # K and V of one 16-token block of one layer, 40 heads of 128, fp16
    return [
        # the smallest call there is: a 1-byte transfer that pads the IV sequence
        _batch("nop_enc"),
        # control traffic between swaps: short transfers of one size, out and back
        _batch("small_64x4KiB_both", direction="both", chunks=64, lo=4 * KIB, hi=4 * KIB),
        # control traffic of every size with headers, arriving
        _batch("small_ragged_dec", direction="dec", chunks=300, lo=1, hi=8 * KIB, ragged=0.7,
               aad=64),
        # one KV block swapped out on demand
        _batch("kv_block_enc", lo=kv, hi=kv, payload="half", aad=16, aad_fixed=True),
        # one piece of a weight layer swapped in
        _batch("layer_piece_dec", direction="dec", lo=2 * MIB, hi=2 * MIB, payload="half"),
        # a request's KV blocks swapped out straight into bounce buffers in host memory
        _batch("kv_bounce_enc", chunks=16, lo=kv, hi=kv, payload="half", aad=16, aad_fixed=True,
               bounce=True),
        # adapters of a few hundred odd sizes, with headers
        _batch("adapters_both", direction="both", chunks=300, lo=16 * KIB, hi=MIB, ragged=0.3,
               mix=1, aad=64),
        # the KV cache of many requests, out and back
        _batch("kv_cache_both", direction="both", chunks=4096, lo=kv, hi=kv, payload="half",
               aad=16, aad_fixed=True),
        # mixed traffic from short to long, a third of it ragged
        _batch("mixed_enc", chunks=2000, lo=16 * KIB, hi=8 * MIB, ragged=0.3, mix=2, aad=64),
        # a decoder layer of a large model swapped in, some pieces damaged on the way
        _batch("layer_dec", direction="dec", chunks=1728, lo=2 * MIB, hi=2 * MIB, payload="half",
               tampered=0.01),
        # tenants with keys of their own and of every length, and IVs that are not 96 bits long
        _batch("tenants_both", path="keys", direction="both", chunks=240, lo=4 * KIB, hi=2 * MIB,
               ragged=0.5, mix=3, iv_bytes=16, aad=32),
        # weights offloaded layer by layer in a loop: the pipe predicts, a receiver that counts
        # transfers decrypts
        {"name": "pipe_layers", "path": "pipe", "chunks": 8, "lo": 2 * MIB, "hi": 2 * MIB,
         "depth": 4},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    kind = rng.choice(("small", "few", "few", "some", "many", "many", "keys", "pipe"))
    if kind == "pipe":
        size = log_int(200 * KIB, 4 * MIB) // 16 * 16
        return {"path": "pipe", "chunks": rng.randint(5, 16), "lo": size, "hi": size, "depth": 4}
    case = _batch(direction=rng.choice(("enc", "dec", "both")), mix=rng.randrange(1, 1 << 30),
                  ragged=rng.choice((0.0, 0.3, 0.7)), aad=rng.choice((0, 16, 64)),
                  payload=rng.choice(("bytes", "half")),
                  key_bytes=rng.choice((16, 24, 32, 32, 32, 32)))
    if kind == "small":
        case.update(chunks=log_int(1, 512), lo=1, hi=log_int(16, 8 * KIB))
    elif kind == "few":
        lo = log_int(9 * KIB, 4 * MIB)
        case.update(chunks=log_int(1, 24), lo=lo, hi=min(8 * MIB, log_int(lo, 4 * lo)),
                    bounce=rng.random() < 0.2)
    elif kind == "some":
        lo = log_int(KIB, 128 * KIB)
        case.update(chunks=log_int(25, 600), lo=lo, hi=log_int(2 * lo, 16 * lo))
    elif kind == "many":
        # 0.1 to 1.3 GB in pieces of 16 KiB to 4 MiB
        total, size = log_int(100 * MIB, 1250 * MIB), log_int(16 * KIB, 4 * MIB)
        case.update(chunks=max(32, min(20000, total // size)), lo=size,
                    hi=size if rng.random() < 0.5 else size + size // 3)
    else:
        case.update(path="keys", chunks=log_int(6, 600), lo=log_int(KIB, 16 * KIB),
                    hi=log_int(64 * KIB, 2 * MIB), iv_bytes=rng.choice((12, 16)),
                    key_bytes=32)
    if case["path"] == "batch" and rng.random() < 0.15:
        case["iv_bytes"] = rng.choice((8, 16))
    if case["direction"] == "dec" and rng.random() < 0.3:
        case["tampered"] = 0.02
    return case


def _lengths(case):
    """the chunks' lengths and AAD lengths: functions of the case alone"""
    n, lo, hi = case["chunks"], case["lo"], case["hi"]
    rng = np.random.default_rng([31, case.get("mix", 0), n, lo, hi])
    lens = np.floor(np.exp(rng.uniform(np.log(lo), np.log(hi + 1), n))).astype(np.int64)
    lens = np.clip(lens, lo, hi)
    even = rng.random(n) >= case.get("ragged", 0.0)
    lens = np.where(even & (lens >= 16), lens // 16 * 16, lens)
    lens = np.where(~even & (lens % 16 == 0), lens - 1, lens)
    aad = case.get("aad", 0)
    alens = np.full(n, aad) if case.get("aad_fixed") else rng.integers(0, aad + 1, n)
    return np.maximum(lens, 1).astype(np.uint64), alens.astype(np.uint32)


def _layout(lens):
    padded = (lens.astype(np.int64) + ALIGN - 1) // ALIGN * ALIGN
    offsets = np.zeros(lens.size, np.uint64)
    offsets[1:] = np.cumsum(padded)[:-1]
    return offsets, int(padded.sum())


def _payload(kind, nbytes, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if kind == "half":
        return torch.empty((nbytes + 1) // 2, dtype=torch.float16, device="cuda").normal_(
            0.0, 1.0, generator=gen).view(torch.uint8)[:nbytes]
    words = torch.randint(-(1 << 62), 1 << 62, ((nbytes + 7) // 8,), dtype=torch.int64,
                          device="cuda", generator=gen)
    return words.view(torch.uint8)[:nbytes]


class _Batch:
    """buffers and descriptor arrays of one batch"""

    def __init__(self, case, seed):
        rng = np.random.default_rng([seed, 17])
        n = case["chunks"]
        self.direction = case["direction"]
        self.lens, self.aad_lens = _lengths(case)
        offsets, total = _layout(self.lens)
        # a counter for 96-bit IVs, as the transport keeps one; other lengths are random
        if case["iv_bytes"] == 12:
            start = int.from_bytes(rng.bytes(12), "big")
            iv = b"".join(((start + i) % (1 << 96)).to_bytes(12, "big") for i in range(n))
            iv = np.frombuffer(iv, np.uint8)
        else:
            iv = rng.integers(0, 256, n * case["iv_bytes"], dtype=np.uint8)
        self.ivs = torch.from_numpy(iv.copy()).cuda()
        self.plain = _payload(case["payload"], total, seed * 1000003 + 7)
        bounce = case["bounce"]
        self.cipher = torch.zeros(total, dtype=torch.uint8, device="cpu" if bounce else "cuda",
                                  pin_memory=bounce)
        self.tags = torch.zeros(16 * n, dtype=torch.uint8, device="cuda")
        self.back = self.ok = None
        if self.direction != "enc":
            self.back = torch.zeros(total, dtype=torch.uint8, device="cuda")
            self.ok = torch.zeros(n, dtype=torch.uint8, device="cuda")
        self.aad = self.aad_ptrs = None
        if case["aad"]:
            aad = rng.integers(0, 256, int(self.aad_lens.sum()) + 1, dtype=np.uint8)
            self.aad = torch.from_numpy(aad).cuda()
            starts = np.zeros(n, np.uint64)
            starts[1:] = np.cumsum(self.aad_lens)[:-1]
            self.aad_ptrs = np.uint64(self.aad.data_ptr()) + starts
        else:
            self.aad_lens = None
        self.plain_ptrs = np.uint64(self.plain.data_ptr()) + offsets
        self.cipher_ptrs = np.uint64(self.cipher.data_ptr()) + offsets
        if self.back is not None:
            self.back_ptrs = np.uint64(self.back.data_ptr()) + offsets
        self.iv_bytes = case["iv_bytes"]
        if case["path"] == "keys":
            # three tenants with keys of 16, 24 and 32 bytes
            self.keys = [pgcm.expand_key_bytes(rng.bytes(b)) for b in (16, 24, 32)]
            self.key_index = rng.integers(0, 3, n).astype(np.uint32)
        else:
            self.keys = None
            self.key = pgcm.expand_key_bytes(rng.bytes(case["key_bytes"]))
        if self.direction == "dec":
            # what the peer sent, some of it damaged on the way
            self.encrypt()
            torch.cuda.synchronize()
            for i in rng.permutation(n)[:int(round(case["tampered"] * n))]:
                if rng.random() < 0.5:
                    at = int(offsets[i]) + int(rng.integers(0, int(self.lens[i])))
                    self.cipher[at] ^= 1 << int(rng.integers(0, 8))
                else:
                    self.tags[16 * int(i) + int(rng.integers(0, 16))] ^= 1

    def encrypt(self):
        if self.keys is not None:
            pgcm.encrypt_batch_keys(self.keys, self.key_index, self.ivs, self.iv_bytes,
                                    self.aad_ptrs, self.aad_lens, self.plain_ptrs, self.lens,
                                    self.cipher_ptrs, self.tags)
        elif self.iv_bytes != 12:
            pgcm.encrypt_batch(self.key, self.ivs, self.aad_ptrs, self.aad_lens, self.plain_ptrs,
                               self.lens, self.cipher_ptrs, self.tags, iv_bytes=self.iv_bytes)
        else:
            pgcm.encrypt_batch(self.key, self.ivs, self.aad_ptrs, self.aad_lens, self.plain_ptrs,
                               self.lens, self.cipher_ptrs, self.tags)

    def decrypt(self):
        if self.keys is not None:
            pgcm.decrypt_verify_batch_keys(self.keys, self.key_index, self.ivs, self.iv_bytes,
                                           self.aad_ptrs, self.aad_lens, self.cipher_ptrs,
                                           self.lens, self.back_ptrs, self.tags, self.ok)
        elif self.iv_bytes != 12:
            pgcm.decrypt_verify_batch(self.key, self.ivs, self.aad_ptrs, self.aad_lens,
                                      self.cipher_ptrs, self.lens, self.back_ptrs, self.tags,
                                      self.ok, iv_bytes=self.iv_bytes)
        else:
            pgcm.decrypt_verify_batch(self.key, self.ivs, self.aad_ptrs, self.aad_lens,
                                      self.cipher_ptrs, self.lens, self.back_ptrs, self.tags,
                                      self.ok)

    def run(self):
        out = {}
        if self.direction != "dec":
            self.encrypt()
            out["cipher"], out["tags"] = self.cipher, self.tags
        if self.direction != "enc":
            self.decrypt()
            out["back"], out["ok"] = self.back, self.ok
        return out


class _Pipe:
    """layers swapped out in the same order over and over: the pipe encrypts ahead of demand, the
    peer on the other end of the wire decrypts every transfer as it comes"""

    def __init__(self, case, seed):
        rng = np.random.default_rng([seed, 19])
        n, size = case["chunks"], case["lo"]
        self.size, self.n = size, n
        stride = (size + ALIGN - 1) // ALIGN * ALIGN
        self.plain = _payload("half", n * stride, seed * 1000003 + 11)
        self.addrs = [self.plain.data_ptr() + i * stride for i in range(n)]
        self.back = torch.zeros(n * stride, dtype=torch.uint8, device="cuda")
        self.slots = [self.back[i * stride:i * stride + size] for i in range(n)]
        self.nop_byte = torch.zeros(16, dtype=torch.uint8, device="cuda")
        self.ok = torch.zeros(n, dtype=torch.uint8, device="cuda")
        self.oks = [self.ok[i:i + 1] for i in range(n)]
        self.nop_ok = torch.zeros(1, dtype=torch.uint8, device="cuda")
        self.place = {a: i for i, a in enumerate(self.addrs)}
        self.key = pgcm.expand_key(rng.bytes(32))
        iv0 = rng.bytes(12)
        self.receiver = pgcm.Receiver(self.key, iv0)
        self.pipe = pgcm.Pipe(self.key, iv0, self.deliver, depth=case["depth"],
                              max_chunk_bytes=size)

    def deliver(self, kind, addr, length, iv, ciphertext, tag, stream):
        if kind == "nop":
            self.receiver.accept(ciphertext, length, tag, self.nop_byte, self.nop_ok, stream)
            return
        i = self.place[addr]
        self.receiver.accept(ciphertext, length, tag, self.slots[i], self.oks[i], stream)

    def run(self):
        for i in range(0, self.n, 2):        # a synchronisation point after every two layers
            for addr in self.addrs[i:i + 2]:
                self.pipe.request(addr, self.size)
            self.pipe.sync()
        return {"back": self.back, "ok": self.ok}


def prepare(case, seed):
    return _Pipe(case, seed) if case["path"] == "pipe" else _Batch(case, seed)


def run(state):
    return state.run()


def work(case):
    """Each payload byte is read once and written once per direction.  The cipher's work is not
    floating-point: flops stays 0."""
    lens, alens = _lengths(case)
    n, payload = case["chunks"], int(lens.sum())
    if case["path"] == "pipe":
        return {"bytes": 2 * (2 * payload + n * (12 + 16)) + n, "flops": 0}
    once = 2 * payload + n * (case["iv_bytes"] + 16) + (int(alens.sum()) if case["aad"] else 0)
    passes = 2 if case["direction"] == "both" else 1
    return {"bytes": passes * once + (0 if case["direction"] == "enc" else n), "flops": 0}


def tolerance(case):
    """AES-GCM is exact: ciphertext, tags, plaintext and verdicts are the same bytes everywhere."""
    return "exact"
