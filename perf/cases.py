"""Workloads of the 3DES library that stand for its everyday use.

Every case goes through the public Python entry points (tdes.py, serve.py)
as a program would: device buffers and streams from torch, keys as 24-byte
bundles or as schedules a program keeps, descriptors and device schedules of
a batch laid out once.  Payloads are uniform random bytes (ciphertext, media,
compressed files), keys uniform with odd parity.  Sizes are whole 8-byte
blocks; most of them are no round number, as message lengths are in use.

Outputs are bytes, compared exactly.
"""
import math

import numpy as np
import torch

from paper_2007_10752_amd import serve, tdes
from paper_2007_10752_amd import workloads as W

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30

# 32-bit operations of the bitsliced cipher per 8-byte block: 48 rounds of
# about 240 three-input operations and four 32 x 32 bit transposes, on 32
# blocks at once.
OPS_PER_BLOCK = 395.0


def listed():
    return [
        # One database field or token: a program that holds its session's
        # schedule decrypts it into a buffer it owns.  Latency only.
        {"name": "ecb token 1000 B", "path": "ecb", "nbytes": 1000, "decrypt": True,
         "two_key": False, "offset": 0, "keep": True},
        # The paper's smallest GPU sizes (4,096 blocks), called the short way:
        # key bytes in, a new tensor out.
        {"name": "ecb 32 KiB", "path": "ecb", "nbytes": 32 * KiB, "decrypt": False,
         "two_key": False, "offset": 0, "keep": False},
        # A media segment or a large network buffer in counter mode.
        {"name": "ctr segment 64 KB", "path": "ctr", "nbytes": 65528, "offset": 0, "keep": True},
        # A stored file in CBC, decrypted whole.
        {"name": "cbc file 1 MB", "path": "cbc", "nbytes": 1_000_008, "two_key": False,
         "offset": 0, "keep": True},
        # A file somewhat larger than what the smallest launches are good at,
        # at an 8-byte aligned place inside a buffer.
        {"name": "ecb file 12 MB", "path": "ecb", "nbytes": 12_000_008, "decrypt": False,
         "two_key": False, "offset": 8, "keep": True},
        # 64 MiB with a two-key bundle, decrypted (one of the library's own
        # benchmark sizes).
        {"name": "ecb 64 MiB two-key", "path": "ecb", "nbytes": 64 * MiB, "decrypt": True,
         "two_key": True, "offset": 0, "keep": False},
        # A disk image's worth in counter mode, ragged.
        {"name": "ctr image 256 MB", "path": "ctr", "nbytes": 256_000_024, "offset": 0,
         "keep": True},
        # The headline: 1 GiB resident in HBM.
        {"name": "ecb 1 GiB", "path": "ecb", "nbytes": GiB, "decrypt": False, "two_key": False,
         "offset": 0, "keep": False},
        # 16,384 messages, log-normal around 4 KiB, each with its own key and
        # direction, schedules on the device already.
        {"name": "batch 16384 messages", "path": "batch", "n_msgs": 16384, "median": 4096,
         "sigma": 1.0, "from_keys": False},
        # A small batch straight from raw keys: expansion on the device, then
        # one submit.
        {"name": "batch 300 messages from keys", "path": "batch", "n_msgs": 300, "median": 4096,
         "sigma": 1.0, "from_keys": True},
        # Pinned host memory in and out, PCIe included.
        {"name": "host pinned 16 MB", "path": "host", "nbytes": 16_000_000, "decrypt": False,
         "staged": False},
        # A burst of requests of the server's standard mix, until the last one
        # is done.
        {"name": "serve burst 400", "path": "serve", "n_reqs": 400, "max_bytes": 16 * MiB},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _blocks(rng, lo, hi):
    """Bytes in whole blocks, log-uniform."""
    return max(1, round(_log(rng, lo, hi) / 8)) * 8


def draw(rng):
    path = rng.choice(("ecb", "ecb", "ecb", "ctr", "cbc", "batch", "batch", "host", "serve"))
    if path == "ecb":
        return {"path": path, "nbytes": _blocks(rng, 8, 512 * MiB),
                "decrypt": rng.random() < 0.5, "two_key": rng.random() < 0.25,
                "offset": rng.choice((0, 0, 0, 8)), "keep": rng.random() < 0.5}
    if path == "ctr":
        return {"path": path, "nbytes": _blocks(rng, 8, 512 * MiB),
                "offset": rng.choice((0, 0, 0, 8)), "keep": rng.random() < 0.5}
    if path == "cbc":
        return {"path": path, "nbytes": _blocks(rng, 8, 512 * MiB),
                "two_key": rng.random() < 0.25, "offset": rng.choice((0, 0, 0, 8)),
                "keep": rng.random() < 0.5}
    if path == "batch":
        n = round(_log(rng, 4, 20000))
        return {"path": path, "n_msgs": n, "median": round(_log(rng, 64, 16384)),
                "sigma": rng.choice((0.0, 0.5, 1.0)), "from_keys": rng.random() < 0.5}
    if path == "host":
        return {"path": path, "nbytes": _blocks(rng, 4 * KiB, 64 * MiB),
                "decrypt": rng.random() < 0.5, "staged": rng.random() < 0.4}
    return {"path": path, "n_reqs": round(_log(rng, 1, 1200)),
            "max_bytes": round(_log(rng, 8 * KiB, 16 * MiB))}


def _lengths(case, seed):
    """A batch's or a burst's message lengths.  They depend on the case
    alone (the seed draws payloads and keys), so that passes over inputs of
    different seeds do the same amount of work."""
    if case["path"] == "batch":
        return W.batched_layout(7 + case["n_msgs"], n_msgs=case["n_msgs"], median=case["median"],
                                sigma=case["sigma"])["lengths"]
    n = case["n_reqs"]
    g = W.rng(11 + n)
    # the server's standard size bands, each cut off at the case's largest
    probs = np.array([b[0] for b in W.SIZE_BANDS])
    band = g.choice(len(W.SIZE_BANDS), size=n, p=probs / probs.sum())
    lo = np.minimum([b[1] for b in W.SIZE_BANDS], case["max_bytes"] // 2)[band]
    hi = np.minimum([b[2] for b in W.SIZE_BANDS], case["max_bytes"])[band]
    size = np.exp(np.log(lo) + g.random(n) * (np.log(hi) - np.log(lo)))
    return (np.ceil(size / 8) * 8).astype(np.int64)


def _random(nbytes, seed, offset=0):
    """Uniform random bytes on the GPU, `offset` bytes into their buffer."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    words = torch.randint(-2 ** 63, 2 ** 63 - 1, ((nbytes + offset) // 8,), dtype=torch.int64,
                          device="cuda", generator=g)
    return words.view(torch.uint8)[offset:]


def prepare(case, seed):
    path = case["path"]
    gen = W.rng(W.SEED_BASE + seed)
    if path in ("ecb", "ctr", "cbc"):
        key = bytes(W.key_bundle(gen, two_key=case.get("two_key", False)))
        off = case["offset"]
        s = {"path": path, "key": key, "x": _random(case["nbytes"], seed, off), "out": None,
             "iv": bytes(W.uniform_bytes(gen, 8)), "decrypt": case.get("decrypt", False)}
        if case["keep"]:  # a program that keeps its schedule and its output buffer
            s["key"] = tdes.key_schedule(key)
            s["out"] = torch.zeros(case["nbytes"] + off, dtype=torch.uint8, device="cuda")[off:]
        return s
    if path == "host":
        h = torch.empty(case["nbytes"], dtype=torch.uint8, pin_memory=not case["staged"])
        h.copy_(_random(case["nbytes"], seed))
        s = {"path": path, "key": tdes.key_schedule(W.key_bundle(gen)), "in": h,
             "out": torch.zeros(case["nbytes"], dtype=torch.uint8,
                                pin_memory=not case["staged"]),
             "decrypt": case["decrypt"], "pipe": None}
        if case["staged"]:
            s["pipe"] = tdes.HostPipeline()
        return s
    lengths = _lengths(case, seed)
    n, total = len(lengths), int(lengths.sum())
    keys = W.key_bundles(gen, n)
    dirs = gen.integers(0, 2, size=n).astype(np.uint32)
    starts = np.concatenate([[0], np.cumsum(lengths)[:-1]]).astype(np.int64)
    if path == "batch":
        s = {"path": path, "x": _random(total, seed),
             "out": torch.zeros(total, dtype=torch.uint8, device="cuda"),
             "batch": tdes.Batch(keys, starts, starts, lengths, dirs), "keys": None}
        if case["from_keys"]:
            s["keys"] = torch.from_numpy(keys).to("cuda")
        torch.cuda.synchronize()
        return s
    room = (lengths + 255) // 256 * 256  # the server's results start at multiples of 256
    arena = torch.zeros(int(room.sum()) + MiB, dtype=torch.uint8, device="cuda")
    pool = _random(total, seed)
    reqs = np.zeros(n, dtype=serve.REQUEST)
    reqs["key24"], reqs["dir"], reqs["nbytes"] = keys, dirs, lengths
    reqs["d_in"] = np.uint64(pool.data_ptr()) + starts.astype(np.uint64)
    reqs["tag"] = np.arange(n, dtype=np.uint64)
    torch.cuda.synchronize()  # the server's streams don't wait for torch's
    return {"path": path, "pool": pool, "arena": arena, "reqs": reqs, "used": int(room.sum()),
            "server": serve.Server(arena.data_ptr(), arena.numel(),
                                   budget_bytes=4 * arena.numel()), "live": None}


def run(s):
    path = s["path"]
    if path == "ecb":
        return tdes.ecb(s["key"], s["x"], s["out"], decrypt=s["decrypt"])
    if path == "ctr":
        return tdes.ctr(s["key"], s["iv"], s["x"], s["out"])
    if path == "cbc":
        return tdes.cbc_decrypt(s["key"], s["iv"], s["x"], s["out"])
    if path == "host":
        if s["pipe"] is not None:
            return s["pipe"].run(s["key"], s["in"], s["out"], decrypt=s["decrypt"])
        return tdes.ecb_host(s["key"], s["in"], s["out"], decrypt=s["decrypt"])
    if path == "batch":
        b = s["batch"]
        if s["keys"] is not None:
            tdes.schedule_expand(s["keys"].data_ptr(), b.n_sched, b.sched.data_ptr(), b.stream)
        return b.submit(s["x"], s["out"])
    # serve: give the last burst's results back, submit this one, wait for it
    server = s["server"]
    if s["live"] is not None:
        server.release_many(s["live"])
    server.submit(s["reqs"])
    got, left = [], len(s["reqs"])
    while left:
        c = server.progress()
        if len(c):
            if c["status"].any():
                raise RuntimeError("a request failed")
            got.append(c["d_out"])
            left -= len(c)
    s["live"] = np.concatenate(got)
    return s["arena"][: s["used"]]


def work(case):
    nbytes = case["nbytes"] if "nbytes" in case else int(_lengths(case, 0).sum())
    keys = 0
    if case["path"] in ("batch", "serve"):
        n = case["n_msgs"] if case["path"] == "batch" else case["n_reqs"]
        # a descriptor and the key material of its direction, or the raw key
        keys = n * (32 + (24 if case.get("from_keys", True) else 400))
    return {"bytes": 2.0 * nbytes + keys, "flops": OPS_PER_BLOCK * nbytes / 8}
