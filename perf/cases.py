"""Performance cases of the multi-chain AES-256-GCM library, over its Python entry points.

A case is one call (or the call pair of the keystream-ahead path) on inputs of one layout. Every result is
bytes: plaintext, ciphertext, tags and accept flags, which GCM determines bit for bit, so every case is
compared exactly.

`op` names the entry point: decrypt and encrypt (uniform chains), eager (plaintext before its tag check, on two
streams), otp (the keystream generated ahead, then XOR and tag check), ragged-decrypt and ragged-encrypt
(variable-size samples, each cut into chains), h2d and d2h (the chunked pipelines over pinned host memory).
`len` is the payload in bytes (the ragged ops draw their sample sizes from the seed), `chain` the chain size,
`aad` the AAD bytes per chain. `keep` says whether the program passes output buffers that it keeps (a serving
loop) or lets the call allocate them.
"""
import math

import numpy as np
import torch

import paper_2410_15240_amd as F
import workloads as W

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30
CHUNK = 8 * MiB


def listed():
    return [
        # One decoded 224 x 224 RGB image as 16 chains with a 1-byte serial number: the smallest call that a
        # per-sample loader makes. Launches and latency.
        dict(name="decrypt-image-147KiB", op="decrypt", len=3 * 224 * 224, chain=9408, aad=1, keep=True),
        # 1 MiB in 64 KiB chains, the benchmark's small workload.
        dict(name="decrypt-1MiB", op="decrypt", len=MiB, chain=64 * KiB, aad=0, keep=True),
        # The benchmark's image batch at its shortest and its middle chain size, and the encrypting side.
        dict(name="decrypt-64MiB-4KiB", op="decrypt", len=64 * MiB, chain=4 * KiB, aad=32, keep=False),
        dict(name="decrypt-64MiB-64KiB", op="decrypt", len=64 * MiB, chain=64 * KiB, aad=32, keep=False),
        dict(name="encrypt-64MiB-16KiB", op="encrypt", len=64 * MiB, chain=16 * KiB, aad=32, keep=False),
        # Model weights at start-up and gradients leaving the GPU: the largest calls.
        dict(name="decrypt-weights-1GiB", op="decrypt", len=GiB, chain=MiB, aad=0, keep=True),
        dict(name="encrypt-gradients-256MiB", op="encrypt", len=256 * MiB, chain=256 * KiB, aad=0, keep=True),
        # A length and a chain size that divide nothing: partial blocks, a short last chain, an odd AAD.
        dict(name="decrypt-odd-40MB", op="decrypt", len=40000003, chain=10000, aad=13, keep=False),
        # Eager evaluation of the image batch: the plaintext is released before its tags are checked.
        dict(name="eager-64MiB-64KiB", op="eager", len=64 * MiB, chain=64 * KiB, aad=32, keep=False),
        # One pipeline chunk with its keystream generated ahead, then applied and checked.
        dict(name="otp-8MiB", op="otp", len=8 * MiB, chain=MiB, aad=0, keep=True),
        # A batch of 1024 compressed images of their own sizes, 16 chains each.
        dict(name="ragged-decrypt-1024", op="ragged-decrypt", len=1024 * 110 * KiB, samples=1024, per=16, aad=1,
             keep=False),
        # Host to device: pinned ciphertext copied in chunks and decrypted in place.
        dict(name="h2d-64MiB", op="h2d", len=64 * MiB, chain=MiB, aad=32, keep=True),
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    op = rng.choice(["decrypt"] * 5 + ["encrypt"] * 4 + ["eager", "otp", "ragged-decrypt", "ragged-decrypt",
                                                          "ragged-encrypt", "h2d", "d2h"])
    aad = rng.choice([0, 0, 1, 13, 32, 32])
    keep = rng.random() < 0.5
    if op.startswith("ragged"):
        n = _log(rng, 4, 1500)
        return dict(op=op, len=n * 110 * KiB, samples=n, per=rng.choice([4, 8, 16, 16]), aad=1, keep=keep)
    if op in ("h2d", "d2h"):
        chain = rng.choice([64 * KiB, 256 * KiB, MiB])
        return dict(op=op, len=_log(rng, 8 * MiB, 128 * MiB) + rng.choice([0, 5]), chain=chain, aad=aad, keep=True)
    n = _log(rng, 64 * KiB, 256 * MiB)
    chain = _log(rng, KiB, MiB) // 16 * 16
    if rng.random() < 0.5:   # powers of two are what most programs choose
        n, chain = 1 << (n.bit_length() - 1), 1 << (chain.bit_length() - 1)
    return dict(op=op, len=n, chain=min(chain, (n + 15) // 16 * 16), aad=aad, keep=keep)


def _payload(n, gen):
    # Incompressible bytes: what arrives is ciphertext, and the path does the same work for any plaintext.
    words = torch.randint(-(1 << 63), (1 << 63) - 1, ((n + 7) // 8,), dtype=torch.int64, device="cuda", generator=gen)
    return words.view(torch.uint8)[:n]


def _aad(n, a, length, chain):
    if a == 0:
        return None
    if a == 32:
        return torch.from_numpy(W.index_length_aad(length, chain)).cuda()
    full = (np.arange(n, dtype=np.uint64)[:, None] + 7 * np.arange(a, dtype=np.uint64)[None, :]) & np.uint64(255)
    return torch.from_numpy(full.astype(np.uint8)).cuda()


def _ragged_layout(case, rs):
    # Sample sizes of compressed images (log-normal), in a buffer that the program sized for any batch of that many.
    n = case["samples"]
    room = int(n * 132 * KiB + 500 * KiB * math.sqrt(n)) // 16 * 16
    lens = np.clip(np.round(110 * KiB * np.exp(0.6 * rs.standard_normal(n))), 4 * KiB, MiB)
    lens = np.floor(lens * min(1.0, 0.999 * room / lens.sum()))
    off, ln, total = F.sample_chains(lens.astype(np.uint64), case["per"])
    assert total <= room
    return off, ln, room


def prepare(case, seed):
    rs = np.random.RandomState(seed % (1 << 32))
    key, iv = rs.bytes(32), rs.bytes(12)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    op, a, chain = case["op"], case["aad"], case.get("chain", 0)
    s = dict(case, key=key, iv=iv, out=None, res=None)
    if op.startswith("ragged"):
        s["off"], s["ln"], room = _ragged_layout(case, rs)
        n = s["off"].size
        pt = _payload(room, gen)
        s["aad_t"] = torch.from_numpy(np.tile(np.arange(case["per"], dtype=np.uint8), case["samples"])).cuda().reshape(n, 1)
        if op == "ragged-decrypt":
            s["in"] = pt.clone()   # the gaps between samples hold what they held
            s["tags"] = F.encrypt_tag_ragged(key, iv, s["off"], s["ln"], pt, s["aad_t"], out=s["in"])[1]
            s["in"][int(s["off"][n // 2]) + 5] ^= 4   # one chain was tampered with
            # Bytes between chains stay as they were, so the program keeps a cleared buffer.
            s["out"] = torch.zeros_like(pt)
        else:
            s["in"], s["out"] = pt, torch.zeros_like(pt)
        if case["keep"]:
            s["res"] = torch.empty((n, 16) if op == "ragged-encrypt" else n, dtype=torch.uint8, device="cuda")
        return s
    length = case["len"]
    n = F.num_chains(length, chain)
    pt = _payload(length, gen)
    aad = s["aad_t"] = _aad(n, a, length, chain)
    if op == "encrypt":
        s["in"] = pt
        if case["keep"]:
            s["out"], s["res"] = torch.empty_like(pt), torch.empty((n, 16), dtype=torch.uint8, device="cuda")
        return s
    if op == "d2h":
        s["in"], s["out"] = pt, torch.empty_like(pt)
        s["res"] = torch.empty((n, 16), dtype=torch.uint8, device="cuda")
        s["h_ct"] = torch.empty(length, dtype=torch.uint8, pin_memory=True)
        s["h_tags"] = torch.empty((n, 16), dtype=torch.uint8, pin_memory=True)
        s["copy"], s["compute"] = torch.cuda.Stream(), torch.cuda.Stream()
        return s
    ct, tags = F.encrypt_tag(key, iv, chain, pt, aad)
    ct[(n // 2) * chain + 5] ^= 4   # one chain was tampered with
    s["in"], s["tags"] = ct, tags
    if op == "h2d":
        s["h_ct"], s["h_tags"] = ct.cpu().pin_memory(), tags.cpu().pin_memory()
        s["h_aad"] = None if aad is None else aad.cpu().pin_memory()
        s["out"] = torch.empty(length, dtype=torch.uint8, device="cuda")
        s["res"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        s["stage"] = torch.empty(max(F.stage_bytes(length, chain, a, CHUNK, 0), 1), dtype=torch.uint8, device="cuda")
        s["copy"], s["compute"] = torch.cuda.Stream(), torch.cuda.Stream()
        return s
    if op == "eager":
        s["check"] = torch.cuda.Stream()
    if op == "otp":
        s["ks"] = torch.empty(length, dtype=torch.uint8, device="cuda")
    if case["keep"]:
        s["out"], s["res"] = torch.empty_like(ct), torch.empty(n, dtype=torch.uint8, device="cuda")
    return s


def run(s):
    op = s["op"]
    if op == "decrypt":
        return F.decrypt_verify(s["key"], s["iv"], s["chain"], s["in"], s["tags"], s["aad_t"], out=s["out"], ok=s["res"])
    if op == "encrypt":
        return F.encrypt_tag(s["key"], s["iv"], s["chain"], s["in"], s["aad_t"], out=s["out"], tags=s["res"])
    if op == "eager":
        e = F.decrypt_eager(s["key"], s["iv"], s["chain"], s["in"], s["tags"], s["aad_t"], out=s["out"], ok=s["res"],
                            verify_stream=s["check"])
        return e.plaintext, e.ok
    if op == "otp":
        ks = F.keystream(s["key"], s["iv"], s["chain"], s["len"], out=s["ks"])
        return F.apply_verify(s["key"], s["iv"], s["chain"], s["in"], ks, s["tags"], s["aad_t"], out=s["out"], ok=s["res"])
    if op == "ragged-decrypt":
        return F.decrypt_verify_ragged(s["key"], s["iv"], s["off"], s["ln"], s["in"], s["tags"], s["aad_t"],
                                       out=s["out"], ok=s["res"])
    if op == "ragged-encrypt":
        return F.encrypt_tag_ragged(s["key"], s["iv"], s["off"], s["ln"], s["in"], s["aad_t"], out=s["out"],
                                    tags=s["res"])
    if op == "h2d":
        return F.pipeline_h2d(s["key"], s["iv"], s["chain"], s["h_ct"], s["h_tags"], s["h_aad"], chunk_bytes=CHUNK,
                              depth=0, stage=s["stage"], out=s["out"], ok=s["res"], copy_stream=s["copy"],
                              compute_stream=s["compute"])
    if op == "d2h":
        return F.pipeline_d2h(s["key"], s["iv"], s["chain"], s["in"], s["aad_t"], chunk_bytes=CHUNK, out=s["out"],
                              tags=s["res"], h_ct=s["h_ct"], h_tags=s["h_tags"], copy_stream=s["copy"],
                              compute_stream=s["compute"])
    raise ValueError(op)


def work(case):
    """Payload in and out, 16 bytes of tag, the AAD and (decrypting) one flag per chain. The arithmetic is table
    lookups and XORs on bytes, no floating-point operations."""
    n = case["samples"] * case["per"] if case["op"].startswith("ragged") else -(-case["len"] // case["chain"])
    b = 2 * case["len"] + n * (16 + case["aad"]) + (0 if "encrypt" in case["op"] or case["op"] == "d2h" else n)
    if case["op"] == "otp":
        b += 2 * case["len"]   # the keystream is written, then read
    return {"bytes": b, "flops": 0}


def tolerance(case):
    return "exact"
