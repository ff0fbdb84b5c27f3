"""GPU parity where the work plan takes chains apart in its different ways.

Each layout pins one way the planner lays a launch out on a 256-CU GPU: 16, 32 or
64 lanes per item; whole chains or segments with a segment 0 shorter than the rest
(which runs only the iterations its blocks need); one pass of wave-items, or
several with a last one that leaves waves idle (their numbering spreads it over
the CUs). The results are compared bit for bit with the CPU oracle: plaintext and
flags with one tampered chain, ciphertext and tags, and the two modes that check
tags without AES. The plan pinned beside a layout is that of decrypt + verify and
encrypt + tag; the other modes weigh their costs differently (test_hostrt.py checks
that the layouts together take every mode through 16, 32 and 64 lanes, whole chains
and segments)."""
import ctypes

import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

# length, chain bytes, AAD bytes, (lanes_log2, split, more than one pass)
LAYOUTS = [
    (16181855, 21728, 13, (4, 1, 0)),
    (19440397, 2320, 1, (4, 1, 1)),
    (13447333, 8208, 32, (5, 1, 0)),
    (31839236, 18448, 0, (5, 1, 1)),
    (15317645, 33664, 0, (6, 1, 0)),
    (31792379, 17456, 13, (6, 1, 1)),
    (12876048, 784, 0, (5, 0, 1)),
    (35867559, 3888, 32, (6, 0, 1)),
    (14959, 7248, 5, (6, 1, 0)),
    (440001, 60016, 5, (6, 1, 0)),
    (2999999, 10000, 7, (6, 1, 0)),
    (263735, 16, 0, (4, 0, 1)),
    (12819, 48, 5, (6, 0, 0)),
    (3794, 16, 0, (6, 0, 0)),
    (27803887, 6784, 1, (4, 1, 1)),
    (31764477, 1856, 13, (5, 0, 1)),
]


@pytest.fixture(scope="module")
def F():
    import paper_2410_15240_amd as F
    F.lib()
    return F


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("length,chain,abytes,want", LAYOUTS)
def test_layout_matches_the_oracle(F, length, chain, abytes, want):
    out = (ctypes.c_uint64 * 7)()
    assert F.lib().fastrack_plan(ctypes.c_uint64(length), ctypes.c_uint64(chain), ctypes.c_uint32(256), out) == 0
    wave_items = -(-int(out[4]) // (64 >> int(out[0])))
    assert (int(out[0]), int(out[6]), int(wave_items > 4096)) == want, list(out)
    w = W.random_case(length % 1000, length, chain, aad_bytes=abytes)
    aad = W.case_aad(w, chain) if abytes else None
    d_aad = dev(aad) if abytes else None
    ct, tags = oracle.chains_encrypt(w.key, w.base_iv, chain, w.payload, aad, abytes)
    got_ct, got_tags = F.encrypt_tag(w.key, w.base_iv, chain, dev(w.payload), d_aad)
    assert np.array_equal(host(got_tags), tags)
    assert np.array_equal(host(got_ct), ct)
    n = W.n_chains(length, chain)
    W.flip_bit(ct[(n // 3) * chain:], 77)
    pt, ok = oracle.chains_decrypt(w.key, w.base_iv, chain, ct, tags, aad, abytes)
    assert ok.sum() == n - 1 and ok[n // 3] == 0
    d_ct, d_tags = dev(ct), dev(tags)
    got = F.decrypt_verify(w.key, w.base_iv, chain, d_ct, d_tags, d_aad)
    assert np.array_equal(host(got[1]), ok)
    assert np.array_equal(host(got[0]), pt)
    e = F.decrypt_eager(w.key, w.base_iv, chain, d_ct, d_tags, d_aad)
    assert e.rejected() == [n // 3]
    assert np.array_equal(host(e.plaintext), pt)
    ks = F.keystream(w.key, w.base_iv, chain, length)
    got = F.apply_verify(w.key, w.base_iv, chain, d_ct, ks, d_tags, d_aad)
    assert np.array_equal(host(got[1]), ok)
    assert np.array_equal(host(got[0]), pt)


def test_captured_on_a_stream_without_scratch(F):
    """A graph captured on a stream that no call has used yet, where the plan would cut the
    chains and nothing can be allocated: they run whole, and every replay gives the eager
    results."""
    import torch
    n, blocks = 4111, 289
    length, chain = n * blocks * 16, blocks * 16
    w = W.random_case(5, length, chain)
    ct, tags = oracle.chains_encrypt(w.key, w.base_iv, chain, w.payload, None, 0)
    tags = tags.copy()
    W.flip_bit(tags.reshape(-1)[77 * 16:], 77)
    want_ok = np.ones(n, np.uint8)
    want_ok[77] = 0
    d_ct, d_tags = dev(ct), dev(tags)
    pt, ok = F.decrypt_verify(w.key, w.base_iv, chain, d_ct, d_tags)
    F.decrypt_verify(w.key, w.base_iv, chain, d_ct, d_tags)
    assert np.array_equal(host(ok), want_ok)
    out, flags = torch.zeros_like(pt), torch.zeros_like(ok)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        F.decrypt_verify(w.key, w.base_iv, chain, d_ct, d_tags, out=out, ok=flags)
    for _ in range(3):
        out.zero_()
        flags.zero_()
        g.replay()
        assert np.array_equal(host(flags), want_ok)
        assert np.array_equal(host(out), w.payload)
        F.decrypt_verify(w.key, w.base_iv, chain, d_ct, d_tags)


def test_captured_on_a_stream_of_ragged_calls(F):
    """A call whose chains are cut, captured on a stream that only ragged calls have used: it is
    accepted, and every replay gives the eager results, also after a ragged call that needs
    more scratch than any uniform one has come between."""
    import torch
    length, chain = 1 << 20, 64 << 10
    w = W.random_case(6, length, chain)
    ct, tags = oracle.chains_encrypt(w.key, w.base_iv, chain, w.payload, None, 0)
    W.flip_bit(tags.reshape(-1)[3 * 16:], 5)
    want_ok = np.ones(16, np.uint8)
    want_ok[3] = 0
    d_ct, d_tags = dev(ct), dev(tags)
    out, flags = torch.zeros_like(d_ct), torch.zeros(16, dtype=torch.uint8, device="cuda")
    cut = W.ragged_case(4003, [70000, 5, 200000, 0, 33], None, 0)
    many = W.ragged_case(4004, [16] * 240000 + [3 << 20], None, 0)   # over 480,000 partials and masks
    s = torch.cuda.Stream()
    bufs = {}

    def ragged(r):
        off, ln = r.extra["chain_off"], r.extra["chain_len"]
        if id(r) not in bufs:
            bufs[id(r)] = (oracle.ragged_encrypt(r.key, r.base_iv, off, ln, r.payload, None, 0), dev(r.payload))
        (want_c, want_t), pt = bufs[id(r)]
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            c, t = F.encrypt_tag_ragged(r.key, r.base_iv, off, ln, pt, out=torch.zeros_like(pt))
        assert np.array_equal(host(t), want_t) and np.array_equal(host(c), want_c)

    ragged(cut)
    F.decrypt_verify(w.key, w.base_iv, chain, d_ct, d_tags)   # (the key's tables, on another stream)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        F.decrypt_verify(w.key, w.base_iv, chain, d_ct, d_tags, out=out, ok=flags)
    for between in (None, many, cut, None):
        if between is not None:
            ragged(between)
        out.zero_()
        flags.zero_()
        torch.cuda.synchronize()
        g.replay()
        assert np.array_equal(host(flags), want_ok)
        assert np.array_equal(host(out), w.payload)
