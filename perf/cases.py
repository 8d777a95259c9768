"""Timed workloads of the attestation library: what is prepared, what one pass
is, and what the pass cannot do without.

Every case calls the library through its Python binding the way a program that
verifies attestations does.  Sizes and distributions are those of the
repository's workloads (`paper_2603_10242_amd/workload.py`): the 4,096
transaction batch, the 100,000 transaction block, the throughput sweep, the
256 uneven blocks, serving requests, paper-form attestations, key streams,
Merkle roots and hash-chain segments.

Inputs are drawn on the GPU from the seed.  The credentials a client attaches
come from a plain SHA-256 on torch tensors (FIPS 180-4, RFC 2104, RFC 5869;
one hash chain per tensor element), which shares nothing with the library;
the expected results (`exact`) are that SHA-256's and the corruption plan's.
The ends of hash-chain segments come from the workload client (OpenSSL).
"""
import hashlib
import math

import numpy as np
import torch

from paper_2603_10242_amd import ace, workload

INFO_16 = b"ACEGF-V1-MEMPOOL"
INFO_ATTEST = b"ACEGF-V1-MEMPOOL-ATTEST"
# purpose strings of one identity's key streams (seven purposes, two validator keys)
STREAM_INFOS = [b"ACEGF-V1-PURPOSE-%d" % k for k in range(7)] + [b"ACEGF-V1-VALIDATOR", b"ACEGF-V1-VOTE"]
VALU_PER_BLOCK = 1384  # integer operations of one SHA-256 block on this instruction set


def listed():
    return [
        # the smallest call: one transaction against a resident key cache, in a
        # loop that may not allocate (a wallet's or a mempool's single check)
        {"name": "verify_one", "path": "verify", "entry": "noalloc", "form": "hmac", "keys": "mid",
         "n": 1, "blocks": 1, "n_id": 1024, "lengths": "lognormal", "ids": "uniform"},
        # the smallest batch of the workloads, keys derived in the call
        {"name": "verify_tiny", "path": "verify", "entry": "batch", "form": "hmac", "keys": "rev",
         "n": 4096, "blocks": 1, "n_id": 1024, "lengths": "fixed128", "ids": "uniform"},
        # a serving request of the mean size, resident keys
        {"name": "verify_request", "path": "verify", "entry": "batch", "form": "hmac", "keys": "mid",
         "n": 2903, "blocks": 1, "n_id": 1 << 20, "lengths": "lognormal", "ids": "zipf"},
        # one block of a slot: keys change with the slot, so they are derived in the call
        {"name": "verify_block", "path": "verify", "entry": "batch", "form": "hmac", "keys": "rev",
         "n": 100_000, "blocks": 1, "n_id": 50_000, "lengths": "uniform96-512", "ids": "zipf"},
        # the sweep's ordinary size (odd), resident keys
        {"name": "verify_1m", "path": "verify", "entry": "batch", "form": "hmac", "keys": "mid",
         "n": 1_000_003, "blocks": 1, "n_id": 1 << 20, "lengths": "lognormal", "ids": "uniform"},
        # the throughput sweep's largest batch, keys derived in the call (the benchmark's default)
        {"name": "verify_16m", "path": "verify", "entry": "batch", "form": "hmac", "keys": "rev",
         "n": 16 << 20, "blocks": 1, "n_id": 1 << 20, "lengths": "lognormal", "ids": "uniform"},
        # many uneven blocks in one captured pass
        {"name": "graph_256_blocks", "path": "verify", "entry": "graph", "form": "hmac", "keys": "mid",
         "n": 7_657_765, "blocks": 256, "n_id": 1 << 20, "lengths": "lognormal", "ids": "zipf"},
        # paper-form attestations with payload binding
        {"name": "attest_2m", "path": "verify", "entry": "batch", "form": "attest", "keys": "rev",
         "n": 2 << 20, "blocks": 1, "n_id": 1 << 18, "lengths": "payload", "ids": "uniform"},
        # every purpose and validator key of a registry
        {"name": "derive_9_streams", "path": "derive", "n_id": 131_072, "streams": 9, "keys_out": True,
         "mids_out": True},
        # attestation roots of the uneven blocks: 72-byte records
        {"name": "merkle_256_trees", "path": "merkle", "n": 7_657_765, "trees": 256, "leaf": "record72"},
        # a replay of many slots' ticks
        {"name": "chain_segments", "path": "chain", "n": 262_144, "steps": 1024, "ragged": False},
        # requests from host memory through the serving engine, results back in host memory
        {"name": "serve_requests", "path": "serve", "n": 139_296, "requests": 48, "n_id": 1 << 20,
         "lengths": "lognormal", "ids": "zipf"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["verify"] * 5 + ["derive", "merkle", "chain", "serve"])
    if path == "verify":
        form = rng.choice(["hmac", "hmac", "attest"])
        entry = rng.choice(["batch", "batch", "noalloc", "graph"]) if form == "hmac" else "batch"
        n = _log_uniform(rng, 1, 2_000_000 if entry == "noalloc" else 4_000_000)
        keys = rng.choice(["mid", "rev"])
        n_id = _log_uniform(rng, 16, 1 << 20)
        if keys == "rev":  # one to sixteen transactions an identity, as in the workloads
            n_id = max(1, min(n // rng.randint(1, 16), 1 << 20))
        if entry == "noalloc" and keys == "rev":
            n, n_id = min(n, 1_000_000), min(n_id, 1 << 18)
        return {"path": "verify", "entry": entry, "form": form, "keys": keys, "n": n,
                "blocks": min(n, _log_uniform(rng, 1, 300)) if rng.random() < 0.5 else 1, "n_id": n_id,
                "lengths": "payload" if form == "attest" else
                rng.choice(["lognormal", "lognormal", "uniform96-512", "fixed128"]),
                "ids": rng.choice(["uniform", "zipf"])}
    if path == "derive":
        mids = rng.random() < 0.8
        return {"path": "derive", "n_id": _log_uniform(rng, 100, 400_000), "streams": rng.randint(1, 9),
                "keys_out": not mids or rng.random() < 0.5, "mids_out": mids}
    if path == "merkle":
        n = _log_uniform(rng, 100, 4_000_000)
        return {"path": "merkle", "n": n, "trees": min(n, _log_uniform(rng, 1, 300)),
                "leaf": rng.choice(["record72", "record72", "uniform96-512"])}
    if path == "chain":
        n = _log_uniform(rng, 64, 262_144)
        return {"path": "chain", "n": n, "steps": _log_uniform(rng, 16, min(4096, (1 << 27) // n)),
                "ragged": rng.random() < 0.3}
    requests = rng.randint(4, 64)
    return {"path": "serve", "n": requests * _log_uniform(rng, 100, 4000), "requests": requests,
            "n_id": _log_uniform(rng, 1024, 1 << 20), "lengths": "lognormal", "ids": "zipf"}


# ------------------------------------------------------------------ SHA-256 on torch tensors
def _primes(n):
    out, k = [], 2
    while len(out) < n:
        if all(k % p for p in out):
            out.append(k)
        k += 1
    return out


def _root_bits(p, degree):
    """First 32 bits of the fractional part of the square or cube root of p."""
    x, lo, hi = p << (32 * degree), 0, 1 << 40
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if mid ** degree <= x else (lo, mid)
    return lo & 0xFFFFFFFF


def _i32(v):
    return v - (1 << 32) if v >= 1 << 31 else v


_K = [_i32(_root_bits(p, 3)) for p in _primes(64)]
_IV = [_i32(_root_bits(p, 2)) for p in _primes(8)]


def _shr(x, n):
    return (x >> n) & ((1 << (32 - n)) - 1)


def _rotr(x, n):
    return _shr(x, n).bitwise_or_(x << (32 - n))


def _xor3(a, b, c):
    return a.bitwise_xor_(b).bitwise_xor_(c)


def _compress(state, W):
    """One block: state and W are lists of 8 and 16 int32 tensors (or ints)."""
    W = list(W)
    a, b, c, d, e, f, g, h = state
    for t in range(64):
        if t >= 16:
            x, y = W[(t - 15) & 15], W[(t - 2) & 15]
            w = _xor3(_rotr(x, 7), _rotr(x, 18), _shr(x, 3)).add_(W[t & 15]).add_(W[(t - 7) & 15])
            W[t & 15] = w.add_(_xor3(_rotr(y, 17), _rotr(y, 19), _shr(y, 10)))
        t1 = _xor3(_rotr(e, 6), _rotr(e, 11), _rotr(e, 25)).add_(((f ^ g) & e) ^ g).add_(h).add_(W[t & 15])
        t1.add_(_K[t])
        t2 = _xor3(_rotr(a, 2), _rotr(a, 13), _rotr(a, 22)).add_(((a | b) & c) | (a & b))
        a, b, c, d, e, f, g, h = t2.add_(t1), a, b, c, t1.add_(d), e, f, g
    return [x + y for x, y in zip((a, b, c, d, e, f, g, h), state)]


def _const(v, like):
    return torch.full_like(like, _i32(v & 0xFFFFFFFF))


def _start(like):
    return [_const(v, like) for v in _IV]


def _pad_words(words, total_bytes, like):
    """The rest of a final block after whole words: marker, zeros, bit length."""
    out = list(words) + [_const(0x80000000, like)]
    return out + [_const(0, like) for _ in range(15 - len(out))] + [_const(8 * total_bytes, like)]


def _swap(x):
    return (x << 24) | ((x << 8) & 0xFF0000) | ((x >> 8) & 0xFF00) | ((x >> 24) & 0xFF)


def _words_of(rows):
    """uint8 [n, 4k] -> list of k big-endian int32 tensors."""
    w = _swap(rows.contiguous().view(torch.int32))
    return [w[:, k].contiguous() for k in range(w.shape[1])]


def _bytes_of(words):
    """List of k int32 tensors -> uint8 [n, 4k], big-endian."""
    return _swap(torch.stack(words, 1)).contiguous().view(torch.uint8)


def _host_words(data, like):
    pad = data + b"\0" * (-len(data) % 4)
    return [_const(int.from_bytes(pad[4 * k:4 * k + 4], "big"), like) for k in range(len(pad) // 4)]


def _hash_messages(state, prefix, msg, off):
    """Chains the padded messages msg[off[i]:off[i+1]] onto `state` (bit lengths
    count `prefix` bytes before them).  msg: uint8, 8 spare bytes at its end."""
    L = off[1:] - off[:-1]
    nb = (L + 9 + 63) // 64
    order = torch.argsort(nb, descending=True)
    per = torch.bincount(nb).flip(0).cumsum(0).flip(0).tolist()  # messages with at least b blocks
    st = [x[order] for x in state]
    L, first = L[order], off[:-1][order]
    words = msg[: msg.numel() // 4 * 4].view(torch.int32)
    # by the message bytes a word has (0: none and no marker; 1..5: zero to four)
    keep = torch.tensor([0, 0, 0xFF000000, 0xFFFF0000, 0xFFFFFF00, 0xFFFFFFFF], device=msg.device)
    mark = torch.tensor([0, 1 << 31, 1 << 23, 1 << 15, 1 << 7, 0], device=msg.device)
    for b in range(len(per) - 1):
        n = per[b + 1]
        W = []
        for j in range(16):
            at = first[:n] + (64 * b + 4 * j)
            k = (at >> 2).clamp_(max=words.numel() - 2)
            two = (words[k].to(torch.int64) & 0xFFFFFFFF) | (words[k + 1].to(torch.int64) << 32)
            w = _swap((two >> ((at & 3) << 3)).to(torch.int32))
            have = (L[:n] - (64 * b + 4 * j)).clamp_(-1, 4) + 1
            W.append((w & keep[have].to(torch.int32)) | mark[have].to(torch.int32))
        last = (64 * b + 64 >= L[:n] + 9)
        bits = (L[:n] + prefix) * 8
        W[14] = torch.where(last, (bits >> 32).to(torch.int32), W[14])
        W[15] = torch.where(last, (bits & 0xFFFFFFFF).to(torch.int32), W[15])
        for x, y in zip(st, _compress([x[:n] for x in st], W)):
            x[:n] = y
    out = [torch.empty_like(x) for x in st]
    for x, y in zip(out, st):
        x[order] = y
    return out


def _midstates(key):
    """HMAC states after K0 ^ ipad and K0 ^ opad of 32-byte keys (lists of 8 words)."""
    both = []
    for pad in (0x36363636, 0x5C5C5C5C):
        W = [k ^ _i32(pad) for k in key] + [_const(pad, key[0]) for _ in range(8)]
        both.append(_compress(_start(key[0]), W))
    return both


def _hmac(ipad, opad, words, nbytes):
    """HMAC of messages of whole words that fit one block after the key block."""
    inner = _compress(ipad, _pad_words(words, 64 + nbytes, words[0]))
    return _compress(opad, _pad_words(inner, 96, words[0]))


def _hkdf(rev, salt, info):
    """HKDF-SHA256 keys (8 words) of uint8 [n, 32] root entropies."""
    ikm = _words_of(rev)
    k0 = (hashlib.sha256(salt).digest() if len(salt) > 64 else salt).ljust(64, b"\0")
    one = ikm[0][:1]
    pads = [[x.expand_as(ikm[0]) for x in _compress(_start(one), _host_words(bytes(v ^ p for v in k0), one))]
            for p in (0x36, 0x5C)]
    ip, op = _midstates(_hmac(pads[0], pads[1], ikm, 32))
    tail = info + b"\x01"
    block = tail + b"\x80" + b"\0" * (-(len(tail) + 9) % 64) + (8 * (64 + len(tail))).to_bytes(8, "big")
    for q in range(0, len(block), 64):
        ip = _compress(ip, _host_words(block[q:q + 64], ikm[0]))
    return _compress(op, _pad_words(ip, 96, ikm[0]))


# ------------------------------------------------------------------ inputs
class _Draw:
    """Random inputs of one case, on the GPU, from its seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def bytes(self, *shape):
        return torch.randint(0, 256, shape, dtype=torch.uint8, device="cuda", generator=self.g)

    def ints(self, lo, hi, n):
        return torch.randint(lo, hi, (n,), dtype=torch.int64, device="cuda", generator=self.g)

    def lengths(self, kind, n):
        if kind == "lognormal":  # median 200, sigma 0.75, within [64, 1232]
            z = torch.randn(n, dtype=torch.float64, device="cuda", generator=self.g)
            return torch.exp(math.log(200.0) + 0.75 * z).round_().clamp_(64, 1232).to(torch.int64)
        lo, hi = {"uniform96-512": (96, 512), "payload": (130, 154), "fixed128": (128, 128),
                  "record72": (72, 72)}[kind]
        return self.ints(lo, hi + 1, n)

    def ids(self, kind, n, n_id):
        if kind == "uniform":
            return self.ints(0, n_id, n)
        cdf = torch.arange(1, n_id + 1, dtype=torch.float64, device="cuda").pow_(-1.1).cumsum_(0)
        u = torch.rand(n, dtype=torch.float64, device="cuda", generator=self.g) * cdf[-1]
        rank = torch.searchsorted(cdf, u, right=True).clamp_(max=n_id - 1)
        return torch.randperm(n_id, device="cuda", generator=self.g)[rank]

    def bad(self, n, seed, share=0.005):
        """Distinct indices of the invalid ones.  Of a batch too small for the
        share every second seed has one, so that its result tells its inputs."""
        if share * n < 1.5:
            return torch.tensor([seed // 2 % n] if seed % 2 else [], dtype=torch.int64, device="cuda")
        return torch.unique(self.ints(0, n, int(share * n + 0.5)))


def _sizes(total, parts):
    """`parts` uneven sizes (lognormal, sigma 1) that add up to total, each at
    least 1: a property of the case, as its count is."""
    w = np.exp(np.random.default_rng([total, parts]).standard_normal(parts))
    s = 1 + np.floor(w / w.sum() * (total - parts)).astype(np.int64)
    s[s.argmax()] += total - s.sum()
    return s.tolist()


def _offsets(L):
    off = torch.zeros(L.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(L, 0, out=off[1:])
    return off


def _flip(rows, which, bit):
    """Flips bit `bit` of rows[which] (uint8 [n, k])."""
    at = bit >> 3
    rows[which, at] = rows[which, at] ^ (1 << (bit & 7)).to(torch.uint8)


def _transactions(case, seed):
    """A batch: registry, messages, ids, check records and the plan's verdicts."""
    r = _Draw(seed)
    n, n_id, attest = case["n"], case["n_id"], case.get("form") == "attest"
    rev = r.bytes(n_id, 32)
    salt = r.bytes(8 if attest else 32).cpu().numpy().tobytes()
    info = INFO_ATTEST if attest else INFO_16
    ids = r.ids(case["ids"], n, n_id)
    off = _offsets(r.lengths(case["lengths"], n))
    msg = r.bytes(int(off[-1]) + 8)  # spare bytes for the generator's word reads
    # 0.5% invalid: a flipped credential bit, a flipped message bit, another identity's key
    bad = r.bad(n, seed)
    kind = r.ints(0, 3 if n_id > 1 else 2, bad.numel())
    signer = ids.clone()
    wrong = bad[kind == 2]
    if wrong.numel():
        signer[wrong] = (ids[wrong] + r.ints(1, n_id, wrong.numel())) % n_id
    ip, op = _midstates(_hkdf(rev, salt, info))
    keyed = [[x[signer] for x in s] for s in (ip, op)]
    if attest:
        digest = _hash_messages(_start(signer.to(torch.int32)), 0, msg, off)
        dom = _host_words(salt, digest[0])
        tags = _bytes_of(digest + dom + _hmac(keyed[0], keyed[1], digest + dom, 40))
    else:
        inner = _hash_messages(keyed[0], 64, msg, off)
        tags = _bytes_of(_compress(keyed[1], _pad_words(inner, 96, inner[0])))
    cut, turn = bad[kind == 0], bad[kind == 1]
    _flip(tags, cut, r.ints(0, 8 * tags.shape[1], cut.numel()))
    at = off[turn] + r.ints(0, 64, turn.numel())
    msg[at] = msg[at] ^ 1
    valid = torch.ones(n, dtype=torch.bool, device="cuda")
    valid[bad] = False
    sizes = _sizes(n, case["blocks"]) if case.get("blocks", 1) > 1 else [n]
    return dict(rev=rev, salt=salt, info=info, msg=msg[:-8], off=off, ids=ids.to(torch.int32), tags=tags,
                valid=valid, sizes=sizes)


def _pack(valid):
    """bool [n] -> int32 words, bit i % 32 of word i / 32."""
    v = torch.zeros((valid.numel() + 31) // 32 * 32, dtype=torch.int64, device=valid.device)
    v[: valid.numel()] = valid
    w = (v.view(-1, 32) << torch.arange(32, device=valid.device)).sum(1)
    return torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32)


def _words(n):
    return (n + 31) // 32


def _keyset(case, t):
    if case.get("keys") == "rev":
        return ace.rev_keyset(t["rev"], t["salt"], t["info"])
    return ace.midstate_keyset(t["rev"], t["salt"], t["info"])


def _verify_state(case, seed):
    t = _transactions(case, seed)
    mask = torch.zeros(sum(_words(s) for s in t["sizes"]), dtype=torch.int32, device="cuda")
    count = torch.zeros(len(t["sizes"]), dtype=torch.int64, device="cuda")
    blocks, at, word = [], 0, 0
    for k, s in enumerate(t["sizes"]):
        off = t["off"][at:at + s + 1]
        first, last = int(off[0]), int(off[-1])
        blocks.append(ace.DeviceBlock(t["msg"][first:last].clone(), off - first, t["ids"][at:at + s],
                                      t["tags"][at:at + s], mask[word:word + _words(s)], count[k:k + 1], s))
        at, word = at + s, word + _words(s)
    keys = _keyset(case, t)
    st = dict(path=case["path"], entry=case["entry"], attest=case["form"] == "attest", keys=keys, blocks=blocks,
              mask=mask, count=count)
    if case["entry"] == "graph":
        st["graph"] = ace.Graph(keys, case["blocks"], case["n"], ace.ACE_BUCKETED)
    elif case["entry"] == "batch":
        st["ws"] = ace.workspace(ace.verify_workspace_size(keys, blocks))
    return st


def _derive_inputs(case, seed):
    r = _Draw(seed)
    rev = r.bytes(case["n_id"], 32)
    return rev, [(r.bytes(32).cpu().numpy().tobytes(), STREAM_INFOS[k]) for k in range(case["streams"])]


def _derive_state(case, seed):
    rev, streams = _derive_inputs(case, seed)
    shape = (case["streams"], case["n_id"])
    return dict(path="derive", rev=rev, streams=streams,
                key=torch.zeros(shape + (32,), dtype=torch.uint8, device="cuda") if case["keys_out"] else None,
                mid=torch.zeros(shape + (16,), dtype=torch.int32, device="cuda") if case["mids_out"] else None)


def _merkle_inputs(case, seed):
    r = _Draw(seed)
    sizes = _sizes(case["n"], case["trees"])
    trees = []
    for s in sizes:
        off = _offsets(r.lengths(case["leaf"], s))
        trees.append((r.bytes(int(off[-1]) + 8), off, s))
    return trees


def _merkle_state(case, seed):
    roots = torch.zeros((case["trees"], 32), dtype=torch.uint8, device="cuda")
    trees = [(data[:-8], off, s, roots[k]) for k, (data, off, s) in enumerate(_merkle_inputs(case, seed))]
    return dict(path="merkle", trees=trees, roots=roots, ws=ace.merkle_roots(trees))


def _chain_inputs(case, seed):
    r = _Draw(seed)
    n = case["n"]
    start = r.bytes(n, 32)
    # Up to 16 segments start one hash apart on the same chain, so that making
    # the ends takes about steps + 16 hashes a chain; 0.5% of the ends are wrong.
    chains = (n + 15) // 16
    s = r.bytes(chains, 32).cpu().numpy()
    steps = r.ints(1, case["steps"] + 1, chains).cpu().numpy() if case["ragged"] else np.full(chains, case["steps"])
    steps = steps.astype(np.uint32)
    e = workload.client_hash_chain(s, steps)
    starts, ends, once = [s], [e], np.ones(chains, np.uint32)
    for _ in range(15):
        starts.append(workload.client_hash_chain(starts[-1], once))
        ends.append(workload.client_hash_chain(ends[-1], once))
    start, end = (torch.from_numpy(np.concatenate(v)[:n]).cuda() for v in (starts, ends))
    bad = r.bad(n, seed)
    _flip(end, bad, r.ints(0, 256, bad.numel()))
    valid = torch.ones(n, dtype=torch.bool, device="cuda")
    valid[bad] = False
    return start, end, torch.from_numpy(np.tile(steps, 16)[:n].view(np.int32).copy()).cuda(), valid


def _chain_state(case, seed):
    start, end, steps, _ = _chain_inputs(case, seed)
    return dict(path="chain", start=start, end=end, steps=steps if case["ragged"] else case["steps"],
                mask=torch.zeros(_words(case["n"]), dtype=torch.int32, device="cuda"),
                count=torch.zeros(1, dtype=torch.int64, device="cuda"))


def _serve_state(case, seed):
    t = _transactions(case, seed)
    msg, off, ids, tags = (t[k].cpu().numpy() for k in ("msg", "off", "ids", "tags"))
    requests, at = [], 0
    for s in _sizes(case["n"], case["requests"]):
        o = off[at:at + s + 1].astype(np.uint64)
        requests.append((msg[int(o[0]):int(o[-1])].copy(), o - o[0], ids[at:at + s].astype(np.uint32),
                         tags[at:at + s].copy()))
        at += s
    keys = _keyset(case, t)
    # as large as a loaded engine of this size needs it: every request staged, a few batches in flight
    arena = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
    stream = ace.Stream.create(keys, arena, 192 << 20)
    return dict(path="serve", stream=stream, requests=requests)


def prepare(case, seed):
    return {"verify": _verify_state, "derive": _derive_state, "merkle": _merkle_state, "chain": _chain_state,
            "serve": _serve_state}[case["path"]](case, seed)


def run(state):
    path = state["path"]
    if path == "verify":
        if state["entry"] == "graph":
            state["graph"].launch(state["blocks"])
        elif state["entry"] == "noalloc":
            ace.verify_batch_noalloc(state["keys"], state["blocks"])
        elif state["attest"]:
            ace.verify_attestations(state["keys"], state["blocks"], ws=state["ws"])
        else:
            ace.verify_batch(state["keys"], state["blocks"], ws=state["ws"])
        return {"bitmask": state["mask"], "count": state["count"]}
    if path == "derive":
        ace.derive_keys_multi(state["rev"], state["streams"], key_out=state["key"], mid_out=state["mid"])
        return {k: state[k] for k in ("key", "mid") if state[k] is not None}
    if path == "merkle":
        ace.merkle_roots(state["trees"], ws=state["ws"])
        return state["roots"]
    if path == "chain":
        ace.poh_verify(state["start"], state["end"], state["steps"], state["mask"], state["count"])
        return {"bitmask": state["mask"], "count": state["count"]}
    stream = state["stream"]
    tickets = [stream.submit(*r) for r in state["requests"]]
    masks, counts = [], []
    for t in tickets:
        m, c = stream.result(t)
        stream.release(t)
        masks.append(m)
        counts.append(c)
    return {"bitmask": np.concatenate(masks).view(np.int32), "count": np.array(counts, np.int64)}


# ------------------------------------------------------------------ expected results and work
def _split_pack(valid, sizes):
    masks, counts, at = [], [], 0
    for s in sizes:
        masks.append(_pack(valid[at:at + s]))
        counts.append(int(valid[at:at + s].sum()))
        at += s
    return {"bitmask": torch.cat(masks), "count": torch.tensor(counts)}


def exact(case, seed):
    path = case["path"]
    if path in ("verify", "serve"):
        t = _transactions(case, seed)
        return _split_pack(t["valid"], t["sizes"] if path == "verify" else _sizes(case["n"], case["requests"]))
    if path == "chain":
        return _split_pack(_chain_inputs(case, seed)[3], [case["n"]])
    if path == "derive":
        rev, streams = _derive_inputs(case, seed)
        keys = [_hkdf(rev, salt, info) for salt, info in streams]
        out = {}
        if case["keys_out"]:
            out["key"] = torch.stack([_bytes_of(k) for k in keys])
        if case["mids_out"]:
            out["mid"] = torch.stack([torch.stack(sum(_midstates(k), []), 1) for k in keys])
        return out
    if case["trees"] > 16:
        return None  # level by level on tensors this takes too long
    roots = []
    for data, off, n in _merkle_inputs(case, seed):
        like = torch.zeros(n, dtype=torch.int32, device="cuda")
        nodes = _hash_messages(_start(like), 0, data, off)
        while n > 1:
            W = [x[0:n - 1:2] for x in nodes] + [x[1:n:2] for x in nodes]
            up = _compress(_start(W[0]), W)
            up = _compress(up, _pad_words([], 64, W[0]))
            nodes = [torch.cat([u, x[n - 1:]]) if n & 1 else u for u, x in zip(up, nodes)]
            n = (n + 1) // 2
        roots.append(_bytes_of(nodes))
    return torch.cat(roots)


def _length_moments(kind):
    """Mean length and mean SHA-256 blocks of a message of this kind."""
    if kind == "lognormal":
        x = np.linspace(-6, 6, 20001)
        L = np.clip(np.rint(np.exp(math.log(200.0) + 0.75 * x)), 64, 1232)
        p = np.exp(-x * x / 2)
        p /= p.sum()
    else:
        lo, hi = {"uniform96-512": (96, 512), "payload": (130, 154), "fixed128": (128, 128),
                  "record72": (72, 72)}[kind]
        L = np.arange(lo, hi + 1)
        p = np.full(L.shape, 1.0 / L.size)
    return float((p * L).sum()), float((p * np.ceil((L + 9) / 64)).sum())


def work(case):
    path = case["path"]
    if path in ("verify", "serve"):
        L, nb = _length_moments(case["lengths"])
        n, n_id, attest = case["n"], case["n_id"], case.get("form") == "attest"
        used = n_id if case.get("keys") == "rev" else min(n, n_id)
        row = 32 if case.get("keys") == "rev" else 64
        blocks = n * (nb + (2 if attest else 1)) + (8 * n_id if case.get("keys") == "rev" else 0)
        return {"bytes": n * (L + (72 if attest else 32) + 8 + 4 + 0.125) + row * used, "flops": VALU_PER_BLOCK * blocks}
    if path == "derive":
        rows = case["n_id"] * case["streams"]
        return {"bytes": 32 * case["n_id"] + rows * (32 * case["keys_out"] + 64 * case["mids_out"]),
                "flops": VALU_PER_BLOCK * rows * (8 if case["mids_out"] else 6)}
    if path == "merkle":
        L, nb = _length_moments(case["leaf"])
        return {"bytes": case["n"] * (L + 8) + 32 * case["trees"],
                "flops": VALU_PER_BLOCK * (case["n"] * nb + 2 * (case["n"] - case["trees"]))}
    mean = (case["steps"] + 1) / 2 if case["ragged"] else case["steps"]
    return {"bytes": 64.125 * case["n"], "flops": VALU_PER_BLOCK * case["n"] * mean}
