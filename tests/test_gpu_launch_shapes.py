"""Launch shapes chosen by a call's size, at the sizes where one gives way to
the next, against the CPU oracle.  Integer work: tolerance 0."""
import numpy as np
import pytest

import oracle
from paper_2603_10242_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ace(need_gpu):
    import torch
    from paper_2603_10242_amd import ace as A
    A.load()
    torch.cuda.set_device(0)
    A.set_tuning(**A.default_tuning())
    yield A
    A.set_tuning(**A.default_tuning())


@pytest.mark.parametrize("n_id,n_streams", [(255, 11), (65_281, 10), (65_537, 10), (40_001, 17)])
def test_derive_multi_tiles_per_workgroup(ace, n_id, n_streams):
    """One and two tiles of 256 keys per workgroup (two from 2,560 tiles over a
    launch's streams on a 256-CU device), ragged last tiles, two launches."""
    import torch
    r = np.random.default_rng(n_id)
    rev = r.integers(0, 256, (n_id, 32), dtype=np.uint8)
    streams = [(r.integers(0, 256, k % 65, dtype=np.uint8).tobytes(), bytes(range(3 * k % 65)))
               for k in range(n_streams)]
    print("derive_multi n_id=%d streams=%d" % (n_id, n_streams), flush=True)
    mid = torch.empty((n_streams, n_id, 16), dtype=torch.int32, device="cuda")
    ace.derive_keys_multi(ace.to_device(rev), streams, mid_out=mid)
    pick = np.unique(np.concatenate([np.arange(0, n_id, 97), [0, n_id - 1]]))
    got = mid[:, torch.from_numpy(pick).cuda()].cpu().numpy().view(np.uint32)
    for k, (salt, info) in enumerate(streams):
        want = oracle.hmac_midstates(oracle.derive_keys(rev[pick], salt, info, 8))
        assert np.array_equal(got[k], np.asarray(want).reshape(-1, 16)), k


@pytest.mark.parametrize("n_id,n_streams", [(80_123, 9), (72_706, 9)])
def test_derive_multi_odd_tiles(ace, n_id, n_streams):
    """313 and 285 tiles per stream: an odd number with two tiles per workgroup
    (2,817 tiles, an even share of the CUs) and with one (2,565)."""
    test_derive_multi_tiles_per_workgroup(ace, n_id, n_streams)


def test_time_of_derivations_past_an_even_share(ace):
    """40 tiles more than ten per CU cost about one round of one tile, at most 14%
    (two tiles per workgroup: a round of two, 18%)."""
    import torch
    us = []
    for tiles in (2_560, 2_600):
        rev = torch.zeros((256 * tiles, 32), dtype=torch.uint8, device="cuda")
        mid = torch.empty((256 * tiles, 16), dtype=torch.int32, device="cuda")
        best = float("inf")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                ace.derive_keys_multi(rev, [(b"s", b"i")], mid_out=mid)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 100)
        us.append(best)
    print("2,560 tiles %.1f us, 2,600 %.1f" % tuple(us), flush=True)
    assert us[1] <= 1.14 * us[0]


def attestations(n, n_id, n_blocks, seed):
    w = W.paper_attestations(n=n, n_id=n_id, seed=seed, lengths=lambda r, k: r.integers(0, 400, size=k))
    return w, w.payload, w.poff, w.att, w.domain


def sweep(n, n_id, n_blocks, seed):
    w = W.generate("shape", seed, n=n, n_id=n_id, lengths=W.lognormal_lengths, p_invalid=0.02,
                   kinds=(W.KIND_TAG, W.KIND_MSG, W.KIND_KEY))
    return w, w.msg, w.off, w.tags, w.salt


# wave tiles on a 256-CU device: one workgroup (up to 4), one wave per SIMD (1,024), one workgroup
# per CU (16,384), two per CU and more
@pytest.mark.parametrize("n,n_blocks", [(1, 1), (64, 1), (65, 1), (256, 1), (257, 1), (700, 9), (65_536, 1),
                                        (65_537, 1), (66_000, 300), (131_071, 1), (131_073, 1), (1_048_576, 1),
                                        (1_048_640, 1), (1_050_000, 41)])
@pytest.mark.parametrize("form", ["hmac", "attest"])
def test_open_calls_at_shape_edges(ace, n, n_blocks, form):
    """Open calls with resident and derived keys, as one block or many uneven
    ones (empty ones among them), some offsets decreasing and identities
    unregistered; every bitmask word and count."""
    import torch
    attest = form == "attest"
    n_id = max(2, min(n // 3, 20_000))
    w, msg, off, tags, salt = (attestations if attest else sweep)(n, n_id, n_blocks, n + 7)
    ids = w.ids.copy()
    ids[5::1009] = n_id + 3
    r = np.random.default_rng(n)
    cuts = np.sort(np.concatenate([[0, n], r.integers(0, n + 1, n_blocks - 1)]))
    if n_blocks > 3:
        cuts[2] = cuts[1]
    print("%s n=%d blocks=%d" % (form, n, n_blocks), flush=True)
    d_msg, rev = ace.to_device(msg if msg.size else np.zeros(4, np.uint8)), ace.to_device(w.rev)
    blocks, want = [], []
    for a, b in zip(cuts[:-1], cuts[1:]):
        o = off[a:b + 1].copy()
        if b - a > 200:
            o[100] = o[101] + 1     # decreasing: transaction 100 cannot be valid, 99 reads past its end
        blk = ace.upload_block(None, o, ids[a:b], tags[a:b], msg_dev=d_msg, record_bytes=72 if attest else 32)
        want.append((oracle.verify_attest if attest else oracle.verify_batch)(w.keys, msg, o, ids[a:b],
                                                                              tags[a:b], 8))
        blocks.append(blk)
    for ks in (ace.midstate_keyset(rev, salt, w.info), ace.rev_keyset(rev, salt, w.info)):
        for blk in blocks:
            blk.bitmask.fill_(-1)
            blk.count.fill_(99)
        (ace.verify_attestations if attest else ace.verify_batch)(ks, blocks)
        torch.cuda.synchronize()
        for k, (blk, (mask, count)) in enumerate(zip(blocks, want)):
            m, c = blk.result()
            assert c == count and np.array_equal(m, mask), k


def test_graph_replays_of_changing_size(ace):
    """One capture of the local form replayed for batches of a few and of many
    wave tiles per workgroup, and for none."""
    import torch
    w, msg, off, tags, salt = sweep(300_000, 5_000, 1, 3)
    d_msg = ace.to_device(msg)
    ks = ace.midstate_keyset(ace.to_device(w.rev), salt, w.info)
    g = ace.Graph(ks, 64, 1_200_000)
    for cuts in ([0, 300_000], [0, 17, 17, 3_000, 200_001], [5, 6], [0, 0], list(range(0, 300_001, 5_000))):
        print("graph blocks=%d" % (len(cuts) - 1), flush=True)
        blocks = [ace.upload_block(None, off[a:b + 1], w.ids[a:b], tags[a:b], msg_dev=d_msg)
                  for a, b in zip(cuts[:-1], cuts[1:])]
        for blk in blocks:
            blk.bitmask.fill_(-1)
            blk.count.fill_(99)
        for _ in range(2):
            g.launch(blocks)
        torch.cuda.synchronize()
        for blk, a, b in zip(blocks, cuts[:-1], cuts[1:]):
            m, c = blk.result()
            mask, count = oracle.verify_batch(w.keys, msg, off[a:b + 1], w.ids[a:b], tags[a:b], 8)
            assert c == count and np.array_equal(m, mask), (a, b)
    g.close()


def all_valid(ace, n, bad=()):
    """n copies of one valid transaction (64-byte message), those at `bad` with a
    flipped credential bit: block, keyset, expected mask."""
    import torch
    w = W.generate("copies", 11, n=64, n_id=1, lengths=lambda r, k: np.full(k, 64), p_invalid=0.0)
    ks = ace.midstate_keyset(ace.to_device(w.rev), w.salt, w.info)
    tags = torch.from_numpy(w.tags[:1].copy()).cuda().repeat(n, 1)
    truth = np.ones(n, bool)
    for i in bad:
        tags[i, 5] ^= 1
        truth[i] = False
    blk = ace.DeviceBlock(ace.to_device(w.msg[:64]).repeat(n), torch.arange(n + 1, device="cuda") * 64,
                          torch.zeros(n, dtype=torch.int32, device="cuda"), tags,
                          torch.full(((n + 31) // 32,), -1, dtype=torch.int32, device="cuda"),
                          torch.full((1,), 99, dtype=torch.int64, device="cuda"), n)
    return blk, ks, truth


# wave tiles: none to a few per workgroup, the edges of a dealt row, of one and two rounds of
# workgroups, of both workgroup widths
@pytest.mark.parametrize("tiles", [1, 2, 255, 256, 257, 511, 513, 767, 1_024, 1_025, 1_281, 2_047, 2_048, 2_049, 2_304,
                                   2_305, 4_999, 16_383, 16_384, 16_385, 32_767, 32_769, 40_001, 65_537])
def test_every_tile_once_in_the_local_form(ace, tiles):
    """Whichever workgroup takes which tiles: every mask word written, every
    transaction counted once."""
    import torch
    n = 64 * tiles - 29
    blk, ks, truth = all_valid(ace, n, bad={0, n // 3, n - 1})
    print("tiles=%d" % tiles, flush=True)
    ace.verify_batch(ks, [blk], flags=ace.ACE_BUCKETED)
    torch.cuda.synchronize()
    mask, count = blk.result()
    assert count == int(truth.sum())
    assert np.array_equal(mask, W.pack_bits(truth))


def time_of_lengths(ace, L, reps=10, attest=False, flags=0):
    """Microseconds of a call over messages of these lengths (a tensor on the
    device), resident keys; the best of five."""
    import torch
    n = L.numel()
    verify = ace.verify_attestations if attest else ace.verify_batch
    ks = ace.midstate_keyset(torch.zeros((64, 32), dtype=torch.uint8, device="cuda"), b"s", b"i")
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(L, 0, out=off[1:])
    blk = ace.DeviceBlock(torch.zeros(int(off[-1]), dtype=torch.uint8, device="cuda"), off,
                          torch.arange(n, dtype=torch.int32, device="cuda") % 64,
                          torch.zeros((n, 72 if attest else 32), dtype=torch.uint8, device="cuda"),
                          torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda"),
                          torch.zeros(1, dtype=torch.int64, device="cuda"), n)
    ws = ace.workspace(ace.verify_workspace_size(ks, [blk], flags))
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            verify(ks, [blk], ws=ws, flags=flags)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / reps)
    return best


def lengths_in_order(order, n):
    r = np.random.default_rng(n)
    if order == "one place":
        L = r.integers(64, 100, n)
        L[n // 2: n // 2 + n // 128] = 1_200
        return L
    if order == "runs of 128 tiles":
        return np.where(np.arange(n) // 8_192 % 2, 80, 800)
    return np.sort(W.lognormal_lengths(r, n))


@pytest.mark.parametrize("n", [300_000, 1_000_000])
@pytest.mark.parametrize("order", ["sorted", "one place", "runs of 128 tiles"])
def test_time_of_ordered_lengths(ace, n, order):
    """A call whose message lengths are ordered takes about the time of the same
    messages shuffled: at most 1.5 times (with one consecutive share per
    workgroup 1.5 to 5 times)."""
    import torch
    L = torch.from_numpy(lengths_in_order(order, n).astype(np.int64)).cuda()
    ordered = time_of_lengths(ace, L)
    shuffled = time_of_lengths(ace, L[torch.randperm(n, device="cuda")])
    print("n=%d %s: %.1f us, shuffled %.1f us" % (n, order, ordered, shuffled), flush=True)
    assert ordered <= 1.5 * shuffled


@pytest.mark.parametrize("n", [1_000_000, 8_000_000])
def test_time_of_a_few_long_messages(ace, n):
    """One message of 20,000 bytes among 2,048 of 100: its chain of 313 blocks is
    waited for once, at most three quarters as long again, whatever the call's size
    (sorted in four rounds of workgroups, 8M transactions waited four times)."""
    import torch
    L = torch.full((n,), 100, dtype=torch.int64, device="cuda")
    short = time_of_lengths(ace, L, 3)
    L[1000::2048] = 20_000
    chain = time_of_lengths(ace, L[1000:1001], 3)
    mixed = time_of_lengths(ace, L, 3)
    print("n=%d: %.0f us, all short %.0f, one long message alone %.0f" % (n, mixed, short, chain), flush=True)
    # the long messages' own blocks are a twentieth of the others'
    assert mixed <= 1.2 * short + 1.75 * chain


@pytest.mark.parametrize("n", [100_000, 200_000])
@pytest.mark.parametrize("lengths", ["130-154", "0-1200"])
def test_time_of_open_attestations(ace, n, lengths):
    """An open call of attestations takes the form that suits its payloads: at most
    1.25 times the faster of in order and sorted (in order, payloads of 0 to 1,200
    bytes took 1.5 times)."""
    import torch
    lo, hi = (130, 155) if lengths == "130-154" else (0, 1_201)
    L = torch.randint(lo, hi, (n,), device="cuda")
    us = [time_of_lengths(ace, L, attest=True, flags=f) for f in (0, ace.ACE_ORDERED, ace.ACE_BUCKETED)]
    print("n=%d %s: open %.1f us, in order %.1f, sorted %.1f" % (n, lengths, *us), flush=True)
    assert us[0] <= 1.25 * min(us[1:])


# wave tiles per workgroup on a 256-CU device: one, a few, sixteen (the most that are not sorted
# where all are of one block count) and seventeen
@pytest.mark.parametrize("n", [50, 20_000, 65_600, 100_001, 262_144, 262_145])
@pytest.mark.parametrize("form", ["hmac", "attest"])
def test_messages_of_one_block_count(ace, n, form):
    """Lengths that all fill the same number of blocks, some transactions invalid,
    some identities unregistered, then (last) every identity unregistered."""
    import torch
    n_id = max(2, min(n // 4, 5_000))
    even = lambda r, k: r.integers(120, 170, k)  # three blocks after the key block, or without it
    if form == "attest":
        w = W.paper_attestations(n=n, n_id=n_id, seed=n, lengths=even)
        msg, off, tags, salt = w.payload, w.poff, w.att, w.domain
    else:
        w = W.generate("even", n, n=n, n_id=n_id, lengths=even, p_invalid=0.02)
        msg, off, tags, salt = w.msg, w.off, w.tags, w.salt
    print("%s n=%d" % (form, n), flush=True)
    check = oracle.verify_attest if form == "attest" else oracle.verify_batch
    ks = ace.midstate_keyset(ace.to_device(w.rev), salt, w.info)
    ids = w.ids.copy()
    for gone in (slice(0, 0), slice(3, None, 1_009), slice(n // 2, n // 2 + 100), slice(None)):
        ids[gone] = n_id + 1
        blk = ace.upload_block(msg, off, ids, tags, record_bytes=72 if form == "attest" else 32)
        blk.bitmask.fill_(-1)
        blk.count.fill_(99)
        (ace.verify_attestations if form == "attest" else ace.verify_batch)(ks, [blk], flags=ace.ACE_BUCKETED)
        torch.cuda.synchronize()
        mask, count = blk.result()
        omask, ocount = check(w.keys, msg, off, ids, tags, 8)
        assert count == ocount and np.array_equal(mask, omask)


@pytest.mark.parametrize("sizes", [[100_003], [7_000] * 36 + [0, 1], [3] * 139 + [1024], [5] * 140 + [1025],
                                   [2] * 281, [262_145, 1, 2_000], [9] * 513, [513, 512, 511, 514, 1024]])
def test_merkle_stages(ace, sizes):
    """Trees reduced by levels, by chunks of 1,024 nodes and by both, and tables
    of one, two and three launches."""
    import torch
    r = np.random.default_rng(len(sizes) + sizes[0])
    n = sum(sizes)
    off = np.zeros(n + 1, np.uint64)
    np.cumsum(r.choice([72, 72, 72, 0, 40, 130], n), out=off[1:])
    data = r.integers(0, 256, int(off[-1]) + 1, dtype=np.uint8)
    print("merkle stages %s" % sizes[:3], flush=True)
    d_data = ace.to_device(data)
    roots = torch.zeros((len(sizes), 32), dtype=torch.uint8, device="cuda")
    trees, at = [], 0
    for k, s in enumerate(sizes):
        trees.append((d_data, ace.to_device(off[at:at + s + 1]), s, roots[k]))
        at += s
    ace.merkle_roots(trees)
    torch.cuda.synchronize()
    assert np.array_equal(roots.cpu().numpy(), oracle.merkle_roots(data, off, sizes))


# 64 segments are one workgroup, 32,768 the most that take two waves per 64 on a 256-CU device
@pytest.mark.parametrize("n", [1, 64, 65, 1_000, 32_768, 32_769])
@pytest.mark.parametrize("ragged", [False, True])
def test_chain_segments_at_shape_edges(ace, n, ragged):
    import torch
    r = np.random.default_rng(n)
    steps = r.integers(0, 40, n) if ragged else 17
    w = W.poh_segments(n, steps, seed=n + 3, n_invalid=min(n // 2, 50))
    print("chain n=%d ragged=%s" % (n, ragged), flush=True)
    omask, ocount = oracle.poh_verify(w.start, w.end, w.steps, 8)
    mask = torch.full(((n + 31) // 32,), -1, dtype=torch.int32, device="cuda")
    count = torch.full((1,), 77, dtype=torch.int64, device="cuda")
    d_steps = ace.to_device(w.steps) if ragged or len(set(w.steps.tolist())) > 1 else int(w.steps[0])
    ace.poh_verify(ace.to_device(w.start), ace.to_device(w.end), d_steps, mask, count)
    torch.cuda.synchronize()
    assert int(count.item()) == ocount
    assert np.array_equal(mask.cpu().numpy().view(np.uint32), omask)


# 32,768 identities over all streams are the most that take two waves per 64
@pytest.mark.parametrize("n_id,n_streams", [(1, 1), (64, 3), (65, 1), (32_768, 1), (32_769, 1), (3_640, 9), (3_650, 9)])
def test_derive_at_shape_edges(ace, n_id, n_streams):
    """Keys and midstates of one stream (salts and infos of every block count)
    and of several; outputs asked for separately and together."""
    import torch
    r = np.random.default_rng(n_id + n_streams)
    rev = r.integers(0, 256, (n_id, 32), dtype=np.uint8)
    d_rev = ace.to_device(rev)
    pick = np.unique(np.concatenate([np.arange(0, n_id, 61), [0, n_id - 1]]))
    print("derive n_id=%d streams=%d" % (n_id, n_streams), flush=True)

    def check(key, mid, salt, info):
        want = oracle.derive_keys(rev[pick], salt, info, 8)
        if key is not None:
            assert np.array_equal(key[pick].cpu().numpy(), want)
        if mid is not None:
            assert np.array_equal(mid[pick].cpu().numpy().view(np.uint32), oracle.hmac_midstates(want))

    pairs = [(r.integers(0, 256, s, dtype=np.uint8).tobytes(), bytes(range(i))) for s, i in
             ((0, 0), (32, 16), (64, 54), (65, 55), (1024, 255))]
    for salt, info in pairs:
        key = torch.zeros((n_id, 32), dtype=torch.uint8, device="cuda")
        mid = torch.zeros((n_id, 16), dtype=torch.int32, device="cuda")
        ace.derive_keys(d_rev, salt, info, key_out=key, mid_out=mid)
        check(key, mid, salt, info)
    only = torch.zeros((n_id, 16), dtype=torch.int32, device="cuda")
    ace.derive_keys(d_rev, pairs[1][0], pairs[1][1], mid_out=only)
    check(None, only, *pairs[1])
    streams = [pairs[k % 3] for k in range(n_streams)]
    keys = torch.zeros((n_streams, n_id, 32), dtype=torch.uint8, device="cuda")
    ace.derive_keys_multi(d_rev, streams, key_out=keys)
    for k, (salt, info) in enumerate(streams):
        check(keys[k], None, salt, info)


def with_faults(w_off, ids, n_id, n):
    """Offsets and identities with, per 640 transactions, one that starts past its end
    at a tile's first place (its neighbours read past their own ends, and the next one
    starts below the tile's first offset), one in the middle of a tile, and one
    unregistered."""
    off, ids = w_off.copy(), ids.copy()
    for at in range(64, n - 4, 640):
        off[at] = off[at + 1] + 5
    for at in range(300, n - 4, 640):
        off[at] = off[at + 1] + 3
    ids[7::640] = n_id + 2
    return off, ids


# sizes of calls that are sorted within workgroups, few and many tiles each
@pytest.mark.parametrize("n", [700, 5_000, 70_000, 300_001])
@pytest.mark.parametrize("form", ["hmac", "attest"])
def test_local_form_with_faulty_offsets(ace, n, form):
    import torch
    attest = form == "attest"
    n_id = 500
    w, msg, off, tags, salt = (attestations if attest else sweep)(n, n_id, 1, n + 11)
    off, ids = with_faults(off, w.ids, n_id, n)
    print("%s n=%d" % (form, n), flush=True)
    mask, count = (oracle.verify_attest if attest else oracle.verify_batch)(w.keys, msg, off, ids, tags, 8)
    blk = ace.upload_block(None, off, ids, tags, msg_dev=ace.to_device(msg), record_bytes=72 if attest else 32)
    blk.bitmask.fill_(-1)
    ks = ace.midstate_keyset(ace.to_device(w.rev), salt, w.info)
    (ace.verify_attestations if attest else ace.verify_batch)(ks, [blk], flags=ace.ACE_BUCKETED)
    torch.cuda.synchronize()
    m, c = blk.result()
    assert c == count and np.array_equal(m, mask)


@pytest.mark.parametrize("keys", ["midstate", "rev"])
@pytest.mark.parametrize("wide", [False, True])
def test_global_bins_of_small_replays(ace, keys, wide):
    """A graph whose maxima are beyond the local form, replayed for small batches:
    the binned kernel of large calls over wide records, faulty offsets, unregistered
    identities, unaligned messages and uneven blocks."""
    import torch
    n, n_id = 6_000, 700
    w = W.generate("bins", 77, n=n, n_id=n_id, lengths=lambda r, k: r.choice([0, 1, 55, 56, 64, 119, 200, 1_232, 5_000], k),
                   p_invalid=0.02, kinds=(W.KIND_TAG, W.KIND_KEY))
    off, ids = with_faults(w.off, w.ids, n_id, n)
    lead = 3  # no message is 4-byte aligned by itself
    d_msg = ace.to_device(np.concatenate([np.zeros(lead, np.uint8), w.msg]))
    old = ace.set_tuning(wide_min_len=200) if wide else None
    try:
        make = ace.midstate_keyset if keys == "midstate" else ace.rev_keyset
        g = ace.Graph(make(ace.to_device(w.rev), w.salt, w.info), 400, 2_200_000, ace.ACE_BUCKETED)
    finally:
        if wide:
            ace.set_tuning(**old)
    for cuts in ([0, n], [0, 1, 1, 65, 300, 301, 5_000, n], [2_000, 2_063], list(range(0, n + 1, 30))):
        print("%s wide=%s blocks=%d" % (keys, wide, len(cuts) - 1), flush=True)
        blocks = [ace.upload_block(None, off[a:b + 1] + np.uint64(lead), ids[a:b], w.tags[a:b], msg_dev=d_msg)
                  for a, b in zip(cuts[:-1], cuts[1:])]
        for blk in blocks:
            blk.bitmask.fill_(-1)
            blk.count.fill_(99)
        for _ in range(2):
            g.launch(blocks)
        torch.cuda.synchronize()
        for blk, a, b in zip(blocks, cuts[:-1], cuts[1:]):
            m, c = blk.result()
            mask, count = oracle.verify_batch(w.keys, w.msg, off[a:b + 1], ids[a:b], w.tags[a:b], 8)
            assert c == count and np.array_equal(m, mask), (a, b)
    g.close()


@pytest.mark.parametrize("form", ["hmac", "attest"])
def test_global_bins_of_many_small_blocks(ace, form):
    """33,000 blocks of two transactions are more wave tiles than the local form takes."""
    import torch
    attest = form == "attest"
    blocks_n, n_id = 33_000, 300
    n = 2 * blocks_n
    w, msg, off, tags, salt = (attestations if attest else sweep)(n, n_id, 1, 5)
    off, ids = with_faults(off, w.ids, n_id, n)
    print("%s blocks=%d" % (form, blocks_n), flush=True)
    d_msg, d_off, d_ids, d_tags = (ace.to_device(x) for x in (msg, off, ids.astype(np.uint32), tags))
    mask = torch.full((blocks_n,), -1, dtype=torch.int32, device="cuda")
    count = torch.full((blocks_n,), 99, dtype=torch.int64, device="cuda")
    blocks = [ace.DeviceBlock(d_msg, d_off[2 * b:2 * b + 3], d_ids[2 * b:2 * b + 2], d_tags[2 * b:2 * b + 2],
                              mask[b:b + 1], count[b:b + 1], 2) for b in range(blocks_n)]
    ks = ace.midstate_keyset(ace.to_device(w.rev), salt, w.info)
    (ace.verify_attestations if attest else ace.verify_batch)(ks, blocks, flags=ace.ACE_BUCKETED)
    torch.cuda.synchronize()
    # a block's message area ends at its own last offset, which changes no verdict
    omask, ocount = (oracle.verify_attest if attest else oracle.verify_batch)(w.keys, msg, off, ids, tags, 8)
    bits = np.unpackbits(omask.view(np.uint8), bitorder="little")[:n].reshape(-1, 2)
    assert np.array_equal(mask.cpu().numpy().view(np.uint32), bits[:, 0] + 2 * bits[:, 1])
    assert np.array_equal(count.cpu().numpy(), bits.sum(1)) and ocount == bits.sum()


# captured forms of up to two waves per CU's tile, of one wave per SIMD, and the same on request
@pytest.mark.parametrize("max_blocks,max_tx", [(8, 2_000), (16, 50_000)])
@pytest.mark.parametrize("keys", ["midstate", "rev"])
@pytest.mark.parametrize("ordered", [False, True])
def test_small_graphs(ace, max_blocks, max_tx, keys, ordered):
    """Graphs that hold no more than a wave per SIMD, replayed at their maxima, for
    fewer transactions and blocks, for none, and at the maxima again."""
    import torch
    n_id = 900
    w, msg, off, tags, salt = sweep(max_tx, n_id, 1, max_tx)
    off, ids = with_faults(off, w.ids, n_id, max_tx)
    make = ace.midstate_keyset if keys == "midstate" else ace.rev_keyset
    g = ace.Graph(make(ace.to_device(w.rev), salt, w.info), max_blocks, max_tx, ace.ACE_ORDERED if ordered else 0)
    d_msg = ace.to_device(msg)
    full = [max_tx * k // max_blocks for k in range(max_blocks + 1)]
    for cuts in ([0, max_tx], full, [5, 6], [0, 0], [0, 64, 64, 65, 1_500], [100, 164], full):
        print("graph %d/%d %s ordered=%s blocks=%d" % (max_blocks, max_tx, keys, ordered, len(cuts) - 1), flush=True)
        blocks = [ace.upload_block(None, off[a:b + 1], ids[a:b], tags[a:b], msg_dev=d_msg)
                  for a, b in zip(cuts[:-1], cuts[1:])]
        for blk in blocks:
            blk.bitmask.fill_(-1)
            blk.count.fill_(99)
        for _ in range(2):
            g.launch(blocks)
            ace.verify_batch(make(ace.to_device(w.rev), salt, w.info), blocks[:1])  # other work between replays
        for blk in blocks:
            blk.count.fill_(99)
        g.launch(blocks)
        torch.cuda.synchronize()
        for blk, a, b in zip(blocks, cuts[:-1], cuts[1:]):
            m, c = blk.result()
            mask, count = oracle.verify_batch(w.keys, msg, off[a:b + 1], ids[a:b], tags[a:b], 8)
            assert c == count and np.array_equal(m, mask), (a, b)
    g.close()


@pytest.mark.parametrize("n_blocks", [1_023, 1_024, 1_025, 2_049, 5_000])
def test_graph_plan_of_many_blocks(ace, n_blocks):
    """The plan kernel scans 1,024 blocks at a time: prefixes of one, two, three and
    five passes, empty blocks among them."""
    import torch
    n_id = 300
    r = np.random.default_rng(n_blocks)
    sizes = r.integers(0, 4, n_blocks)
    sizes[n_blocks // 2] = 500
    n = int(sizes.sum())
    w, msg, off, tags, salt = sweep(n, n_id, 1, 9)
    print("plan blocks=%d tx=%d" % (n_blocks, n), flush=True)
    g = ace.Graph(ace.midstate_keyset(ace.to_device(w.rev), salt, w.info), n_blocks, n)
    d_msg, d_off, d_ids, d_tags = (ace.to_device(x) for x in (msg, off, w.ids.astype(np.uint32), tags))
    cuts = np.concatenate([[0], np.cumsum(sizes)])
    words = np.concatenate([[0], np.cumsum((sizes + 31) // 32)])
    mask = torch.full((int(words[-1]) + 1,), -1, dtype=torch.int32, device="cuda")
    count = torch.full((n_blocks,), 99, dtype=torch.int64, device="cuda")
    blocks = [ace.DeviceBlock(d_msg, d_off[a:b + 1], d_ids[a:b], d_tags[a:b], mask[int(words[k]):int(words[k + 1])],
                              count[k:k + 1], int(b - a)) for k, (a, b) in enumerate(zip(cuts[:-1], cuts[1:]))]
    for some in (blocks, blocks[:7], blocks):
        mask.fill_(-1)
        count.fill_(99)
        g.launch(some)
    torch.cuda.synchronize()
    omask, _ = oracle.verify_batch(w.keys, msg, off, w.ids, tags, 8)
    bits = np.unpackbits(omask.view(np.uint8), bitorder="little")
    got, counts = mask.cpu().numpy().view(np.uint32), count.cpu().numpy()
    for k, (a, b) in enumerate(zip(cuts[:-1], cuts[1:])):
        mine = bits[a:b]
        assert counts[k] == mine.sum(), k
        assert np.array_equal(got[words[k]:words[k + 1]], W.pack_bits(mine.astype(bool))[:(b - a + 31) // 32]), k
    g.close()


@pytest.mark.parametrize("n", [32_767, 32_768, 32_769])
@pytest.mark.parametrize("keys", ["midstate", "rev"])
def test_open_calls_at_the_pair_edge(ace, n, keys):
    """512 wave tiles are the most that take two waves each on a 256-CU device."""
    import torch
    n_id = 2_000
    w, msg, off, tags, salt = sweep(n, n_id, 1, n)
    off, ids = with_faults(off, w.ids, n_id, n)
    print("pair edge n=%d %s" % (n, keys), flush=True)
    blk = ace.upload_block(msg, off, ids, tags)
    blk.bitmask.fill_(-1)
    make = ace.midstate_keyset if keys == "midstate" else ace.rev_keyset
    ace.verify_batch(make(ace.to_device(w.rev), salt, w.info), [blk])
    torch.cuda.synchronize()
    mask, count = oracle.verify_batch(w.keys, msg, off, ids, tags, 8)
    m, c = blk.result()
    assert c == count and np.array_equal(m, mask)
