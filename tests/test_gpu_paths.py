"""Kernels and dispatch branches at the sizes where they can go wrong, against the CPU oracle
(tests/parity.py: integers exactly, values within its stated tolerance)."""
import numpy as np
import pytest
import torch

from paper_2112_07221_amd import workloads as wl
from parity import Pair, run_workload

pytestmark = pytest.mark.gpu


def fill_hbm(leave):
    """Takes all of HBM but `leave` bytes (or a little less); returns what holds it."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    while torch.cuda.mem_get_info()[0] > leave and len(held) < 64:
        held.append(torch.empty(max(2 << 20, torch.cuda.mem_get_info()[0] - leave), dtype=torch.uint8, device="cuda:0"))
    assert leave - (8 << 20) < torch.cuda.mem_get_info()[0] <= leave
    return held


@pytest.mark.parametrize("cap", [1, 2])
def test_light_weight_lfu_over_a_border_of_the_first_digit(cap):
    """A cap of 1 leaves rows of the batch that can be evicted unstamped (their trim has a kernel of its
    own for the count); at iteration 2048 the policy key's first digit changes."""
    w = wl.WORKLOADS[1].scaled(batch=12, vocab=3_000, capacity=200, s=3, policy=wl.LFU_LIGHT)
    T = 2_070
    ids, grads, table = wl.IdStream(w).batches(T), wl.grad_pool(w), wl.table_init(w)
    p = Pair(w, table, lfu_cap=cap)
    try:
        ids_dev = torch.from_numpy(ids).to(p.dev)
        for t in range(T):
            p.lookup(ids[t], check_values=t % 64 == 0, ids_dev=ids_dev[t])
            p.update(ids[t], grads[t % len(grads)], ids_dev=ids_dev[t])
            if t % 256 == 0 or t >= 2_040:
                p.compare_state(values=False)
                p.compare_counters()
        p.flush_and_compare()
    finally:
        p.close()


@pytest.mark.parametrize("ahead", [0, 1, 2])
@pytest.mark.parametrize("n,vocab", [(1, 5), (1_024, 2_047), (1_025, 2_048), (2_730, 300), (2_731, 300), (5_461, 70_000), (5_462, 70_000),
                                     (8_192, 1_000_000), (8_193, 1_000_000), (131_072, 4_000_000), (131_073, 4_194_304),
                                     (262_144, 100_000), (262_145, 100_000), (262_145, 17_000_000), (20_000, 8_400_000),
                                     (4_096, 1_000_000), (4_097, 1_000_000), (16_384, 50_000), (16_385, 50_000), (32_768, 300_000), (32_769, 300_000),
                                     (65_536, 1_000_000), (65_537, 1_000_000), (524_288, 900_000), (524_289, 900_000)])
def test_every_way_a_batch_is_sorted(n, vocab, ahead):
    """One workgroup or two stages, carried or alone, on either side of the sizes at which one gives way to the other (4096 ids that nobody
    announced), a tile ends (1024) and there are more ranges (from 64, at 16384 ids, to 1024), of vocabularies whose ranges take one
    to four passes: the distinct keys and the gradient sums of a no-cache step.  Gradients are
    small integers and lr is 1, so every sum is exact."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n + ahead)
    steps = 4
    ids = [rng.integers(0, vocab, n) if t % 2 else np.minimum((rng.random(n) ** 6 * vocab).astype(np.int64), vocab - 1) for t in range(steps)]
    ids[1][n // 2] = -1 if n > 1 else ids[1][0]                       # (an id outside the vocabulary sorts behind every key)
    g = [torch.from_numpy(rng.integers(-8, 9, (n, 4)).astype(np.float32)).to(dev) for _ in range(steps)]
    table = torch.zeros(vocab, 4, device=dev)
    want = np.zeros((vocab, 4))
    cache = hc.HetCache(1, 4, 0, hc.POLICY_NONE, n, hc.OPT_SGD)
    try:
        cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
        d_ids = [torch.from_numpy(x).to(dev) for x in ids]
        out = torch.empty(n, 4, device=dev)
        for t in range(1, ahead):
            cache.prefetch(d_ids[t])
        for t in range(steps):
            if ahead and t + ahead < steps:
                cache.prefetch(d_ids[t + ahead])
            cache.lookup(d_ids[t], out)
            cache.update(d_ids[t], g[t], 1.0)
            ok = ids[t] >= 0
            got = out.cpu().numpy()
            assert np.array_equal(got[ok], want[ids[t][ok]]) and not got[~ok].any()
            assert np.array_equal(cache.last_lookup()[0], np.unique(ids[t][ok]))
            np.add.at(want, ids[t][ok], -g[t].cpu().numpy()[ok].astype(np.float64))
        assert np.array_equal(table.cpu().numpy(), want.astype(np.float32))
    finally:
        cache.close()


def drawn_positions(n, draws=256):
    """The positions whose ids cut a batch into ranges (sort_part_body's samples)."""
    t = np.arange(draws, dtype=np.uint64)
    lo, hi = t * n // draws, (t + 1) * n // draws
    return (lo + ((t * 0x9E3779B9 % 2**32) * (hi - lo) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("policy,ahead", [(0, 0), (2, 0), (0, 1), (2, 2)])
@pytest.mark.parametrize("n,vocab", [(300, 2_100), (4_097, 2_100), (16_384, 3_000_000), (16_385, 1_000_000), (65_537, 4_000_000), (262_144, 70_000)])
def test_batches_sorted_in_ranges(n, vocab, policy, ahead):
    """Ranges of one key, of no key and of more keys than a workgroup sorts at a time (all drawn positions hold other keys
    than the rest of the batch), keys that fill several ranges, ids outside the vocabulary, keys at both ends of it, cut by orders
    like and unlike the batch's, in kernels of their own and carried.  Whole numbers and lr 1, so rows are exact."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    drawn = drawn_positions(n)
    misled = rng.integers(vocab // 2, vocab // 2 + min(vocab // 2, 3 * n), n)
    misled[rng.random(n) < 0.3] = vocab // 2 + 5
    misled[drawn] = rng.integers(0, 256, 256)
    popular = np.minimum((rng.random(n) ** 4 * vocab).astype(np.int64), vocab - 1)
    popular[rng.random(n) < 0.4] = vocab - 1
    popular[rng.random(n) < 0.2] = 0
    bad = rng.integers(0, vocab, n)
    bad[rng.random(n) < 0.3] = -7
    bad[rng.random(n) < 0.1] = vocab
    bad[0] = 1 << 40
    same = np.full(n, vocab // 3)
    batches = [rng.integers(0, vocab, n), misled, popular, same, np.sort(misled), bad, np.full(n, -1), popular[::-1].copy()]
    table, want = torch.zeros(vocab, 4, device=dev), np.zeros((vocab, 4))
    cache = hc.HetCache(1 if policy == 2 else n // 3, 4, 100, policy, n, hc.OPT_SGD)
    try:
        cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
        out = torch.empty(n, 4, device=dev)
        dids = [torch.from_numpy(ids).to(dev) for ids in batches]
        for t, ids in enumerate(batches):
            d, g = dids[t], rng.integers(-8, 9, (n, 4)).astype(np.float32)
            if ahead and t + ahead < len(batches):
                cache.prefetch(dids[t + ahead])
            cache.lookup(d, out)
            ok = (ids >= 0) & (ids < vocab)
            got = out.cpu().numpy()
            assert np.array_equal(got[ok], want[ids[ok]]) and not got[~ok].any(), t
            assert np.array_equal(cache.last_lookup()[0], np.unique(ids[ok])), t
            cache.update(d, torch.from_numpy(g).to(dev), 1.0)
            np.add.at(want, ids[ok], -g[ok].astype(np.float64))
        assert cache.flush() == hc.HET_ERANGE                          # (the ids outside)
        assert np.array_equal(table.cpu().numpy(), want.astype(np.float32))
    finally:
        cache.close()


def over_full_batch(kind, n, vocab, times, rng):
    """A batch whose ids are spread over the vocabulary at the positions that decide where ranges begin, and elsewhere make one range far
    too full: `kind` says by what, `times` how many workgroups of 256 threads could sort as much as what sorts it."""
    ids = rng.integers(0, vocab, n)
    plain = np.ones(n, dtype=bool)
    for draws in (256, 1024):
        plain[drawn_positions(n, draws)] = False
    free = rng.permutation(np.flatnonzero(plain))
    at = vocab // 2 + 11
    for count, first, keys in {"some": [(1_300, at, vocab // 400)], "popular": [(4_700, at, 1)], "popular_and_some": [(2_500, at, 1), (700, at - 60, 120)],
                               "two_popular": [(1_900, at, 1), (1_900, at + 1, 1)], "many": [(6_000, at, vocab // 400)], "many_close": [(6_000, at, 150)],
                               "first": [(3_000, 0, 1)], "last": [(3_000, vocab - 1, 1)], "outside": [(3_000, -1, 1)]}[kind]:
        ids[free[:count * times]] = rng.integers(first, first + keys, count * times)
        free = free[count * times:]
    return ids


@pytest.mark.parametrize("kind", ["some", "popular", "popular_and_some", "two_popular", "many", "many_close", "first", "last", "outside"])
@pytest.mark.parametrize("n,vocab,ahead", [(30_000, 20_000, 1), (30_000, 300_000, 1), (30_000, 1 << 23, 1), (70_000, 5_000_000, 1), (200_000, 5_000_000, 0)])
def test_ranges_that_hold_too_many_keys(n, vocab, ahead, kind):
    """Sorted in kernels that carry it or in their own, with cuts from a batch unlike: the distinct keys, whole-number gradient sums, and, against
    a run that sorts the other way, every bit of sums that depend on the order of a key's gradients."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n + vocab)
    batches = [rng.integers(0, vocab, n)] + [over_full_batch(kind, n, vocab, 1 if ahead else 8, rng) if t % 2 else rng.integers(0, vocab, n) for t in range(1, 5)]
    whole = [rng.integers(-8, 9, (n, 1)).astype(np.float32) for _ in batches]
    wide = [(rng.standard_normal((n, 1)) * 2.0 ** rng.integers(-60, 60, (n, 1))).astype(np.float32) for _ in batches]
    tables = []
    for announced, grads in ((ahead, whole), (ahead, wide), (1 - ahead, wide)):
        table, want = torch.zeros(vocab, 1, device=dev), np.zeros((vocab, 1))
        cache = hc.HetCache(1, 1, 0, hc.POLICY_NONE, n, hc.OPT_SGD)
        try:
            cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
            out = torch.empty(n, 1, device=dev)
            dids = [torch.from_numpy(ids).to(dev) for ids in batches]
            for t, ids in enumerate(batches):
                if announced and t + 1 < len(batches):
                    cache.prefetch(dids[t + 1])
                cache.lookup(dids[t], out)
                ok = ids >= 0
                assert np.array_equal(cache.last_lookup()[0], np.unique(ids[ok])), t
                cache.update(dids[t], torch.from_numpy(grads[t]).to(dev), 1.0)
                if grads is whole:
                    assert np.array_equal(out.cpu().numpy()[ok], want[ids[ok]]), t
                    np.add.at(want, ids[ok], -grads[t][ok].astype(np.float64))
            torch.cuda.synchronize()
            tables.append(table.cpu().numpy())
            if grads is whole:
                assert np.array_equal(tables[-1], want.astype(np.float32))
        finally:
            cache.close()
    assert np.array_equal(tables[1].view(np.uint32), tables[2].view(np.uint32))


def test_a_range_of_a_wide_interval_that_holds_too_many_keys():
    """Keys of 26 bits in the last range, whose beginning came from a batch of small keys: five passes through memory."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    n, vocab, rng = 30_000, 60_000_000, np.random.default_rng(1)
    small, large = [rng.integers(0, 900, n) for _ in range(3)], [rng.integers(0, 900, n) for _ in range(2)]
    for ids in large:
        plain = np.ones(n, dtype=bool)
        plain[drawn_positions(n, 256)] = plain[drawn_positions(n, 1024)] = False
        some = rng.permutation(np.flatnonzero(plain))[:5_000]
        ids[some] = rng.integers(900, vocab, 5_000)
    batches = [small[0], large[0], small[1], large[1], small[2]]
    table, want = torch.zeros(vocab, 1, device=dev), np.zeros((vocab, 1))
    cache = hc.HetCache(1, 1, 0, hc.POLICY_NONE, n, hc.OPT_SGD)
    try:
        cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
        out = torch.empty(n, 1, device=dev)
        dids = [torch.from_numpy(ids).to(dev) for ids in batches]
        for t, ids in enumerate(batches):
            if t + 1 < len(batches):
                cache.prefetch(dids[t + 1])
            cache.lookup(dids[t], out)
            assert np.array_equal(out.cpu().numpy(), want[ids]) and np.array_equal(cache.last_lookup()[0], np.unique(ids)), t
            g = rng.integers(-8, 9, (n, 1)).astype(np.float32)
            cache.update(dids[t], torch.from_numpy(g).to(dev), 1.0)
            np.add.at(want, ids, -g.astype(np.float64))
        assert np.array_equal(table.cpu().numpy(), want.astype(np.float32))
    finally:
        cache.close()


@pytest.mark.parametrize("share", [0.01, 0.02, 0.04])
def test_a_rare_key_that_becomes_popular_does_not_hold_up_the_step(share):
    """The sort of a batch of 106496 ids, a new one of which makes up 1 to 4 %, carried by the update with cuts from the batch before: its longest
    workgroup lives 13 to 40 us (11 to 13 if the popularity stays).  Bound: 100 us; where a range's keys were searched again for every
    part of it, 160 us and more."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    n, vocab, steps = 106_496, 1_000_000, 12
    rng = np.random.default_rng(3)
    p = np.cumsum(np.arange(1, vocab // 26 + 1) ** -1.05)
    perm = [rng.permutation(vocab // 26) for _ in range(26)]

    def batch(t):
        ids = np.stack([f * (vocab // 26) + perm[f][np.searchsorted(p, rng.random(n // 26) * p[-1])] for f in range(26)], axis=1).reshape(-1)
        if t % 2:
            ids[rng.random(n) < share] = rng.integers(0, vocab)
        return torch.from_numpy(ids).to(dev)

    ids = [batch(t) for t in range(steps)]
    table = torch.zeros(vocab, 64, device=dev)
    out, grads = torch.empty(n, 64, device=dev), torch.zeros(n, 64, device=dev)
    cache = hc.HetCache(1, 64, 0, hc.POLICY_NONE, n, hc.OPT_SGD)
    try:
        cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
        rec = torch.zeros(1 << 13, hc.TRACE_WORDS, dtype=torch.int64, device=dev)
        longest = []
        for t in range(steps):
            if t + 1 < steps:
                cache.prefetch(ids[t + 1])
            cache.lookup(ids[t], out)
            rec.zero_()
            cache.profile_trace(rec, "apply_kernel")
            cache.update(ids[t], grads, 0.1)
            torch.cuda.synchronize()
            cache.profile_trace(None, "apply_kernel")
            r = rec.cpu().numpy()
            stage = r[r[:, 6] == 1]
            if t % 2 == 0 and t > 1 and t + 1 < steps:          # (the next batch has the new key)
                assert len(stage) > 0
                longest.append((stage[:, 5] - stage[:, 0]).max() / 100.0)      # (the counter runs at 100 MHz)
        assert np.median(longest) < 100.0, longest
    finally:
        cache.close()


def test_batches_of_two_kinds_in_turn_are_divided_as_evenly_as_of_one():
    """The sort of batches of 400000 ids of two populations in turn, one ahead, carried by the update: the cuts come from the order before the
    last one.  Its longest workgroup lives 12 us, as that of one population; with cuts made anew of drawn keys 54 to 68.
    Bound: twice that of one population, measured beside it."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    n, vocab, steps = 400_000, 500_000, 14
    rng = np.random.default_rng(4)
    p = np.cumsum(np.arange(1, vocab + 1) ** -1.05)
    perm = rng.permutation(vocab)
    longest = []
    for kinds in (1, 2):
        ids = [perm[np.searchsorted(p, rng.random(n) * p[-1])] for t in range(steps)]
        ids = [torch.from_numpy(x // 4 + vocab // 2 if kinds == 2 and t % 2 else x).to(dev) for t, x in enumerate(ids)]
        table = torch.zeros(vocab, 16, device=dev)
        out, grads = torch.empty(n, 16, device=dev), torch.zeros(n, 16, device=dev)
        cache = hc.HetCache(1, 16, 0, hc.POLICY_NONE, n, hc.OPT_SGD)
        try:
            cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
            rec = torch.zeros(1 << 14, hc.TRACE_WORDS, dtype=torch.int64, device=dev)
            lives = []
            for t in range(steps):
                if t + 1 < steps:
                    cache.prefetch(ids[t + 1])
                cache.lookup(ids[t], out)
                rec.zero_()
                cache.profile_trace(rec, "apply_kernel")
                cache.update(ids[t], grads, 0.1)
                torch.cuda.synchronize()
                cache.profile_trace(None, "apply_kernel")
                r = rec.cpu().numpy()
                stage = r[r[:, 6] == 1]
                if 2 < t < steps - 1:
                    assert len(stage) > 0
                    lives.append((stage[:, 5] - stage[:, 0]).max() / 100.0)      # (the counter runs at 100 MHz)
            longest.append(np.median(lives))
        finally:
            cache.close()
    assert longest[1] < 2 * longest[0], longest


@pytest.mark.parametrize("ahead", [1, 2, 3])
@pytest.mark.parametrize("host", [False, True])
def test_batches_of_two_kinds_and_of_several_sizes(ahead, host):
    """Cuts from the order before the last one while announcements take the buffers it lies in: batches of two populations and of three sizes, one
    to three ahead, announcements withdrawn, lookups nobody announced, updates of other ids.  Whole numbers and lr 1, so rows are exact."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(ahead)
    vocab, steps = 200_000, 24
    sizes = [(30_000, 30_000, 45_000, 9_000)[t // 2 % 4] for t in range(steps)]
    ids = [rng.integers(0, vocab, n) if t % 2 else np.minimum((rng.random(n) ** 3 * vocab / 8).astype(np.int64), vocab - 1) for t, n in enumerate(sizes)]
    dids = [torch.from_numpy(x).to(dev) for x in ids]
    table = torch.zeros(vocab, 1, pin_memory=True) if host else torch.zeros(vocab, 1, device=dev)
    clock = torch.zeros(vocab, dtype=torch.int32, pin_memory=True) if host else torch.zeros(vocab, dtype=torch.int32, device=dev)
    want = np.zeros(vocab)
    cache = hc.HetCache(20_000, 1, 100, hc.POLICY_LFU, max(sizes), hc.OPT_SGD)
    try:
        cache.attach_backing(table, None, clock, hc.BACKING_PINNED_HOST if host else hc.BACKING_HBM)
        for t in range(1, ahead):
            cache.prefetch(dids[t])
        for t, n in enumerate(sizes):
            if t % 11 == 10:
                cache.prefetch_cancel()
            if t + ahead < steps:
                cache.prefetch(dids[t + ahead])
            out = torch.empty(n, 1, device=dev)
            if t % 7 == 5:
                other = torch.from_numpy(rng.integers(0, vocab, 12_000)).to(dev)
                cache.lookup(other, torch.empty(12_000, 1, device=dev))
            cache.lookup(dids[t], out)
            assert np.array_equal(out.cpu().numpy()[:, 0], want[ids[t]]), t
            assert np.array_equal(cache.last_lookup()[0], np.unique(ids[t])), t
            g = rng.integers(-8, 9, n).astype(np.float32)
            mine = dids[t].clone() if t % 5 == 3 else dids[t]
            cache.update(mine, torch.from_numpy(g[:, None]).to(dev), 1.0)
            np.subtract.at(want, ids[t], g.astype(np.float64))
        assert cache.flush() == 0
        assert np.array_equal(table.cpu().numpy()[:, 0], want.astype(np.float32))
    finally:
        cache.close()


@pytest.mark.parametrize("ahead", [1, 2])
@pytest.mark.parametrize("n", [400, 4_096, 4_097, 16_384, 16_385, 32_768, 32_769, 65_536, 65_537, 131_072, 131_073, 262_144, 262_145, 524_288, 524_289, 1 << 20])
def test_the_sort_of_an_announced_batch_has_no_kernel_of_its_own(n, ahead):
    """Table in HBM, lookups and updates in turn: both stages are carried, for one and two batches ahead, on either side of the sizes at
    which the ranges' number and who carries a stage change.  Whole numbers and lr 1, so rows are exact."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    vocab, steps = 1_000_000, 6
    ids = [np.minimum((rng.random(n) ** 3 * vocab).astype(np.int64), vocab - 1) for _ in range(steps)]
    dids = [torch.from_numpy(x).to(dev) for x in ids]
    table, want = torch.zeros(vocab, 1, device=dev), np.zeros(vocab)
    cache = hc.HetCache(1, 1, 0, hc.POLICY_NONE, n, hc.OPT_SGD)
    try:
        cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
        out = torch.empty(n, 1, device=dev)
        for t in range(1, ahead):
            cache.prefetch(dids[t])
        for t in range(steps):
            if t + ahead < steps:
                cache.prefetch(dids[t + ahead])
            if t == 1:                                   # (the first batch was not announced)
                cache.profile_begin()
            cache.lookup(dids[t], out)
            assert np.array_equal(out.cpu().numpy()[:, 0], want[ids[t]]), t
            g = rng.integers(-8, 9, n).astype(np.float32)
            cache.update(dids[t], torch.from_numpy(g[:, None]).to(dev), 1.0)
            np.subtract.at(want, ids[t], g.astype(np.float64))
        assert "sort_stage_kernel" not in cache.profile_end()
        assert np.array_equal(table.cpu().numpy()[:, 0], want.astype(np.float32))
    finally:
        cache.close()


@pytest.mark.parametrize("n", [2_000, 8_000, 32_768, 32_769])
def test_lookups_alone_leave_the_sorts_of_small_batches_to_one_kernel_each(n):
    """Lookups only, two batches ahead: the second kernel of a lookup carries the first stage of one batch and the second of another (up
    to 32768 ids), instead of the eviction before it one and itself the other."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    vocab, steps = 300_000, 8
    rng = np.random.default_rng(n)
    ids = [torch.from_numpy(rng.integers(0, vocab, n)).to(dev) for _ in range(steps + 2)]
    table = torch.randn(vocab, 16, device=dev)
    out = torch.empty(n, 16, device=dev)
    rec = torch.zeros(1 << 13, hc.TRACE_WORDS, dtype=torch.int64, device=dev)
    tiles, ranges = -(-n // 1024), 64 if n <= 16_384 else 128
    cache = hc.HetCache(40_000, 16, 100, hc.POLICY_LRU, n, hc.OPT_SGD)
    try:
        cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
        cache.prefetch(ids[1])
        for t in range(steps):
            cache.prefetch(ids[t + 2])
            rec.zero_()
            cache.profile_trace(rec, "fill_gather_kernel")
            cache.lookup(ids[t], out)
            torch.cuda.synchronize()
            cache.profile_trace(None, "fill_gather_kernel")
            assert torch.equal(out, table[ids[t]]), t
            if t >= 4:
                assert int((rec[:, 6] == 1).sum()) == (tiles + ranges if n <= 32_768 else ranges), t
    finally:
        cache.close()

@pytest.mark.parametrize("ahead", [0, 1])
def test_lookups_alone_fetch_their_rows_themselves_under_rowwise_adagrad(ahead):
    """Lookups only, row-wise Adagrad: one launch of the second kernel for each (rows left to an update that does not come take another), and
    with updates again their fetches are the updates'.  Rows and accumulators against a run that looks up once per update."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    n, vocab, steps = 3_000, 60_000, 6
    rng = np.random.default_rng(ahead)
    ids = [torch.from_numpy(rng.integers(0, vocab, n)).to(dev) for _ in range(3 * steps)]
    grads = torch.from_numpy(rng.standard_normal((n, 64)).astype(np.float32)).to(dev)
    start = torch.randn(vocab, 64, device=dev)
    results = []
    for extra in (True, False):
        table, state = start.clone(), torch.zeros(vocab, 1, device=dev)
        cache = hc.HetCache(5_000, 64, 100, hc.POLICY_LFU, n, hc.OPT_ADAGRAD_ROWWISE, 1e-8)
        try:
            cache.attach_backing(table, state, torch.zeros(vocab, dtype=torch.int32, device=dev))
            out = torch.empty(n, 64, device=dev)
            if extra:
                for t in range(steps):
                    if ahead:
                        cache.prefetch(ids[t + 1])
                    if t == 1:
                        cache.profile_begin()
                    cache.lookup(ids[t], out)
                    assert torch.equal(out, table[ids[t]]), t
                assert cache.profile_end()["fill_gather_kernel"][1] == steps - 1
            for t in range(steps, 2 * steps):            # lookup and update in turn; now and then a lookup more
                if extra and t % 3 == 0:
                    cache.lookup(ids[t + steps], out)
                    cache.lookup(ids[t + 1], out)
                cache.lookup(ids[t], out)
                cache.update(ids[t], grads, 0.1)
            assert cache.flush() == 0
            results.append((table.cpu(), state.cpu()))
        finally:
            cache.close()
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])


def test_announced_batches_of_all_sizes_in_turn():
    """Small batches behind the largest and before them, two ahead, with updates left out and lookups nobody announced in between."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(9)
    vocab, sizes = 500_000, [600_000, 300, 32_768, 1 << 20, 32_769, 5_000, 4_096, 1, 524_289, 70_000, 20_000, 900, 700_000, 20_000, 20_000, 20_000, 20_000]
    ids = [rng.integers(0, vocab, n) for n in sizes]
    dids = [torch.from_numpy(x).to(dev) for x in ids]
    table, want = torch.zeros(vocab, 1, device=dev), np.zeros(vocab)
    cache = hc.HetCache(60_000, 1, 100, hc.POLICY_LRU, 1 << 20, hc.OPT_SGD)
    try:
        cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
        cache.prefetch(dids[1])
        for t, n in enumerate(sizes):
            if t + 2 < len(sizes):
                cache.prefetch(dids[t + 2])
            out = torch.empty(n, 1, device=dev)
            if t % 5 == 2:
                other = torch.from_numpy(rng.integers(0, vocab, 9_000)).to(dev)
                cache.lookup(other, torch.empty(9_000, 1, device=dev))
            cache.lookup(dids[t], out)
            assert np.array_equal(out.cpu().numpy()[:, 0], want[ids[t]]), t
            if t % 3 != 1 and t < 13:
                g = rng.integers(-8, 9, n).astype(np.float32)
                cache.update(dids[t], torch.from_numpy(g[:, None]).to(dev), 1.0)
                np.subtract.at(want, ids[t], g.astype(np.float64))
        assert cache.flush() == 0
        assert np.array_equal(table.cpu().numpy()[:, 0], want.astype(np.float32))
    finally:
        cache.close()

@pytest.mark.parametrize("policy,s", [(0, 3), (1, 3), (3, 0)])
@pytest.mark.parametrize("batch,vocab,capacity", [(158, 60_000, 9_000), (631, 300_000, 20_000), (2_521, 300_000, 40_000)])
def test_lookups_of_batches_sorted_in_ranges(batch, vocab, capacity, policy, s):
    """Classes, slots, clocks and victims of batches nobody announced, of 64, 128 and 256 ranges."""
    w = wl.WORKLOADS[1].scaled(batch=batch, vocab=vocab, capacity=capacity, s=s, policy=policy, dim=8)
    run_workload(w, 7, state_every=1)


@pytest.mark.parametrize("full", [False, True])
def test_key_index_in_hbm_and_where_hbm_has_no_room(full):
    """If HBM has no room for the index of a table's keys when the table is attached, a hash table of the cached keys
    takes its place; lookups and updates that fetch, hit and evict read the same either way (whole numbers, so sums are
    exact)."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    vocab, n, cap = 64_000_000, 3_000, 2_000                          # (an index of 256 MB)
    rng = np.random.default_rng(3)
    table, clock = torch.zeros(vocab, 4, device=dev), torch.zeros(vocab, dtype=torch.int32, device=dev)
    out = torch.empty(n, 4, device=dev)
    cache = hc.HetCache(cap, 4, 100, hc.POLICY_LRU, n, hc.OPT_SGD)
    try:
        filler = fill_hbm(200_000_000) if full else None
        before = torch.cuda.mem_get_info()[0]
        cache.attach_backing(table, None, clock)
        taken = before - torch.cuda.mem_get_info()[0]
        assert taken < 64_000_000 if full else taken > 240_000_000
        del filler
        torch.cuda.empty_cache()
        want = {}
        for t in range(6):
            ids = np.concatenate([rng.integers(0, vocab, n - 1_000), rng.integers(0, 600, 999), [vocab - 1]])
            g = rng.integers(-8, 9, (n, 4)).astype(np.float32)
            d = torch.from_numpy(ids).to(dev)
            cache.lookup(d, out)
            assert np.array_equal(out.cpu().numpy(), np.array([want.get(i, np.zeros(4)) for i in ids.tolist()]))
            cache.update(d, torch.from_numpy(g).to(dev), 1.0)
            for i, row in zip(ids.tolist(), g):
                want[i] = want.get(i, np.zeros(4)) - row
        assert cache.stats()["resident"] == cap
        assert cache.flush() == hc.HET_OK
        keys = np.array(sorted(want))
        assert np.array_equal(table[torch.from_numpy(keys).to(dev)].cpu().numpy(), np.array([want[k] for k in keys.tolist()]))
        assert float(table.abs().sum(dtype=torch.float64)) == float(np.abs(np.array(list(want.values()))).sum())
    finally:
        cache.close()


@pytest.mark.parametrize("dim", [3, 4, 64, 132])
@pytest.mark.parametrize("length", [1, 30, 31, 32, 33, 34, 63, 64, 65, 97, 161])
def test_runs_of_every_length_over_tile_borders(length, dim):
    """Runs of one length at every offset from the update's tiles (of 64 or 128 sorted positions): a run of up to 32
    positions is summed beyond the border by the tile it begins in, a longer one in parts.  Whole numbers and lr 1,
    so sums are exact; the last tile ends in invalid ids."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    vocab = 4_000
    rng = np.random.default_rng(length)
    keys = np.repeat(np.arange(2_000, 2_200), length)
    batches = [np.concatenate([np.arange(o), keys, np.full(7, -1)]) for o in range(0, 129, 16 if length > 40 else 8)]     # (o other keys shift the runs)
    for policy in (hc.POLICY_NONE, hc.POLICY_LRU):
        cache = hc.HetCache(300, dim, 0, policy, len(batches[-1]), hc.OPT_SGD)
        table, want = torch.zeros(vocab, dim, device=dev), np.zeros((vocab, dim))
        try:
            cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
            for b in batches:
                ids = rng.permutation(b)
                g = rng.integers(-8, 9, (len(ids), dim)).astype(np.float32)
                d = torch.from_numpy(ids).to(dev)
                cache.lookup(d, torch.empty(len(ids), dim, device=dev))
                cache.update(d, torch.from_numpy(g).to(dev), 1.0)
                np.add.at(want, ids[ids >= 0], -g[ids >= 0].astype(np.float64))
            assert cache.flush() == hc.HET_ERANGE                      # (the ids of -1)
            assert np.array_equal(table.cpu().numpy(), want.astype(np.float32))
        finally:
            cache.close()


@pytest.mark.parametrize("mode", ["before", "between", "after"])
@pytest.mark.parametrize("batch,vocab,policy", [(315, 70_000, 1), (316, 1_000_000, 0), (600, 2_500_000, 1), (1_300, 300_000, 1)])
def test_sort_stages_carried_by_every_kernel_of_a_step(batch, vocab, policy, mode):
    """Announced one or two ahead: the probe carries stages too, in workgroups of 1024 threads, where the kernels behind
    it are too few."""
    w = wl.WORKLOADS[1].scaled(batch=batch, vocab=vocab, capacity=9_000, s=4, policy=policy, dim=8)
    run_workload(w, 7, state_every=2, prefetch=mode)


@pytest.mark.parametrize("optimizer", [0, 1])
@pytest.mark.parametrize("dim", [3, 16, 128, 260])
@pytest.mark.parametrize("policy,capacity,lfu_cap", [(0, 311, None), (0, 312, None), (0, 700, None), (1, 40, None), (1, 700, None), (3, 700, 1), (3, 200, 2), (3, 700, 16)])
def test_evictions_counted_beside_the_fetches(policy, capacity, lfu_cap, dim, optimizer):
    """Victims are counted in the lookup and dropped beside the update (LRU from a capacity of the batch's 312 ids
    on; LFU, whose victims may be rows of the very batch) or by kernels of their own: lookups that follow
    lookups, flushes and updates with other ids in between.  State, counters, evicted ids and the table's clocks
    after every call; the table's rows too where updates do not push early."""
    w = wl.WORKLOADS[1].scaled(batch=12, vocab=3_000, capacity=capacity, s=3, policy=policy, dim=dim, optimizer=optimizer)
    T = 40
    ids, grads, table = wl.IdStream(w).batches(T + 1), wl.grad_pool(w), wl.table_init(w)
    rng = np.random.default_rng(capacity + dim)
    p = Pair(w, table, lfu_cap=lfu_cap)
    try:
        ids_dev = torch.from_numpy(ids).to(p.dev)
        for t in range(T):
            p.lookup(ids[t], ids_dev=ids_dev[t])
            kind = rng.integers(0, 8) if t > 8 else 7
            if kind == 0:
                p.cache.flush(); p.oracle.flush()
            if kind == 1:
                p.compare_counters()
                continue                                                  # a lookup follows a lookup
            other = kind == 2                                             # (a part of the batch's ids: a buffer of its own)
            b = np.repeat(ids[t][: w.n // 2], 2) if other else ids[t]
            p.update(b, grads[t % len(grads)], ids_dev=None if other else ids_dev[t])
            p.compare_state(values=t % 8 == 0)
            p.compare_counters()
            if dim < 128:
                p.compare_table()
        p.flush_and_compare()
    finally:
        p.close()


@pytest.mark.parametrize("policy,capacity,dim,optimizer", [(0, 1, 16, 1), (0, 40, 3, 0), (0, 40, 16, 1), (0, 40, 128, 1), (0, 40, 260, 1), (0, 40, 16, 2), (0, 100, 128, 0),
                                                           (0, 150, 16, 2), (0, 180, 64, 1), (0, 180, 130, 1), (0, 700, 16, 2), (1, 40, 128, 2), (1, 700, 3, 2), (3, 200, 16, 2), (0, 180, 1_100, 0)])
def test_evictions_beside_the_update_of_any_row_of_the_batch(policy, capacity, dim, optimizer):
    """LRU and fewer slots than the batch has keys: rows of the batch that were found are victims too (the update writes them to
    the table itself); row-wise Adagrad, whose update fetches rows and whose evictions run beside it like the others'."""
    test_evictions_counted_beside_the_fetches(policy, capacity, 2 if policy == 3 else None, dim, optimizer)


def test_evictions_of_hundreds_of_thousands_of_tied_rows():
    """The last victim's slot lies behind the first 64 groups of eviction blocks (524 288 slots)."""
    w = wl.WORKLOADS[1].scaled(batch=26_924, vocab=2_000_000, capacity=650_000, s=100, policy=0, dim=4, optimizer=0)
    rng = np.random.default_rng(5)
    ids = np.stack([rng.permutation(w.vocab)[: w.n] for _ in range(3)])
    ids[1, : w.n // 2] = ids[0, : w.n // 2]
    run_workload(w, 3, ids=ids, state_every=1)


@pytest.mark.parametrize("dim", [1, 4, 20, 64, 100, 128, 130, 256, 260])
@pytest.mark.parametrize("bags", [1, 3, 37, 350])
def test_bags_added_up_by_several_row_groups(bags, dim):
    """A bag's rows shared out among 1 to 256 row groups, within a wave and over several, to bags that are empty, shorter
    than the groups are many, and hundreds of rows long; ids outside the first and the last bag."""
    w = wl.WORKLOADS[5].scaled(batch=bags, vocab=3_000, capacity=400, s=3, dim=dim, optimizer=0)
    rng = np.random.default_rng(bags * 1000 + dim)
    n, T = 1_400, 4
    ids, table = rng.integers(0, w.vocab, (T, n)), wl.table_init(w)
    p = Pair(w, table, max_ids=n)
    try:
        for t in range(T):
            cuts = np.sort(rng.integers(0, n + 1, bags + 1))
            cuts[0] = 0
            if bags > 2:
                cuts[bags // 2] = cuts[bags // 2 - 1]                     # (an empty bag)
            if t % 2:
                cuts[-1] = n
            p.offsets_np, p.offsets = cuts, torch.from_numpy(cuts).to(p.dev)
            d = torch.from_numpy(ids[t]).to(p.dev)
            p.lookup(ids[t], ids_dev=d)
            if t % 2:
                p.update(ids[t], rng.standard_normal((bags, dim)).astype(np.float32), ids_dev=d)
        p.flush_and_compare()
    finally:
        p.close()


@pytest.mark.parametrize("bags,other", [(5, 5), (40, 3), (3, 40), (700, 1)])
def test_updates_by_other_bags_than_the_lookups(bags, other):
    """The lookup leaves the bag of every position for the update; an update with other offsets, or of ids no lookup had, finds
    its own."""
    w = wl.WORKLOADS[5].scaled(batch=bags, vocab=3_000, capacity=600, s=3, dim=16, optimizer=1)
    rng = np.random.default_rng(bags)
    n = 1_000
    ids, table = rng.integers(0, 500, (4, n)), wl.table_init(w)

    def offsets(p, k):
        cuts = np.sort(rng.integers(0, n + 1, k + 1))
        cuts[0] = 0
        p.offsets_np, p.offsets = cuts, torch.from_numpy(cuts).to(p.dev)

    p = Pair(w, table, max_ids=n)
    try:
        for t in range(4):
            d = torch.from_numpy(ids[t]).to(p.dev)
            offsets(p, bags)
            p.lookup(ids[t], ids_dev=d)
            offsets(p, other if t else bags)
            b = ids[t] if t < 2 else np.roll(ids[t], 7)
            p.update(b, rng.standard_normal((len(p.offsets_np) - 1, 16)).astype(np.float32), ids_dev=d if t < 2 else None)
            p.compare_state(values=True)
        p.flush_and_compare()
    finally:
        p.close()


@pytest.mark.parametrize("when", ["before", "between"])
@pytest.mark.parametrize("policy", [0, 1, 2])
@pytest.mark.parametrize("n,vocab", [(200, 3_000), (1_024, 5_000_000), (2_700, 5_000_000), (2_731, 100_000), (5_400, 5_000_000)])
def test_small_batches_whose_sort_was_under_way_when_their_lookup_came(n, vocab, policy, when):
    """One workgroup finishes what the kernels before the lookup carried of a small batch's sort: from the keys
    that were taken when it began, so that ids changed since are flagged, whatever was left of it.  Whole numbers
    and lr 1, so rows are exact."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n + policy)
    steps = 6
    ids = [np.minimum((rng.random(n) ** 3 * vocab).astype(np.int64), vocab - 1) for _ in range(steps)]
    ids[2][n // 2] = -1
    table, want = torch.zeros(vocab, 4, device=dev), np.zeros((vocab, 4), dtype=np.float32)
    cache = hc.HetCache(150, 4, 100, policy, n, hc.OPT_SGD)
    try:
        cache.attach_backing(table, None, torch.zeros(vocab, dtype=torch.int32, device=dev))
        d = [torch.from_numpy(x).to(dev) for x in ids]
        out = torch.empty(n, 4, device=dev)
        for t in range(steps):
            if t and t == steps - 1:
                d[t][n // 3:] = (d[t][n // 3:] + 1) % vocab               # changed after the kernels of the step before had begun its sort
            if when == "before" and t + 1 < steps:
                cache.prefetch(d[t + 1])
            cache.lookup(d[t], out)
            if t == steps - 1:
                break
            if when == "between":
                cache.prefetch(d[t + 1])
            ok = ids[t] >= 0
            got = out.cpu().numpy()
            assert np.array_equal(got[ok], want[ids[t][ok]]) and not got[~ok].any()
            g = rng.integers(-8, 9, (n, 4)).astype(np.float32)
            cache.update(d[t], torch.from_numpy(g).to(dev), 1.0)
            np.add.at(want, ids[t][ok], -g[ok])
            assert cache.stats()["error_bits"] == (1 if t >= 2 else 0)
        assert cache.stats()["error_bits"] & 2
    finally:
        cache.close()


def test_a_table_in_host_memory_attaches_where_hbm_has_room_for_all_but_the_key_index():
    """What only HBM can hold is allocated before the index of the table's keys, which can do without."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    vocab, n, cap = 64_000_000, 3_000, 2_000                          # (index and clocks 256 MB each, rows on their way 512 MB)
    rng = np.random.default_rng(4)
    table = torch.zeros(vocab, 1).pin_memory()
    clock = torch.zeros(vocab, dtype=torch.int32).pin_memory()
    out = torch.empty(n, 1, device=dev)
    cache = hc.HetCache(cap, 1, 100, hc.POLICY_LRU, n, hc.OPT_SGD)
    try:
        filler = fill_hbm(900_000_000)
        before = torch.cuda.mem_get_info()[0]
        cache.attach_backing(table, None, clock, hc.BACKING_PINNED_HOST)
        assert 740_000_000 < before - torch.cuda.mem_get_info()[0] < 850_000_000
        del filler
        torch.cuda.empty_cache()
        want = {}
        for t in range(4):
            ids = np.concatenate([rng.integers(0, vocab, n - 1_000), rng.integers(0, 600, 1_000)])
            g = rng.integers(-8, 9, (n, 1)).astype(np.float32)
            d = torch.from_numpy(ids).to(dev)
            cache.lookup(d, out)
            assert np.array_equal(out.cpu().numpy()[:, 0], np.array([want.get(i, 0.0) for i in ids.tolist()]))
            cache.update(d, torch.from_numpy(g).to(dev), 1.0)
            for i, x in zip(ids.tolist(), g[:, 0].tolist()):
                want[i] = want.get(i, 0.0) - x
        assert cache.flush() == hc.HET_OK
        keys = np.array(sorted(want))
        assert np.array_equal(table.numpy()[keys, 0], np.array([want[k] for k in keys.tolist()]))
    finally:
        cache.close()


def go_on_from(p, t):
    p.cache.set_iteration(t)
    p.oracle.set_iteration(t)


@pytest.mark.parametrize("optimizer,dim", [(0, 16), (1, 128), (2, 8)])
@pytest.mark.parametrize("policy,capacity,lfu_cap", [(0, 200, None), (0, 700, None), (1, 40, None), (1, 700, None), (3, 700, 1), (3, 200, 2)])
def test_select_beyond_four_million_iterations(policy, capacity, lfu_cap, optimizer, dim):
    """From iteration 2^22 the policy key has a third digit of 1, 2, 3 ... bits: the kept histograms' bins widen and
    are counted afresh at 2^22, 2^23, ..., and the third digit is counted beside the fetches.  Across two of these
    borders, where one bin holds all rows of the last iterations, and at the last iterations that are taken;
    with lookups that follow lookups, flushes and updates with other ids in between."""
    w = wl.WORKLOADS[1].scaled(batch=12, vocab=3_000, capacity=capacity, s=3, policy=policy, dim=dim, optimizer=optimizer)
    stretches = [(0, 10), (2 ** 22 - 7, 14), (2 ** 23 - 7, 14), (2 ** 27 + 50, 30), (2 ** 32 - 2 ** 20 - 1, 14)]
    T = sum(n for _, n in stretches)
    ids, grads, table = wl.IdStream(w).batches(T), wl.grad_pool(w), wl.table_init(w)
    rng = np.random.default_rng(capacity + dim)
    p = Pair(w, table, lfu_cap=lfu_cap)
    try:
        ids_dev = torch.from_numpy(ids).to(p.dev)
        t, updated = 0, True
        for start, n in stretches:
            go_on_from(p, start)
            for k in range(n):
                p.lookup(ids[t], ids_dev=ids_dev[t])
                kind = rng.integers(0, 8) if t > 8 and k + 1 < n else 7
                if kind == 0:
                    p.cache.flush(); p.oracle.flush()
                if kind != 1:                                             # (1: a lookup follows a lookup)
                    other = kind == 2
                    b = np.repeat(ids[t][: w.n // 2], 2) if other else ids[t]
                    p.update(b, grads[t % len(grads)], ids_dev=None if other else ids_dev[t])
                    p.compare_state(values=t % 8 == 0)
                p.compare_counters()
                t += 1
        p.flush_and_compare()
    finally:
        p.close()


@pytest.mark.parametrize("policy,lfu_cap", [(0, None), (1, None), (3, 1), (3, 4)])
@pytest.mark.parametrize("gap", [2_040, 2_047, 2_048, 2_049, 5_000, 3 * 2_048 * 2_048 // 4])
def test_rows_used_again_and_evicted_after_thousands_of_iterations(gap, policy, lfu_cap):
    """Rows that lay unused for so many iterations that the probe moves them in the kept histograms one by one, in
    memory (2048 and more), and fewer; then rows of old and new stamps are evicted together."""
    w = wl.WORKLOADS[1].scaled(batch=10, width=26, vocab=5_000, capacity=800, s=50, policy=policy)
    rng = np.random.default_rng(gap)
    n, grads = w.n, wl.grad_pool(w)
    p = Pair(w, wl.table_init(w), lfu_cap=lfu_cap)
    t = 0

    def step(ids):
        nonlocal t
        t += 1
        d = torch.from_numpy(np.ascontiguousarray(ids)).to(p.dev)
        p.lookup(ids, ids_dev=d)
        p.update(ids, grads[t % len(grads)], ids_dev=d)
        p.compare_state(values=t % 4 == 0)
        p.compare_counters()

    try:
        for part in range(3):                                             # 780 rows, each used once
            step(np.arange(part * n, (part + 1) * n))
        go_on_from(p, gap)
        step(rng.permutation(np.repeat(np.arange(0, 3 * n, 6), 2)))       # every sixth of them again
        go_on_from(p, gap + 2_049)
        step(rng.permutation(np.repeat(np.arange(1, 3 * n, 12), 4)))      # others, twice as long ago
        for k in range(12):                                               # and rows are needed
            step(rng.integers(0, 5_000, n))
            if k == 5:
                go_on_from(p, gap + 7_000)
        assert p.cache.stats()["total"]["evicted"] > 1_000
        p.flush_and_compare()
    finally:
        p.close()


def test_the_iteration_count_only_goes_forward_and_not_between_a_lookup_and_its_update():
    from paper_2112_07221_amd import hetcache as hc
    w = wl.WORKLOADS[1].scaled(batch=4, capacity=100)
    ids = wl.IdStream(w).batches(1)
    p = Pair(w, wl.table_init(w))
    try:
        d = torch.from_numpy(ids[0]).to(p.dev)
        p.lookup(ids[0], ids_dev=d)
        with pytest.raises(hc.HetError):
            p.cache.set_iteration(10)
        p.update(ids[0], wl.grad_pool(w)[0], ids_dev=d)
        for bad in (-1, 0, 2 ** 32 - 2 ** 20):
            with pytest.raises(hc.HetError):
                p.cache.set_iteration(bad)
        go_on_from(p, 10)
        p.lookup(ids[0], ids_dev=d)
        p.compare_counters()
    finally:
        p.close()


FIND_VOCAB, FIND_IDS = 64_000_000, 3_000                                  # (the direct index: 256 MB)
# how Find works, policy, table in host memory, one of several workers, capacity
FIND_KINDS = [("hash table", 1, True, False, 1_700), ("hash table", 0, False, False, 1_700), ("hash table", 1, False, False, 1_700),
              ("hash table", 3, False, True, 1_700), ("index in host memory", 1, False, False, 400_000)]


@pytest.fixture(scope="module")
def find_pairs():
    """Of every kind a cache with its index in HBM and one attached when HBM was full, over tables of their own."""
    from paper_2112_07221_amd import hetcache as hc
    dev = torch.device("cuda:0")
    pairs = []
    for where, policy, host, many, cap in FIND_KINDS:
        dim, pair = 2 if host else 4, []
        for k in range(2):
            make = (lambda *a, **kw: torch.zeros(*a, **kw).pin_memory()) if host else (lambda *a, **kw: torch.zeros(*a, device=dev, **kw))
            pair.append((hc.HetCache(cap, dim, 4, policy, FIND_IDS, hc.OPT_SGD, many_writers=many), make(FIND_VOCAB, dim), make(FIND_VOCAB, dtype=torch.int32)))
        pairs.append(pair)

    def attach(entry, host):
        before = torch.cuda.mem_get_info()[0]
        entry[0].attach_backing(entry[1], None, entry[2], hc.BACKING_PINNED_HOST if host else hc.BACKING_HBM)
        return before - torch.cuda.mem_get_info()[0] - (768_000_000 if host else 0)         # (mirror of the clocks, rows on their way)

    try:
        for pair, (_, _, host, _, _) in zip(pairs, FIND_KINDS):
            assert attach(pair[0], host) > 230_000_000
        filler = [fill_hbm(990_000_000)]
        for pair, (where, _, host, _, _) in zip(pairs, FIND_KINDS):
            if where == "index in host memory":
                filler.append(fill_hbm(8 << 20))                          # (no room for a hash table of 17 MB either)
            assert abs(attach(pair[1], host)) < 50_000_000
        del filler
        torch.cuda.empty_cache()
        yield pairs
    finally:
        for pair in pairs:
            for entry in pair:
                entry[0].close()


@pytest.mark.parametrize("kind", range(len(FIND_KINDS)), ids=["-".join(map(str, k[:4])) for k in FIND_KINDS])
def test_find_without_room_for_the_key_index_agrees_with_the_index(find_pairs, kind):
    """Where HBM has no room for 4 bytes per row of the table, a hash table of the cached keys is searched, or the index
    in host memory: the same calls on a cache that has its index in HBM give the same bits everywhere.  Announced and
    other batches, lookups that follow lookups, updates with other ids, flushes."""
    dev = torch.device("cuda:0")
    _, policy, host, _, cap = FIND_KINDS[kind]
    caches, tables, clocks = zip(*find_pairs[kind])
    n, vocab, dim, steps = FIND_IDS, FIND_VOCAB, tables[0].shape[1], 14
    rng = np.random.default_rng(kind)
    ids = [np.where(rng.random(n) < 0.6, rng.integers(0, 900, n) * 71_111, rng.integers(0, vocab, n)) for _ in range(steps)]
    for t in range(3, steps, 3):
        ids[t][:800] = ids[t - 1][:800]
    ids[5][7] = vocab
    d = [torch.from_numpy(x).to(dev) for x in ids]
    part = [x[::3].flip(0).contiguous() for x in d]
    grads = [torch.randn(n, dim, device=dev) for _ in range(3)]
    outs = [torch.empty(n, dim, device=dev) for _ in caches]
    for t, what in enumerate("uulupufuulpufu"):                           # update; lookup next; update of a part of the ids; flush first
        for c, out in zip(caches, outs):
            if t + 1 < steps and t % 4:
                c.prefetch(d[t + 1])
            c.lookup(d[t], out)
        assert torch.equal(outs[0], outs[1])
        assert all(np.array_equal(a, b) for a, b in zip(caches[0].last_lookup(), caches[1].last_lookup()))
        if what == "l":
            continue
        for c in caches:
            if what == "f":
                c.flush()
            x = part[t] if what == "p" else d[t]
            c.update(x, grads[t % 3][: x.numel()], 0.5)
        assert np.array_equal(np.sort(caches[0].last_evicted()), np.sort(caches[1].last_evicted()))
        a, b = caches[0].export_state(), caches[1].export_state()
        assert all(np.array_equal(a[col], b[col]) for col in a)
        assert caches[0].stats() == caches[1].stats()
    total = caches[0].stats()["total"]
    assert total["hit"] > 5_000 and total["miss"] > 10_000 and (total["evicted"] > 10_000 or cap > 100_000)
    for c in caches:
        c.flush()
    assert np.array_equal(caches[0].export_rows()[0], caches[1].export_rows()[0])
    assert torch.equal(tables[0], tables[1]) and torch.equal(clocks[0], clocks[1])
