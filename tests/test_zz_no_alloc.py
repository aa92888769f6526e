"""The entry point for callers that cannot allocate (het_lookup_nocache_static) against the existing
entry point it is a variant of: het_lookup on a cache created with HET_POLICY_NONE."""
import numpy as np
import pytest
import torch

from paper_2112_07221_amd import hetcache as hc

pytestmark = pytest.mark.gpu


def reference(table, ids, max_ids):
    """het_lookup of a HET_POLICY_NONE cache over `table`: (output rows, error bits)."""
    V, D = table.shape
    cache = hc.HetCache(1, D, 0, hc.POLICY_NONE, max_ids, hc.OPT_SGD, 0.0)
    try:
        cg = torch.zeros(V, dtype=torch.int32, device=table.device)
        cache.attach_backing(table, None, cg, hc.BACKING_HBM)
        out = torch.full((ids.numel(), D), float("nan"), device=table.device)
        cache.lookup(ids, out)
        return out, cache.stats()["error_bits"]
    finally:
        cache.close()


@pytest.mark.parametrize("dim", [64, 10])
def test_two_calls_in_a_row_the_second_smaller(dim):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(7)
    V = 200_000
    table = torch.from_numpy(rng.standard_normal((V, dim)).astype(np.float32)).to(dev)
    err = torch.full((1,), 77, dtype=torch.int32, device=dev)
    for n, with_bad in ((50_000, True), (777, False)):
        ids_np = (rng.zipf(1.2, size=n) % V).astype(np.int64)
        if with_bad:
            ids_np[[3, 4000, n - 1]] = [-5, V, 2**40]
        ids = torch.from_numpy(ids_np).to(dev)
        want, want_err = reference(table, ids, n)
        got = torch.full((n, dim), float("nan"), device=dev)
        rc = hc.lookup_nocache_static(table, ids, got, err)
        assert rc == hc.HET_OK, hc.strerror(rc)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), "rows differ from het_lookup's"
        assert int(err.item()) == (want_err & 1) == (1 if with_bad else 0)
        ok = torch.from_numpy((ids_np >= 0) & (ids_np < V)).to(dev)
        plain = torch.where(ok[:, None], table[ids.clamp(0, V - 1)], torch.zeros((), device=dev))
        assert torch.equal(got, plain)


def test_sizes_beyond_the_static_scratch_are_refused():
    dev = torch.device("cuda:0")
    table = torch.zeros(100, 8, device=dev)
    n = hc.NOALLOC_MAX_IDS + 1
    ids = torch.zeros(n, dtype=torch.int64, device=dev)
    out = torch.zeros(n, 8, device=dev)
    assert hc.lookup_nocache_static(table, ids, out) == hc.HET_EINVAL
    assert hc.lookup_nocache_static(table, ids[:0], out) == hc.HET_OK          # nothing to do
    wide = torch.zeros(4, 5000, device=dev)
    assert hc.lookup_nocache_static(wide, ids[:4], torch.zeros(4, 5000, device=dev)) == hc.HET_EINVAL


@pytest.mark.parametrize("n,dim,bad_at", [(1, 64, None), (1, 64, 0), (255, 10, 254), (4_097, 130, None), (8_192, 16, 8_191),
                                          (8_193, 16, 8_192), (40_000, 260, 39_999), (65_536, 4, None), (65_536, 1_023, 17)])
def test_every_variant_of_the_static_lookup_copies_rows_exactly(n, dim, bad_at):
    """Rows are copied, so the result is exact: whole 16-byte pieces or single floats, one piece per lane or
    several, the ids checked inside the launch (up to 8192) or behind a clear."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    V = 3_001
    table = torch.randn(V, dim, generator=gen, device=dev)
    ids = torch.randint(0, V, (n,), generator=gen, device=dev)
    if bad_at is not None:
        ids[bad_at] = V
    err = torch.full((1,), 77, dtype=torch.int32, device=dev)
    want = torch.where((ids < V)[:, None], table[ids.clamp(max=V - 1)], torch.zeros((), device=dev))
    for _ in range(2):
        got = torch.full((n, dim), float("nan"), device=dev)
        assert hc.lookup_nocache_static(table, ids, got, err) == hc.HET_OK
        assert torch.equal(got, want)
        assert int(err.item()) == (0 if bad_at is None else 1)
    assert hc.lookup_nocache_static(table, ids, got.zero_()) == hc.HET_OK          # nobody asks for the error bits
    assert torch.equal(got, want)
