"""The split sort's paths through whole builds: the sizes where a sort is one bucket or
one sweep, names staged by position after a split sort, and a bucket that overflows in
each kind of sort, whose work is repeated with the LSD sort. Overflows are made on
purpose: the sample's positions depend on the count alone, so that keys which stand at
none of them can all be put into one bucket."""

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_1610_03007_amd import SuffixArrayBuilder, SuffixArrayServer

pytestmark = pytest.mark.gpu

ONE_BUCKET = 4608   # pairs of an input sorted as one bucket
LDS_BUCKET = 9216   # pairs of a bucket sorted in LDS at most


@pytest.fixture(scope="module")
def builder():
    b = SuffixArrayBuilder(0, tune_cache="")
    yield b
    b.close()


def lsd_builder():
    """Every sort by the LSD sweeps: an explicit tuning asks for them."""
    b = SuffixArrayBuilder(0, tune_cache="")
    b.set_tuning(**b.tuning())
    return b


def on_gpu(text):
    return torch.from_numpy(np.ascontiguousarray(text, dtype=np.uint8)).to("cuda:0")


def host(sa):
    torch.cuda.synchronize()
    return sa.cpu().numpy().view(np.uint32)


def sampled(count):
    """The positions that the sample of a sort of `count` pairs is drawn from."""
    lf = 0
    while (count >> 9) > (1 << lf):
        lf += 1
    if lf == 11 and (count >> 10) <= 1024:
        lf = 10
    while lf < 10 and (count >> 8) > (1 << lf):
        lf += 1
    over = 12 if lf > 10 else 6 if count > (512 << lf) else 4
    samples = over << lf
    i = np.arange(samples, dtype=np.uint64)
    lo, hi = i * np.uint64(count) // np.uint64(samples), (i + 1) * np.uint64(count) // np.uint64(samples)
    x = (i + np.uint64(0x9e3779b9)) & np.uint64(0xFFFFFFFF)
    for shift, mult in ((16, 0x7feb352d), (15, 0x846ca68b)):
        x = ((x ^ (x >> np.uint64(shift))) * np.uint64(mult)) & np.uint64(0xFFFFFFFF)
    x ^= x >> np.uint64(16)
    return (lo + x % np.maximum(hi - lo, 1)).astype(np.int64)


def unsampled(count, k, of=None):
    """k of the indexes below `count` (or of those in `of`) that the sample leaves out."""
    rest = np.setdiff1d(np.arange(count) if of is None else of, sampled(count))
    return np.random.default_rng(count).choice(rest, k, replace=False)


def sort_launches(b, call):
    b.set_trace(True)
    try:
        b.reset_stats()
        out = call()
        torch.cuda.synchronize()
        return out, b.kernel_stats()["sort_pass"]["launches"]
    finally:
        b.set_trace(False)


@pytest.mark.parametrize("n", [ONE_BUCKET - 1, ONE_BUCKET, ONE_BUCKET + 1])
def test_one_bucket_edge(builder, n):
    rng = np.random.default_rng(n)
    texts = [W.dna(n, seed=n), rng.integers(0, 256, n).astype(np.uint8),
             np.full(n, 3, dtype=np.uint8), np.tile(W.dna(40, seed=n), n)[:n]]
    for t in texts:
        assert np.array_equal(host(builder.build(on_gpu(t))), oracle.sa(t))
        for cut in (1, n // 3, n - 1):
            sa = host(builder.build_batch(on_gpu(t), [0, cut, cut, n]))
            assert np.array_equal(sa[:cut], oracle.sa(t[:cut]))
            assert np.array_equal(sa[cut:], oracle.sa(t[cut:]))


def test_later_round_of_one_bucket(builder):
    """Later rounds whose count goes over the size of one bucket in steps of two."""
    seen = set()
    for copy in range(2317, 2327):
        t = np.random.default_rng(7).integers(0, 4, 60000).astype(np.uint8)
        t[-copy:] = t[:copy]
        assert np.array_equal(host(builder.build(on_gpu(t))), oracle.sa(t, parallel=True))
        seen.add(builder.last_info()["active"][1])
    assert min(seen) <= ONE_BUCKET < max(seen) and max(seen) - min(seen) < 40, seen


def test_staged_names_after_split_sort(builder):
    """A 2^26-byte repetitive text, whose rounds of at least 2^22 suffixes stage their
    names: after each tested round the names are those of the LSD sort, and the finished
    array passes the oracle's check."""
    t = W.repetitive(copies=256, base_len=1 << 18)
    d = on_gpu(t)
    lsd = lsd_builder()
    for rounds in (2, 5, 0):
        got, want = builder.build_rounds(d, rounds), lsd.build_rounds(d, rounds)
        torch.cuda.synchronize()
        assert max(got[2]["active"][1:]) >= 1 << 22 and got[2]["dense_rounds"]
        assert torch.equal(got[1], want[1]), rounds
        assert got[2]["active"] == want[2]["active"]
        if rounds == 0:
            assert torch.equal(got[0], want[0])
    lsd.close()
    assert oracle.check_sa(t, host(builder.build(d)))[0] == 0


def test_overflow_in_two_sweeps(builder):
    n = 3_000_000
    t = np.random.default_rng(1).integers(0, 200, n).astype(np.uint8)
    _, few = sort_launches(builder, lambda: builder.build(on_gpu(t)))
    t[unsampled(n, 2 * LDS_BUCKET)] = 250
    sa, many = sort_launches(builder, lambda: builder.build(on_gpu(t)))
    assert many > few, (few, many)
    assert np.array_equal(host(sa), oracle.sa(t, parallel=True))


def test_overflow_in_a_dense_later_round(builder):
    """Runs of `a` of 40 to 59 between single `b`s. Round 0 (32 characters) leaves nearly
    every suffix, its few keys all sampled; in the dense round after it those that are 40
    from the next `b` have one key, which no sampled position has when the `b`s are
    placed so. The build starts again after a finished round."""
    n = (1 << 21) + 60000
    at = sampled(n)
    hit = np.zeros(n + 200, dtype=bool)
    hit[at] = True

    def text(avoid):
        rng = np.random.default_rng(2)
        t = np.full(n, 97, dtype=np.uint8)
        p = -1
        while True:
            q = p + int(rng.integers(41, 60))
            while avoid and hit[q - 40]:
                q = p + int(rng.integers(41, 60))
            if q >= n:
                return t
            t[q] = 98
            p = q

    launches = []
    for t in (text(False), text(True)):
        sa, k = sort_launches(builder, lambda: builder.build(on_gpu(t)))
        info = builder.last_info()
        assert info["active"][1] >= 1 << 21 and 1 in info["dense_rounds"], info
        assert np.array_equal(host(sa), oracle.sa(t, parallel=True))
        launches.append(k)
    assert launches[1] > launches[0], launches


def test_overflow_in_a_round_that_is_not_fused(builder):
    """sa_build_rounds packs its keys and ranks again; so does a server's first round."""
    n = 20000
    t = np.random.default_rng(3).integers(0, 200, n).astype(np.uint8)
    d = on_gpu(t)
    _, few = sort_launches(builder, lambda: builder.build_rounds(d, 1))
    t[unsampled(n, LDS_BUCKET + 1000)] = 250
    d = on_gpu(t)
    got, many = sort_launches(builder, lambda: builder.build_rounds(d, 1))
    assert many > few, (few, many)
    lsd = lsd_builder()
    want = lsd.build_rounds(d, 1)
    torch.cuda.synchronize()
    assert torch.equal(got[1], want[1])
    lsd.close()
    assert np.array_equal(host(builder.build_rounds(d, 0)[0]), oracle.sa(t))
    server = SuffixArrayServer(capacity_bytes=256 << 20, max_text=1 << 20)
    ticket = server.submit(t)
    done = False
    while not done:
        done, sa, _ = server.poll(ticket)
    assert np.array_equal(sa.view(np.uint32), oracle.sa(t))
    server.close()


@pytest.mark.parametrize("which", ["dc7_sample", "dc7_rest", "dc3_rest"])
def test_overflow_in_difference_covers(builder, which):
    """The first sort of DC7 (its readback comes next), and sorts of DC7 and DC3 after
    which other kernels run before a readback sees the overflow."""
    n = 1_000_003
    t = np.random.default_rng(4).integers(0, 200, n).astype(np.uint8)
    build = builder.build_dc3 if which == "dc3_rest" else builder.build_dc7
    _, few = sort_launches(builder, lambda: build(on_gpu(t)))
    count = [len(range(c, n, 7)) for c in range(7)]
    if which == "dc7_sample":  # entries 7 s, then 7 s + 1, then 7 s + 3
        n0, n1 = count[0] + (n % 7 == 0), count[1] + (n % 7 == 1)
        s = unsampled(n0 + n1 + count[3], LDS_BUCKET + 3000)
        p = np.where(s < n0, 7 * s, np.where(s < n0 + n1, 7 * (s - n0) + 1, 7 * (s - n0 - n1) + 3))
    elif which == "dc7_rest":  # classes 2, 4, 5, 6 in turn: those of class 2, by one character
        nns = count[2] + count[4] + count[5] + count[6]
        p = 7 * (unsampled(nns, LDS_BUCKET + 3000, of=np.arange(0, nns, 4)) // 4) + 2
    else:
        p = 3 * unsampled((n + 2) // 3, LDS_BUCKET + 3000)
    t[p[p < n]] = 250
    sa, many = sort_launches(builder, lambda: build(on_gpu(t)))
    assert many > few, (few, many)
    assert np.array_equal(host(sa), oracle.sa(t, parallel=True))
