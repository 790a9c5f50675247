"""Inputs whose pairs reach the split sort's buckets in an order, or with repeats, that
a sample could miss: the result against the oracle, and the time of a default build
against the same build with the LSD sort (an explicit tuning asks for it), whose sweeps
do not depend on the keys."""

import time

import numpy as np
import pytest
import torch

import oracle
from paper_1610_03007_amd import SuffixArrayBuilder

pytestmark = pytest.mark.gpu

# A default build may take this much of the LSD build's time: it takes 0.4 to 0.9 of it,
# and took 1.4 to 2.1 times as long where its samples or runs went wrong.
SLACK = 1.2


@pytest.fixture(scope="module")
def builders():
    split, lsd = SuffixArrayBuilder(0, tune_cache=""), SuffixArrayBuilder(0, tune_cache="")
    lsd.set_tuning(**lsd.tuning())
    yield split, lsd
    split.close()
    lsd.close()


def best_ms(call):
    best = float("inf")
    for k in range(12):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        call()
        torch.cuda.synchronize()
        if k >= 2:
            best = min(best, time.perf_counter() - t0)
    return best * 1e3


def records(n, values, width, base, first):
    """Fixed-width numbers in the given order, a line each."""
    digits = (values[:, None] // base ** np.arange(width - 1, -1, -1)) % base
    lines = np.concatenate([digits + first, np.full((values.size, 1), 10)], axis=1)
    return np.resize(lines.astype(np.uint8).reshape(-1), n)


def ordered(kind, n):
    rng = np.random.default_rng(n)
    if kind == "counter":
        return records(n, 100_000_000 + 7 * np.arange(n // 10 + 1), 9, 10, 48)
    if kind == "words":
        return records(n, np.sort(rng.integers(0, 20 ** 11, n // 12 + 1)), 11, 20, 97)
    if kind == "reads":
        return records(n, np.sort(rng.integers(0, 4 ** 31, n // 32 + 1)), 31, 4, 97)
    return np.arange(n // 4, dtype=">u4").view(np.uint8)


@pytest.mark.parametrize("n", [1100, 50_000, 1 << 20, 5_000_000])
@pytest.mark.parametrize("kind", ["counter", "words", "reads", "integers"])
def test_ordered_records(builders, kind, n):
    t = ordered(kind, n)
    d = torch.from_numpy(t.copy()).to("cuda:0")
    want = oracle.sa(t, parallel=True)
    for b in builders:
        sa = b.build(d)
        torch.cuda.synchronize()
        assert np.array_equal(sa.cpu().numpy().view(np.uint32), want)
    if n == 1 << 20:  # (the size where one part of a bucket cost most)
        split, lsd = (best_ms(lambda: b.build(d)) for b in builders)
        assert split < SLACK * lsd, (split, lsd)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2047,
                               2049, 4095, 4097])
def test_small_buckets(builders, n):
    """Inputs of one bucket around the sizes where it is split into parts and where its
    last row of pairs is partly filled, with keys of all ones among them."""
    rng = np.random.default_rng(n)
    for t in (rng.integers(0, 256, n), np.full(n, 9), np.sort(rng.integers(0, 4, n)),
              np.where(rng.random(n) < 0.8, 254, rng.integers(0, 255, n))):
        t = t.astype(np.uint8)
        if n > 300:
            t[:255] = np.arange(255)  # 255 codes: the key of eight last bytes is all ones
        sa = builders[0].build(torch.from_numpy(t).to("cuda:0"))
        torch.cuda.synchronize()
        assert np.array_equal(sa.cpu().numpy().view(np.uint32), oracle.sa(t))


def repeats(kind, n):
    if kind == "period":
        return np.tile(np.arange(65, 67, dtype=np.uint8), n // 2 + 1)[:n]
    if kind == "runs":
        return np.random.default_rng(n).integers(0, 250, n // 100 + 1).astype(np.uint8).repeat(100)[:n]
    return np.full(n, 65, dtype=np.uint8)


@pytest.mark.parametrize("kind,n", [("one", 300), ("one", 2000), ("one", 4095), ("one", 4608),
                                    ("period", 4608), ("runs", 4608), ("runs", 1 << 20)])
def test_runs_of_equal_keys(builders, kind, n):
    """Runs of equal keys inside buckets that are no equality buckets: each survivor
    looks for the head of its run."""
    t = repeats(kind, n)
    d = torch.from_numpy(t.copy()).to("cuda:0")
    want = oracle.sa(t, parallel=True)
    for b in builders:
        sa = b.build(d)
        torch.cuda.synchronize()
        assert np.array_equal(sa.cpu().numpy().view(np.uint32), want)
    if (kind, n) in (("one", 4608), ("runs", 1 << 20)):
        split, lsd = (best_ms(lambda: b.build(d)) for b in builders)
        assert split < SLACK * lsd, (split, lsd)


@pytest.mark.parametrize("texts,n", [(2, 2304), (4096, 1000)])
def test_runs_in_a_batch(builders, texts, n):
    """The same in a batch of texts of one byte each: every text is one run."""
    t = np.repeat(np.arange(texts) % 251, n).astype(np.uint8)
    off = np.arange(texts + 1, dtype=np.uint64) * np.uint64(n)
    d = torch.from_numpy(t).to("cuda:0")
    want = torch.arange(n - 1, -1, -1, dtype=torch.int32, device="cuda:0").repeat(texts)
    for b in builders:
        assert torch.equal(b.build_batch(d, off), want)
    if texts == 2:  # (round 0 in one bucket)
        split, lsd = (best_ms(lambda: b.build_batch(d, off)) for b in builders)
        assert split < SLACK * lsd, (split, lsd)
