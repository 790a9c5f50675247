"""Builds whose round-0 sort takes the split sort (sampled splitters, up to two
scattering sweeps, buckets sorted in LDS) against the oracle, at the edges of its
shapes: one bucket in LDS, one sweep, two sweeps, partly filled tiles; keys that
fill equality buckets; and an input whose sample misses most of its keys, so that
a bucket overflows and the LSD sort repeats the work."""

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_1610_03007_amd import SuffixArrayBuilder

pytestmark = pytest.mark.gpu

LDS_PAIRS = 3840  # an input of one bucket


@pytest.fixture(scope="module")
def builder():
    b = SuffixArrayBuilder(0, tune_cache="")
    yield b
    b.close()


def check(b, text):
    t = np.ascontiguousarray(text, dtype=np.uint8)
    sa = b.build(torch.from_numpy(t.copy()).to("cuda:0"))
    torch.cuda.synchronize()
    assert np.array_equal(sa.cpu().numpy().view(np.uint32), oracle.sa(t, parallel=True)), t.size


@pytest.mark.parametrize("n", [1, 2, 63, 127, 128, 129, LDS_PAIRS - 1, LDS_PAIRS, LDS_PAIRS + 1,
                               4 * 2048, 4 * 2048 + 1, (1 << 20) - 1, 1 << 20, (1 << 20) + 1,
                               (1 << 22) - 3, (1 << 22) + 6144 * 3 + 1])
def test_shapes(builder, n):
    check(builder, W.dna(n, seed=n))
    rng = np.random.default_rng(n)
    check(builder, rng.integers(0, 256, n))


@pytest.mark.parametrize("n", [3000, 50001, 1500000, 5000000])
def test_equal_keys(builder, n):
    """Few distinct keys: every key, or all but a few, in equality buckets (among
    them the largest key there is, eight bytes of the last of 255 codes)."""
    rng = np.random.default_rng(n)
    check(builder, np.full(n, 7))
    check(builder, np.where(rng.random(n) < 0.999, 200, rng.integers(0, 200, n)))
    t = np.where(rng.random(n) < 0.9, 255, rng.integers(1, 256, n))
    check(builder, t)
    t = rng.integers(0, 4, n)
    t[n // 4:n // 2] = 2
    check(builder, t)
    check(builder, np.tile(rng.integers(0, 96, 997), n // 997 + 1)[:n])


@pytest.mark.parametrize("mode", ["eager", "lazy"])
@pytest.mark.parametrize("n", [2000, 70001, 3000001])
def test_isa_after_fused_round0(builder, mode, n):
    """Both forms of the ISA after a round 0 that left its positions in the SA, with
    survivors from ordinary and from equality buckets; the text at every alignment."""
    rng = np.random.default_rng(n)
    t = rng.integers(0, 60, n + 3).astype(np.uint8)
    t[n // 5:n // 5 + n // 50] = 9
    t[n // 2:n // 2 + n // 100] = t[n // 3:n // 3 + n // 100]
    d = torch.from_numpy(t).to("cuda:0")
    builder.set_isa_mode(mode)
    try:
        for k in range(4):
            sa = builder.build(d[k:k + n])
            torch.cuda.synchronize()
            assert np.array_equal(sa.cpu().numpy().view(np.uint32),
                                  oracle.sa(t[k:k + n], parallel=True)), (mode, n, k)
            assert builder.last_info()["rounds"] > 1
    finally:
        builder.set_isa_mode("auto")


def mix32(x):
    x = x ^ (x >> 16)
    x = (x * 0x7feb352d) & 0xFFFFFFFF
    x = x ^ (x >> 15)
    x = (x * 0x846ca68b) & 0xFFFFFFFF
    return x ^ (x >> 16)


def test_overflow_repeats_with_lsd(builder):
    n, samples = 20000, 512  # 128 buckets of 4 samples
    rng = np.random.default_rng(5)
    t = rng.integers(1, 256, n).astype(np.uint8)
    for i in range(samples):
        lo, hi = i * n // samples, (i + 1) * n // samples
        p = lo + mix32((i + 0x9e3779b9) & 0xFFFFFFFF) % (hi - lo)
        t[p:p + 8] = 1
    builder.set_trace(True)
    try:
        builder.reset_stats()
        check(builder, rng.integers(1, 256, n))
        few = builder.kernel_stats()["sort_pass"]["launches"]
        builder.reset_stats()
        check(builder, t)
        many = builder.kernel_stats()["sort_pass"]["launches"]
    finally:
        builder.set_trace(False)
    assert many > few + 4, (few, many)


@pytest.mark.parametrize("copies,n", [(400, (1 << 21) + 12345), (5000, 1 << 22)])
def test_later_rounds(builder, copies, n):
    """Rounds of more than 2^21 active suffixes: dense ones (every suffix, values
    generated) and ones over the list of survivors, with the names of each round."""
    rng = np.random.default_rng(copies)
    t = np.tile(rng.integers(0, 96, n // copies + 1), copies)[:n].astype(np.uint8)
    t[rng.integers(0, n, 40)] = 97
    check(builder, t)
    info = builder.last_info()
    assert info["rounds"] > 4 and info["dense_rounds"]


def test_batch_and_dc_builds(builder):
    """The other builds that sort this way: a batch (text number in the keys), DC3
    and DC7, over both local sort shapes."""
    rng = np.random.default_rng(11)
    for total in (9000, 700000, 2600000):
        cuts = np.sort(rng.integers(0, total + 1, 30))
        off = np.concatenate([[0], cuts, [total]]).astype(np.uint64)
        t = rng.integers(0, 3, total).astype(np.uint8)
        t[total // 3:total // 2] = 1
        d = torch.from_numpy(t).to("cuda:0")
        sa = builder.build_batch(d, off)
        torch.cuda.synchronize()
        sa = sa.cpu().numpy().view(np.uint32)
        for a, z in zip(off[:-1], off[1:]):
            if z > a:
                assert np.array_equal(sa[int(a):int(z)], oracle.sa(t[int(a):int(z)], parallel=True))
        for fn in (builder.build_dc3, builder.build_dc7):
            sa = fn(d)
            torch.cuda.synchronize()
            assert np.array_equal(sa.cpu().numpy().view(np.uint32), oracle.sa(t, parallel=True))


@pytest.mark.parametrize("copy", [3, 700, 4000, 9000])
def test_small_later_rounds(builder, copy):
    """Later rounds of a few suffixes, sorted in one workgroup (up to 4608 pairs)
    or just past it, dense in the shortest text: a text that holds one piece twice
    (survivors in two ordered runs), and a batch of such texts (nearly sorted)."""
    rng = np.random.default_rng(copy)
    for n in (2 * copy + 1, 60000):
        t = rng.integers(0, 4, n).astype(np.uint8)
        t[n - copy:] = t[:copy]
        check(builder, t)
        check(builder, t[::-1])
    texts = [np.concatenate([p, p[:k % 5], p]) for k in range(64)
             for p in (rng.integers(0, 20, copy // 100 + 24).astype(np.uint8),)]
    off = np.concatenate([[0], np.cumsum([t.size for t in texts])])
    sa = builder.build_batch(torch.from_numpy(np.concatenate(texts)).to("cuda:0"), off)
    torch.cuda.synchronize()
    sa = sa.cpu().numpy().view(np.uint32)
    for k, t in enumerate(texts):
        assert np.array_equal(sa[off[k]:off[k + 1]], oracle.sa(t)), k


@pytest.mark.parametrize("lo,hi,total", [(0, 3, 20000), (1, 90, 200000), (500, 9000, 1500000),
                                         (2000, 40000, 3000000)])
def test_batch_keys_from_texts(builder, lo, hi, total):
    """Round-0 keys of a batch taken from the texts: tiles inside one text and tiles
    that many share, empty texts, alphabets (code widths) of their own, and an arena
    that starts off a word."""
    rng = np.random.default_rng(total)
    texts, size = [], 0
    while size < total:
        n = int(rng.integers(lo, hi))
        sigma = int(rng.choice([1, 2, 4, 20, 256]))
        texts.append(rng.integers(0, sigma, n).astype(np.uint8) * (255 // max(1, sigma - 1)))
        size += n
    off = np.concatenate([[0], np.cumsum([t.size for t in texts])])
    flat = np.concatenate([[0], *texts]).astype(np.uint8)
    for shift in (0, 1):
        d = torch.from_numpy(flat[1 - shift:]).to("cuda:0")[shift:]
        sa = builder.build_batch(d, off)
        torch.cuda.synchronize()
        sa = sa.cpu().numpy().view(np.uint32)
        for k, t in enumerate(texts):
            assert np.array_equal(sa[off[k]:off[k + 1]], oracle.sa(t)), (k, t.size)


def test_batch_groups():
    """A batch of more suffixes than one split sort takes (1280 * 2^20), whose texts are
    sorted in groups, against the LSD sort of the whole (an explicit tuning asks for
    it)."""
    rng = np.random.default_rng(29)
    sizes = rng.integers(0, 7_000_000, 400)
    off = np.concatenate([[0], np.cumsum(sizes)])
    assert off[-1] > (1280 << 20)
    gen = torch.Generator(device="cuda:0").manual_seed(29)
    d = torch.randint(0, 200, (int(off[-1]),), dtype=torch.uint8, device="cuda:0", generator=gen)
    d[int(off[100]):int(off[130])] %= 3
    d[int(off[200]):int(off[201])] = 7
    got = []
    for explicit in (False, True):
        b = SuffixArrayBuilder(0, tune_cache="")
        if explicit:
            b.set_tuning(**b.tuning())
        got.append(b.build_batch(d, off))
        torch.cuda.synchronize()
        got.append(b.last_info())
        b.close()
    assert torch.equal(got[0], got[2])
    for key in ("rounds", "active"):
        assert got[1][key] == got[3][key]


def test_batch_overflow_repeats_with_lsd(builder):
    """The same in a batch, whose repeat packs the keys that the first try took from
    the texts."""
    n, samples, cut = 20000, 512, 137
    rng = np.random.default_rng(6)
    t = rng.integers(1, 256, n).astype(np.uint8)
    for i in range(samples):
        lo, hi = i * n // samples, (i + 1) * n // samples
        p = lo + mix32((i + 0x9e3779b9) & 0xFFFFFFFF) % (hi - lo)
        t[p:p + 8] = 1
    d = torch.from_numpy(t).to("cuda:0")
    builder.set_trace(True)
    try:
        builder.reset_stats()
        sa = builder.build_batch(d, [0, cut, n])
        torch.cuda.synchronize()
        stats = builder.kernel_stats()
    finally:
        builder.set_trace(False)
    sa = sa.cpu().numpy().view(np.uint32)
    assert np.array_equal(sa[:cut], oracle.sa(t[:cut]))
    assert np.array_equal(sa[cut:], oracle.sa(t[cut:]))
    assert stats["pack_text"]["launches"] == 1 and stats["sort_pass"]["launches"] > 8
