"""Device memory that objects of the library give back when they are closed, while
their builder lives on."""

import numpy as np
import pytest
import torch

from paper_1610_03007_amd import SuffixArrayBuilder

pytestmark = pytest.mark.gpu


def test_closed_index_gives_its_memory_back():
    n = 1 << 26
    rng = np.random.default_rng(n)
    d = torch.from_numpy(rng.integers(32, 128, n).astype(np.uint8)).to("cuda:0")
    first = SuffixArrayBuilder(0, tune_cache="")  # (what the runtime itself takes once)
    first.fm_index(d[:1000], first.build(d[:1000])).close()
    first.close()
    b = SuffixArrayBuilder(0, tune_cache="")
    sa = b.build(d)
    torch.cuda.synchronize()
    free = lambda: torch.cuda.mem_get_info()[0]  # (in whole pages of the runtime's)
    before = free()
    fm = b.fm_index(d, sa)
    size = fm.info()["device_bytes"]
    assert before - free() > size // 2
    fm.close()
    assert before - free() < size // 16
    b.close()
