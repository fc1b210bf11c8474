"""GPU encode at the edges of the split kernel's slices (4096 and 8192
symbols), its 64-symbol chunks and groups of 4 chunks per wave, inputs whose
blocks start at odd bytes, and trees with flat nodes, pairs and single leaves
on one level: the stream equals the oracle's byte for byte."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")


def _source(kind, n, seed):
    r = np.random.default_rng(seed)
    if kind == "zipf":
        return W.draw(r, W.zipf_p(1.1, r), n)
    if kind == "skew":
        return W.draw(r, W.skew_p(), n)
    p = np.zeros(256)
    p[:int(kind)] = 1.0
    return W.draw(r, p, n)


def _check(x, bs, ans, flat):
    print("case", x.size, bs, ans, flat, flush=True)
    want = O.encode(x, bs, ans_mode=ans, flat=flat)
    got = P.pivco_encode(torch.from_numpy(x).cuda(), bs, ans_mode=ans, flat=flat).cpu().numpy()
    assert got.size == want.size and np.array_equal(got, want)


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("kind", ["zipf", "skew", "13", "256"])
@pytest.mark.parametrize("n,bs", [(63, 64), (64, 64), (65, 65), (255, 255), (257, 300), (1023, 1025), (4095, 4095),
                                  (4096, 4096), (4097, 4097), (8193, 8193), (50_001, 7777), (70_000, 70_000)])
def test_small_slices(kind, n, bs, flat):
    _check(_source(kind, n, n), bs, 1, flat)


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("ans", [0, 3])
@pytest.mark.parametrize("bs", [8191, 8192, 8193, 24_577, 1 << 20])
def test_large_slices(bs, ans, flat):
    x = _source("zipf", (8 << 20) + 4321, bs)
    _check(x, bs, ans, flat)


def test_block_of_2_24_symbols():
    """Counts past 24 bits take the 64-bit weights of the code lengths."""
    x = _source("zipf", (1 << 24) + 5, 3)
    _check(x, x.size, 0, False)
