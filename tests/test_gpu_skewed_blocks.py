"""Whole blocks of several tiles whose root keeps most symbols in a leaf: the
levels below the root are merged once for the block.  Sizes and skews on both
sides of the rule (at most 32768, or 16384 for the smaller tiles, symbols below
the root), canonical and flat-subtree trees, every coder and merge variant;
corrupt blocks get the oracle's verdict."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")


def _source(n, rest, seed, k=40):
    """n symbols, exactly `rest` of them not the frequent one."""
    r = np.random.default_rng(seed)
    x = np.full(n, 200, np.uint8)
    p = 0.7 ** np.arange(k)
    x[r.permutation(n)[:rest]] = r.choice(k, size=rest, p=p / p.sum()).astype(np.uint8)
    return x


CASES = [(32_768, 3000), (32_769, 3000), (40_001, 16_384), (40_001, 16_385), (65_536, 20_000), (65_537, 32_768),
         (80_000, 32_769), (100_003, 1), (131_072, 13_000), (131_072, 33_000), (250_000, 9000)]


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("ans", [0, 1, 3])
def test_every_variant(ans, flat):
    xs = [_source(n, rest, n + rest) for n, rest in CASES]
    streams = [torch.from_numpy(O.encode(x, x.size, ans_mode=ans, flat=flat)).cuda() for x in xs]
    for v in range(len(P.pivco_merge_variants())):
        print("variant", v, ans, flat, flush=True)
        outs = [torch.full((x.size,), 0xAB, dtype=torch.uint8, device="cuda") for x in xs]
        t = P.Tune(v, 8, 8, 0)
        plan = P.BatchPlan(streams, outs, tune=t)
        plan.launch()
        assert (plan.statuses() == 0).all()
        for x, o in zip(xs, outs):
            assert np.array_equal(o.cpu().numpy(), x)
        plan.close()


def test_bit_flips_as_the_oracle_decides():
    r = np.random.default_rng(4)
    x = _source(50_000, 9000, 4)
    good = O.encode(x, x.size, ans_mode=0)
    streams, want = [], []
    for _ in range(80):
        b = good.copy()
        p = int(r.integers(len(good) // 3, len(good)))
        b[p] ^= np.uint8(1 << int(r.integers(0, 8)))
        try:
            want.append(O.decode(b))
        except O.OracleError:
            want.append(None)
        streams.append(torch.from_numpy(b).cuda())
    outs = [torch.empty(x.size, dtype=torch.uint8, device="cuda") for _ in streams]
    outs, st = P.pivco_decode_batch(streams, outs)
    for i, w in enumerate(want):
        assert (st[i] == 0) == (w is not None), i
        if w is not None:
            assert np.array_equal(outs[i].cpu().numpy(), w), i
