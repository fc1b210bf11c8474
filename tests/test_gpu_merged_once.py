"""Blocks whose levels below the root are merged once (a root that keeps all but
at most 32768 symbols in a leaf): every batch here is of such blocks alone, as
the rule on the streams' sizes and the blocks' roots decides, which the test
works out for itself.  Symbols below the root from 1 to the limit and one past it, raw
and entropy-coded nodes, the leaf on either side of the root, flat nodes below
it, odd sizes, outputs at any byte, every way to launch; corrupt blocks get the
oracle's verdict beside an intact one."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")

T = 32_768                                     # symbols of a tile
KINDS = {"two": 2, "four": 4, "many": 40}


def _source(kind, n, below, seed=0):
    """n symbols, `below` of them not the frequent one (200)."""
    r = np.random.default_rng(n + below + seed)
    k = KINDS[kind]
    p = np.ones(k) if k < 40 else 0.7 ** np.arange(k)
    x = np.full(n, 200, np.uint8)
    at = r.permutation(n)[:below]
    x[at] = r.choice(k, size=below, p=p / p.sum()).astype(np.uint8)
    x[at[:k]] = np.arange(min(k, below), dtype=np.uint8)       # every symbol of the kind
    return x


def _lengths(stream):
    """Code lengths of a one-block stream."""
    b = stream[48 + 32 + 12:48 + 32 + 12 + 128]
    return np.stack([b & 15, b >> 4], axis=1).reshape(256)


def _allowed(stream, n, copies):
    """Whether a batch of `copies` of this one-block stream may be skewed (the rule
    on sizes): whole blocks of more than a tile, under 3 bits a symbol."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    words = P.pivco_stream_info(torch.from_numpy(stream).cuda())["ans_words"]
    held = stream.size + 4 * words
    split = 65_536 if held > 49_152 else max(65_536, copies * n // (2 * cus))
    return n > T and (n <= split or n > 128 * T) and 8 * held < 3 * n


def _check(x, streams, entries=("batch", "grid", "plain")):
    t = torch.from_numpy(x).cuda()
    for e in entries:
        bufs = [torch.full((x.size + 48,), 0xAB, dtype=torch.uint8, device="cuda") for _ in streams]
        at = [(0, 1, 3, 15, 16)[i % 5] for i in range(len(streams))]
        outs = [b[a:a + x.size] for b, a in zip(bufs, at)]
        if e == "batch":
            _, st = P.pivco_decode_batch(streams, outs)
        elif e == "plain":
            _, st = P.pivco_decode_plain(streams, outs)
        else:
            plan = P.BatchPlan(streams, outs, tune=P.Tune(0, 8, 8, 1))
            plan.launch()
            st = plan.statuses()
            plan.close()
        torch.cuda.synchronize()
        assert (np.asarray(st) == 0).all(), e
        for b, a in zip(bufs, at):
            assert torch.equal(b[a:a + x.size], t), (e, a)
            assert (b[:a] == 0xAB).all() and (b[a + x.size:] == 0xAB).all(), (e, a)


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("ans", [0, 1, 3])
@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("n,below", [(T + 1, 41), (T + 1, 9000), (40_001, 16_000), (50_003, 12_345), (65_535, T - 1),
                                     (65_536, T), (65_536, T + 1)])
def test_blocks(n, below, kind, ans, flat):
    x = _source(kind, n, below)
    s = O.encode(x, n, ans_mode=ans, flat=flat)
    # the root's leaf is the frequent symbol, unless it is no more than the rest
    # together; past the limit the block decodes tile by tile
    assert _lengths(s)[200] == 1 or 2 * below >= n
    print("case", n, below, kind, ans, flat, "allowed", _allowed(s, n, 5), flush=True)
    assert _allowed(s, n, 5) or kind == "many" and below > n // 3
    _check(x, [torch.from_numpy(s).cuda()] * 5)


@pytest.mark.parametrize("below", [1, 30, 5000])
def test_small_rests(below):
    x = _source("many", 60_000, below)
    s = O.encode(x, x.size, ans_mode=0)
    assert _lengths(s)[200] == 1 and _allowed(s, x.size, 5)
    _check(x, [torch.from_numpy(s).cuda()] * 5)


@pytest.mark.parametrize("ans,flat", [(0, False), (1, True), (3, False)])
@pytest.mark.parametrize("n,below", [(65_537, 9000), (131_072, 13_107), (131_071, T), (131_072, T + 1)])
def test_long_blocks_left_whole(n, below, ans, flat):
    """Blocks of more than 64 Ki symbols stay whole in a batch of many."""
    x = _source("four", n, below)
    s = O.encode(x, n, ans_mode=ans, flat=flat)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    copies = 2 * cus + 3
    assert _lengths(s)[200] == 1 and _allowed(s, n, copies)
    print("case", n, below, ans, flat, copies, flush=True)
    _check(x, [torch.from_numpy(s).cuda()] * copies, entries=("batch",))


def test_half_of_the_blocks():
    """Batches around half of the symbols in blocks that are merged once."""
    a = _source("four", 65_536, 9000)
    b = np.random.default_rng(3).integers(0, 4, size=65_536).astype(np.uint8)     # 2 bits, half below the root
    sa, sb = (torch.from_numpy(O.encode(x, x.size)).cuda() for x in (a, b))
    for k in (0, 3, 4, 5, 8):
        streams = [sa] * k + [sb] * (8 - k)
        outs = [torch.empty(65_536, dtype=torch.uint8, device="cuda") for _ in streams]
        _, st = P.pivco_decode_batch(streams, outs)
        assert (st == 0).all()
        for i, o in enumerate(outs):
            assert np.array_equal(o.cpu().numpy(), a if i < k else b), (k, i)


@pytest.mark.parametrize("ans", [0, 1])
def test_bit_flips_as_the_oracle_decides(ans):
    r = np.random.default_rng(6)
    x = _source("many", 50_000, 9000)
    good = O.encode(x, x.size, ans_mode=ans)
    assert _allowed(good, x.size, 81)
    streams, want = [torch.from_numpy(good).cuda()], [x]
    for _ in range(80):
        b = good.copy()
        p = int(r.integers(100, len(good)))
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
