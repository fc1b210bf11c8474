"""PivCo-Golomb decode on both sides of the rule for the workgroup's size (1024
threads and tiles of 16384 values up to 512 blocks in the call, 512 threads and
tiles of 8192 above): block sizes at the edges of both tiles, short codes, long ones
(levels wider than a wave far down), one long code among zeros; corrupt streams
get the oracle's verdict."""
import struct

import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")


def _values(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "short":
        return np.minimum(rng.geometric(0.5, size=n) - 1, 255).astype(np.uint8)
    if kind == "long":
        return rng.integers(0, 256, size=n).astype(np.uint8)
    if kind == "deep":                         # every level but the last as wide as the block
        return np.full(n, 255, np.uint8)
    x = np.zeros(n, np.uint8)
    x[n // 2] = 255
    return x


@pytest.mark.parametrize("kind", ["short", "long", "deep", "spike"])
@pytest.mark.parametrize("bs", [1, 63, 1023, 1025, 8191, 8192, 8193, 16_383, 16_384, 16_385, 24_577, 32_769])
def test_block_sizes(bs, kind):
    x = _values(kind, bs, bs)
    s = torch.from_numpy(O.golomb_encode(x, bs)).cuda()
    tiny = torch.from_numpy(O.golomb_encode(np.zeros(512, np.uint8), 1)).cuda()    # 512 blocks more
    for streams, sizes in (([s], [x.size]), ([s, tiny], [x.size, 512])):
        print("case", kind, bs, len(streams), flush=True)
        outs = [torch.full((n + 16,), 0xAB, dtype=torch.uint8, device="cuda") for n in sizes]
        _, st = P.pivco_golomb_decode(streams, [o[:n] for o, n in zip(outs, sizes)])
        assert (st == 0).all()
        got = outs[0].cpu().numpy()
        assert np.array_equal(got[:bs], x) and (got[bs:] == 0xAB).all()


@pytest.mark.parametrize("blocks", [511, 512, 513])
def test_at_the_rule(blocks):
    x = _values("short", 300 * blocks - 7, blocks)
    s = torch.from_numpy(O.golomb_encode(x, 300)).cuda()
    out = torch.empty(x.size, dtype=torch.uint8, device="cuda")
    _, st = P.pivco_golomb_decode([s], [out])
    assert st[0] == 0 and np.array_equal(out.cpu().numpy(), x)


def _padding(stream):
    """The stream's bits that no bitmap holds, one mask a byte (the decoder does
    not read them; the oracle asks for zeros)."""
    off = struct.unpack_from("<Q", stream, 32)[0]
    comp, n, K = struct.unpack_from("<IIH", stream, off)
    at = off + 12 + 4 * (K - 1)
    mask = np.zeros(len(stream), np.uint8)
    mask[off + comp:] = 0xFF
    for nk in [n] + list(struct.unpack_from(f"<{K - 1}I", stream, off + 12)):
        at += (nk + 7) // 8
        if nk % 8:
            mask[at - 1] = 0xFF << (nk % 8) & 0xFF
    return mask


@pytest.mark.parametrize("kind", ["short", "long"])
@pytest.mark.parametrize("many", [False, True])
def test_bit_flips_as_the_oracle_decides(kind, many):
    r = np.random.default_rng(5)
    x = _values(kind, 17_000, 5)
    good = O.golomb_encode(x, x.size)
    pad = _padding(good)
    streams, want = [torch.from_numpy(good).cuda()], [x]
    for _ in range(600 if many else 60):
        b = good.copy()
        p = int(r.integers(48, len(good)))
        bit = 1 << int(r.integers(0, 8))
        b[p] ^= np.uint8(bit)
        try:
            want.append(O.golomb_decode(b, n=x.size))
        except O.OracleError:
            want.append(x if pad[p] & bit else None)
        streams.append(torch.from_numpy(b).cuda())
    print("case", kind, many, len(streams), flush=True)
    outs = [torch.empty(x.size, dtype=torch.uint8, device="cuda") for _ in streams]
    outs, st = P.pivco_golomb_decode(streams, outs)
    for i, w in enumerate(want):
        assert (st[i] == 0) == (w is not None), i
        if w is not None:
            assert np.array_equal(outs[i].cpu().numpy(), w), i
