"""How a batch's lists reach the device: as kernel arguments or as copies,
by their size.  Batches on both sides of each limit, with jobs in error among
them, decode to the inputs and report every job's own status."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")


@pytest.mark.parametrize("count", [1, 2, 20, 26, 27, 28, 29, 30, 31, 32, 255, 256, 257, 300])
def test_batches_of_small_streams(count):
    rng = np.random.default_rng(count)
    xs = [rng.integers(0, int(rng.integers(2, 60)), size=int(rng.integers(1, 900))).astype(np.uint8) for _ in range(count)]
    streams, outs, want = [], [], []
    for i, x in enumerate(xs):
        s = O.encode(x, 1024, ans_mode=i % 2)
        st = 0
        if i % 7 == 3:                       # another magic number
            s = s.copy()
            s[0] ^= 1
            st = P.E_CORRUPT
        n = x.size
        if i % 11 == 5 and st == 0:          # no room for the output
            n -= 1
            st = P.E_CAPACITY
        streams.append(torch.from_numpy(s).cuda())
        outs.append(torch.full((max(n, 1),), 0xAB, dtype=torch.uint8, device="cuda")[:n])
        want.append(st)
    ws = P.Workspace(P.pivco_decode_workspace(streams, outs))
    outs, st = P.pivco_decode_batch(streams, outs, ws=ws)
    assert st.tolist() == want
    for x, o, w in zip(xs, outs, want):
        if w == 0:
            assert np.array_equal(o.cpu().numpy(), x)


@pytest.mark.parametrize("count", [1, 2, 47, 48, 49, 120])
def test_golomb_batches(count):
    rng = np.random.default_rng(count)
    xs = [np.minimum(rng.geometric(0.5, size=int(rng.integers(0, 900))) - 1, 255).astype(np.uint8) for _ in range(count)]
    streams, outs, want = [], [], []
    for i, x in enumerate(xs):
        s = O.golomb_encode(x, 256)
        st = 0
        if i % 5 == 2:
            s = s.copy()
            s[0] ^= 1
            st = P.E_CORRUPT
        streams.append(torch.from_numpy(s).cuda())
        outs.append(torch.full((max(x.size, 1),), 0xAB, dtype=torch.uint8, device="cuda")[:x.size])
        want.append(st)
    outs, st = P.pivco_golomb_decode(streams, outs)
    assert st.tolist() == want
    for x, o, w in zip(xs, outs, want):
        if w == 0:
            assert np.array_equal(o.cpu().numpy(), x)
