"""The plan kernel's walk over a block's entropy-coded bodies, which checks 64
bodies at a time: blocks of 1..255 of them around that number, and one field of
one body wrong (probability or table, zero bytes, length, chunk length) in the
first, the last and around the 64th.  The verdict is the oracle's and the
sound streams of the same batch decode to their input."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")

BLOCK0 = 48 + 16 * 2                       # one block: the header and two entries of each table


def _bodies(s, n_internal, count_width):
    """Offsets of the bodies of a one-block stream without raw ones."""
    comp = int(s[BLOCK0:BLOCK0 + 4].view(np.uint32)[0])
    o = 140 + (n_internal + 7) // 8 + count_width * n_internal
    at = []
    while o < comp:
        o = (o + 3) & ~3
        at.append(BLOCK0 + o)
        o += 8 + int(s[BLOCK0 + o + 4:BLOCK0 + o + 8].view(np.uint32)[0])
    return at


def _mutants(s, at, chunk_len):
    for j in sorted({0, 62, 63, 64, 65, len(at) - 1}):
        if j >= len(at):
            continue
        for off, add in ((0, 255), (2, 1), (4, 4), (4, -4), (chunk_len, 1)):
            x = s.copy()
            x[at[j] + off] = (int(x[at[j] + off]) + add) & 255
            yield (j, off, add), x


def _check(good, data, at, chunk_len):
    muts = list(_mutants(good, at, chunk_len))
    all_s = [good] + [x for _, x in muts] + [good]
    outs = [torch.empty(data.size, dtype=torch.uint8, device="cuda") for _ in all_s]
    got, status = P.pivco_decode_batch([torch.from_numpy(x).cuda() for x in all_s], outs)
    torch.cuda.synchronize()
    for i in (0, -1):
        assert status[i] == 0 and np.array_equal(got[i].cpu().numpy(), data)
    for (what, x), st, o in zip(muts, status[1:-1], got[1:-1]):
        try:
            want = O.decode(x)
        except O.OracleError:
            assert st != 0, what
            continue
        assert st == 0 and np.array_equal(o.cpu().numpy(), want), what


@pytest.mark.parametrize("chunk_log2", [5, 16])
@pytest.mark.parametrize("nodes", [1, 2, 63, 64, 65, 127, 128, 129, 255])
def test_rans_bodies(nodes, chunk_log2):
    r = np.random.default_rng(nodes)
    m = nodes + 1
    x = r.permutation(np.repeat(np.arange(m, dtype=np.uint8), r.integers(1, 40, m)))
    s = O.encode(x, x.size, ans_mode=2, chunk_log2=chunk_log2)
    info = O.block_info(s, 0)
    assert info["n_internal"] == nodes and info["kind"].all()
    print("case", nodes, chunk_log2, flush=True)
    _check(s, x, _bodies(s, nodes, 2 if x.size <= 65535 else 4), 8)


def test_tans_bodies():
    r = np.random.default_rng(7)
    x = np.zeros(4_200_000, np.uint8)
    for i in range(8):                     # biased bits: most nodes of the upper 7 levels are coded
        x |= (r.random(x.size) < 0.15).astype(np.uint8) << i
    s = O.encode(x, x.size, ans_mode=3, tree_len=np.full(256, 8, np.uint8))
    kind = O.block_info(s, 0)["kind"].astype(bool)
    assert kind.sum() > 65
    t = torch.from_numpy(s).cuda()
    print("case tans", int(kind.sum()), flush=True)
    bad = s.copy()
    bad[-9] ^= 1                           # inside the last body
    out = torch.empty(x.size, dtype=torch.uint8, device="cuda")
    got, status = P.pivco_decode_batch([torch.from_numpy(bad).cuda(), t], [out, torch.empty_like(out)])
    torch.cuda.synchronize()
    assert status[1] == 0 and np.array_equal(got[1].cpu().numpy(), x)
    try:
        want = O.decode(bad)
    except O.OracleError:
        assert status[0] != 0
    else:
        assert status[0] == 0 and np.array_equal(got[0].cpu().numpy(), want)
