"""A workspace that was enough for an encode stays enough: the encoder asks for no
more, for any input size, block size and options, than its first layout did
(below: the areas' sizes, each at a multiple of 256 bytes)."""
import pytest

P = pytest.importorskip("paper_2606_05765_amd.pivco")

NS = [0, 1, 100, 4096, 5000, 65_536, 100_000, 1 << 20, (8 << 20) - 1, 8 << 20, 64 << 20, (1 << 30) + 7]


def _first_layout(n, bs, max_len, ans, chunk_log2):
    nb, spb = -(-n // bs), -(-bs // 4096)
    bits = n * max_len
    chunks = (bits >> chunk_log2) + nb * 255 + 1 if ans else 0
    areas = [nb * 1024 + 16, nb * spb * 1024 + 16, nb * 256 + 16, nb * 4 + 16,      # counts, rows, lengths, modes
             nb * 3520, nb * 88, nb * 255 * 32 if ans else 0, nb * 1216,            # codes, layouts, nodes, headers
             bits // 8 + nb * 287 + 64, (4 * (bits // 32 + nb * 259) if ans else 0) + 64,   # images, bitmaps
             chunks * 40, chunks * 4, (2 * bits + chunks * 160 if ans else 0) + 64, 64, 64]
    total = 0
    for a in areas:
        total = (total + a + 255) // 256 * 256
    return total


@pytest.mark.parametrize("ans", [0, 1, 2, 3])
@pytest.mark.parametrize("bs", [1, 64, 1000, 4096, 8192, 8193, 65_536, 1 << 20, 1 << 30])
def test_no_more_than_the_first_layout(bs, ans):
    for n in NS:
        for max_len in (1, 8, 11, 12):
            for chunk_log2 in (8, 16, 24):
                got = P.pivco_encode_workspace(n, bs, max_len=max_len, ans_mode=ans, chunk_log2=chunk_log2)
                assert got <= _first_layout(n, bs, max_len, ans, chunk_log2), (n, max_len, chunk_log2)
