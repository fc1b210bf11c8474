"""The encode workspace never shrinks as the input grows (one sized for the
longest input of a program serves the shorter ones), in particular where the
encoder goes over to larger slices (8 MiB)."""
import pytest

P = pytest.importorskip("paper_2606_05765_amd.pivco")

NS = [1, 63, 4096, 4097, 8191, 8192, 65_536, 1 << 20, (8 << 20) - 4097, (8 << 20) - 1, 8 << 20, (8 << 20) + 1, 9 << 20,
      64 << 20]


@pytest.mark.parametrize("ans", [0, 1, 3])
@pytest.mark.parametrize("bs", [4096, 8191, 8192, 65_536, 1 << 20, 16 << 20, 1 << 30])
def test_grows_with_n(bs, ans):
    w = [P.pivco_encode_workspace(n, bs, ans_mode=ans) for n in NS]
    assert all(a <= b for a, b in zip(w, w[1:]))


@pytest.mark.parametrize("bs", [1, 64, 8191, 8192, 8193, 65_536, 16 << 20])
def test_golomb_grows_with_n(bs):
    f = P.lib().pivco_golomb_encode_workspace
    w = [f(n, bs) for n in NS]
    assert all(a <= b for a, b in zip(w, w[1:]))
