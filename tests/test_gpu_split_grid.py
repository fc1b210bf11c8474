"""The encoder's split on both sides of its rule for the workgroup's size (1024
threads up to 256 slices of 4096 symbols in the call, 256 threads above), with the
slices in one block, in many, and in blocks that end inside a slice; the stream
equals the oracle's."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")

SLICE = 4096


@pytest.mark.parametrize("ans,flat", [(0, False), (0, True), (1, False), (3, True)])
@pytest.mark.parametrize("slices,bs", [(255, 255 * SLICE), (256, 256 * SLICE), (257, 257 * SLICE), (256, 16 * SLICE),
                                       (257, 16 * SLICE), (256, SLICE), (257, SLICE), (256, 2 * SLICE - 5),
                                       (258, 2 * SLICE - 5)])
def test_at_the_rule(slices, bs, ans, flat):
    r = np.random.default_rng(slices + bs)
    # the last slice is ragged; a block of 2 * SLICE - 5 symbols is two slices
    n = slices // 2 * bs if bs == 2 * SLICE - 5 else slices * SLICE - 7
    x = W.draw(r, W.zipf_p(1.2, r), n)
    print("case", slices, bs, ans, flat, flush=True)
    want = O.encode(x, bs, ans_mode=ans, flat=flat)
    got = P.pivco_encode(torch.from_numpy(x).cuda(), bs, ans_mode=ans, flat=flat)
    assert np.array_equal(got.cpu().numpy(), want)
