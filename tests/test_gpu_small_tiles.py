"""Window starts of a tile's levels: up to 16384 symbols the nodes enter them,
above that a wave per level finds them.  Tiles on both sides of the line, as whole
blocks, as the last tile of whole and of split blocks, with few large nodes and
with many small ones, for every merge variant (each starts its tiles elsewhere);
the decode returns the input of the oracle's stream."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")

SIZES = [1, 1024, 1025, 4096, 16_383, 16_384, 16_385, 32_768, 32_768 + 16_384, 32_768 + 16_385, 65_536,
         3 * 32_768 + 16_384, 3 * 32_768 + 16_385]


def _source(kind, n):
    r = np.random.default_rng(n)
    if kind == "many":                         # 255 internal nodes
        return r.integers(0, 256, size=n).astype(np.uint8)
    return np.minimum(r.geometric(0.45, size=n), 255).astype(np.uint8)


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("kind", ["few", "many"])
def test_sizes(kind, flat):
    xs = [_source(kind, n) for n in SIZES]
    streams = [torch.from_numpy(O.encode(x, x.size, flat=flat)).cuda() for x in xs]
    for v in range(len(P.pivco_merge_variants())):
        print("variant", v, kind, flat, flush=True)
        outs = [torch.full((x.size,), 0xAB, dtype=torch.uint8, device="cuda") for x in xs]
        plan = P.BatchPlan(streams, outs, tune=P.Tune(v, 8, 8, 0))
        plan.launch()
        assert (plan.statuses() == 0).all()
        for x, o in zip(xs, outs):
            assert np.array_equal(o.cpu().numpy(), x)
        plan.close()
