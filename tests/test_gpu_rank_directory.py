"""The rank directory of a resident block: bodies whose superblocks of 256 bits
end at, before and after the threads' shares (one superblock a thread up to 32
KiB of body with 1024 threads, two above; up to four with 512), and the smallest;
the decode returns the input of the oracle's stream, in every merge variant."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")


@pytest.mark.parametrize("n", [1, 33, 8191, 16_000, 16_384, 32_000, 32_600, 32_768, 33_000, 47_900, 55_000, 57_344])
def test_body_sizes(n):
    r = np.random.default_rng(n)
    xs = [r.integers(0, 256, size=n).astype(np.uint8),               # 8 bits a symbol: body of about n bytes
          np.minimum(r.geometric(0.2, size=n), 255).astype(np.uint8)]
    streams = [torch.from_numpy(O.encode(x, n)).cuda() for x in xs]
    for v in range(len(P.pivco_merge_variants())):
        print("variant", v, n, flush=True)
        outs = [torch.full((n,), 0xAB, dtype=torch.uint8, device="cuda") for _ in xs]
        plan = P.BatchPlan(streams, outs, tune=P.Tune(v, 8, 8, 0))
        plan.launch()
        assert (plan.statuses() == 0).all()
        for x, o in zip(xs, outs):
            assert np.array_equal(o.cpu().numpy(), x)
        plan.close()
