"""The autotuner's cached choice is for one kind of batch: batches of the same
shape that are not skewed, whose sizes alone allow it, and that are skewed run
different merge kernels and are timed each for itself (a timing decodes the
batch, a cached choice leaves the outputs alone)."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")

N = 65_536


def _batch(kind):
    r = np.random.default_rng(7)
    if kind == "plain":                        # 5 bits a symbol
        x = r.integers(0, 32, size=N).astype(np.uint8)
    elif kind == "few bits":                   # 2 bits, half of them below the root
        x = r.integers(0, 4, size=N).astype(np.uint8)
    else:                                      # 0.95 in one symbol
        x = np.where(r.random(N) < 0.95, 7, r.integers(0, 4, size=N)).astype(np.uint8)
    return x, [torch.from_numpy(O.encode(x, N)).cuda()] * 8


@pytest.mark.parametrize("order", [("plain", "few bits", "skewed"), ("skewed", "few bits", "plain")])
def test_each_kind_is_timed(order):
    P.pivco_autotune_cache_clear()
    for timed in (True, False):
        for kind in order:
            print("case", kind, timed, flush=True)
            x, streams = _batch(kind)
            outs = [torch.full((N,), 0xAB, dtype=torch.uint8, device="cuda") for _ in streams]
            tune = P.pivco_autotune(streams, outs)
            torch.cuda.synchronize()
            for o in outs:
                if timed:
                    assert np.array_equal(o.cpu().numpy(), x), kind
                else:
                    assert (o == 0xAB).all(), kind
            plan = P.BatchPlan(streams, outs, tune=tune)
            plan.launch()
            assert (plan.statuses() == 0).all()
            for o in outs:
                assert np.array_equal(o.cpu().numpy(), x), kind
            plan.close()
    P.pivco_autotune_cache_clear()
