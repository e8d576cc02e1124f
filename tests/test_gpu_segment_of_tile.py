"""The segment a tile finds for itself, at segment counts around a launch's 32, with
segments of no, one and several tiles and one set of hyperparameters per neighbour."""
import numpy as np
import pytest

import oracle
from tests.helpers import make_shard, o_hyper
import workloads as wl

pytestmark = pytest.mark.gpu

HYPERS = [dict(wl.DEFAULT_HYPER, lr=lr) for lr in (1e-3, 3e-4, 2e-5)]


@pytest.mark.parametrize("count", [1, 2, 31, 32, 33, 63, 64, 65])
def test_every_segment_gets_its_own_scalars(count):
    import paper_2609_18178_amd as pk

    lengths = [(0, 1, 1024, 1500, 4096 + 3, 7)[k * 5 % 6] for k in range(count)]
    segs, off = [], 0
    for k, ln in enumerate(lengths):
        segs.append((off, ln, k % 3))
        off += ln + k % 2
    n = off + 1
    rng = np.random.default_rng(count)
    p, g, m = (rng.standard_normal(n).astype(np.float32) for _ in range(3))
    v = np.abs(rng.standard_normal(n)).astype(np.float32)
    sh = make_shard(p, g, m, v, 31, segments=segs, hypers=HYPERS)
    b = np.zeros(n, np.uint16)
    per, total = oracle.commit_segments(p, g, m, v, b, segs, [o_hyper(h) for h in HYPERS], 3, 31)
    assert pk.to_u64(pk.adamw_commit(sh, 3)) == per + [total]
    assert np.array_equal(sh.param.cpu().numpy().view(np.uint32), p.view(np.uint32))
    assert pk.to_u64(pk.shard_digest(sh)) == per + [total]
