"""The kernels that large shards take, on the segments where they can go wrong: ragged and
unaligned ones behind one segment long enough to lift the call into them (the same segments
alone would take the kernels of small shards).  Everything compares bit for bit."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
from tests.helpers import M64, host_threads, to_device
from tests.test_gpu_alignment import _table

pytestmark = pytest.mark.gpu

# around the passes of a tile (4096 elements each)
MORE = [3 * 4096, 4 * 4096 - 1, 4 * 4096, 4 * 4096 + 1, 7 * 4096 + 1029, 8 * 4096]


def _pk():
    import paper_2609_18178_amd as pk

    return pk


def _segments(shift, lead):
    segs, off = _table(shift, lead)
    for k, ln in enumerate(MORE):
        off = (off + 8) // 8 * 8 + (shift + k) % 8
        segs.append((off, ln, 0))
        off += ln
    return segs, off + 5


def _bits(n, dtype, odd):
    """n words of any pattern."""
    x = np.arange(n, dtype=np.uint32)
    x *= np.uint32(odd)
    return x if dtype == np.uint32 else (x >> np.uint32(16)).astype(np.uint16)


def _digests(digest, segs, goff):
    """digest(first, end, index) of every segment, long ones cut over host threads."""
    cuts = [(o + ln * k // t, o + ln * (k + 1) // t, s) for s, (o, ln, _) in enumerate(segs)
            for t in [host_threads() if ln > 1 << 20 else 1] for k in range(t)]
    per = [0] * len(segs)
    with ThreadPoolExecutor(host_threads()) as ex:
        for (_, _, s), d in zip(cuts, ex.map(lambda c: digest(c[0], c[1], goff + c[0]), cuts)):
            per[s] = (per[s] + d) & M64
    return per + [sum(per) & M64]


@pytest.mark.parametrize("shift", [0, 3])
def test_long_tiles_of_the_state_digest(shift):
    """From 402,653,184 elements on the tiles have four passes."""
    pk = _pk()
    segs, n = _segments(shift, 3 << 27)
    goff = (1 << 32) - 3 * 4096 - 5 - segs[5][0]  # the indices cross 2^32 among the short segments
    p, m, v = (_bits(n, np.uint32, odd).view(np.float32) for odd in (0x9E3779B1, 0x85EBCA77, 0xC2B2AE3D))
    tp, tm, tv = to_device(p, m, v)
    sh = pk.Shard(tp, None, tm, tv, None, goff, segments=segs, hypers=[pk.Hyper()])
    want = _digests(lambda a, z, first: oracle.state_digest(p[a:z], m[a:z], v[a:z], first), segs, goff)
    for _ in range(2):
        assert pk.to_u64(pk.shard_digest(sh)) == want
