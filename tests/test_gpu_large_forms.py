"""The kernels that large shards take, on the segments where they can go wrong: ragged and
unaligned ones behind one segment long enough to lift the call into them (the same segments
alone would take the kernels of small shards).  Everything compares bit for bit."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
import workloads as wl
from tests.helpers import M64, assert_bitwise, g_hyper, host, host_threads, o_hyper, to_device
from tests.test_gpu_alignment import _check_binary32, _check_bf16_state, _table

pytestmark = pytest.mark.gpu

H = wl.DEFAULT_HYPER

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


@pytest.mark.parametrize("bases,shift,goff", [("together", 0, 5), ("together", 6, (1 << 32) - 9000 - (4 << 20)),
                                              ("shifted", 1, 5), ("grad apart", 6, 5), ("copy apart", 1, 5)])
def test_binary32_segments_behind_a_long_one(bases, shift, goff):
    """The state digest's usual kernel (from 3M elements on), and the others' with it."""
    _check_binary32(bases, shift, goff, lead=4 << 20)


@pytest.mark.parametrize("bases,shift,goff", [("together", 0, 5), ("together", 3, (1 << 32) - 300 - (17 << 20)),
                                              ("shifted", 7, (1 << 16) - 300), ("grad apart", 3, 5)])
def test_bf16_state_segments_behind_a_long_one(bases, shift, goff):
    """The usual kernels of BF16 state: the commit's from 16M elements on, the digest's from 1.5M."""
    _check_bf16_state(bases, shift, goff, lead=17 << 20)


@pytest.mark.parametrize("shift", [0, 3])
@pytest.mark.parametrize("lead", [0, 2 << 20, 68 << 20, 136 << 20])
def test_sixteen_bit_digests_of_one_two_and_four_passes(lead, shift):
    """One pass a tile, two from 64M elements on, four from 128M; at a base whose indices
    pass the words where the short index form does not apply."""
    import torch

    pk = _pk()
    segs, n = _segments(shift, lead)
    goff = (5 << 32) + 0x40B50000 - 4096 - segs[1][0]
    p, m, v = (_bits(n, np.uint16, odd) for odd in (0x9E3779B1, 0x85EBCA77, 0xC2B2AE3D))
    tp, tm, tv = to_device(*(x.view(np.int16) for x in (p, m, v)))
    sh = pk.ShardBf16(tp, None, tm, tv, goff, segments=segs, hypers=[pk.Hyper()])
    want = _digests(lambda a, z, first: oracle.state_digest_bf16(p[a:z], m[a:z], v[a:z], first), segs, goff)
    for _ in range(2):
        assert pk.to_u64(pk.shard_digest_bf16(sh)) == want
    f = torch.empty(n, device="cuda")
    sh = pk.Shard(f, None, f, f, tp, goff, segments=segs, hypers=[pk.Hyper()])
    want = _digests(lambda a, z, first: oracle.bf16_digest(p[a:z], first), segs, goff)
    for _ in range(2):
        assert pk.to_u64(pk.bf16_digest(sh)) == want


def _bf16_commit(p, g, m, v, hyper, step, goff):
    """A commit of BF16 state by both sides: every output bitwise where the oracle gives a
    number, NaN where it gives one (the sign and payload of a NaN made by an invalid
    operation are not part of the contract), and the digest of the GPU's own words."""
    pk = _pk()
    t = to_device(*(x.view(np.int16).copy() for x in (p, g, m, v)))
    sh = pk.ShardBf16(*t, goff)
    got = pk.to_u64(pk.adamw_commit_bf16(sh, step, g_hyper(hyper)))
    cuts = [p.size * k // host_threads() for k in range(host_threads() + 1)]

    def part(k):
        s = slice(cuts[k], cuts[k + 1])
        oracle.adamw_commit_bf16(p[s], g[s], m[s], v[s], o_hyper(hyper), step)
        return oracle.state_digest_bf16(*(x[s] for x in out), goff + cuts[k])

    out = [host(x).view(np.uint16) for x in (sh.param, sh.exp_avg, sh.exp_avg_sq)]
    with ThreadPoolExecutor(host_threads()) as ex:
        want = sum(ex.map(part, range(host_threads()))) & M64
    for name, mine, ref in zip(("param", "exp_avg", "exp_avg_sq"), out, (p, m, v)):
        nan = [(x & 0x7FFF) > 0x7F80 for x in (mine, ref)]
        assert np.array_equal(*nan), name
        assert_bitwise(name, np.where(nan[1], 0, mine).astype(np.uint16), np.where(nan[1], 0, ref).astype(np.uint16))
    assert got == [want]
    assert pk.to_u64(pk.shard_digest_bf16(sh)) == [want]


@pytest.fixture(scope="module")
def bf16_state():
    """(p, g, m, v) of training's distribution, more than the BF16 commit's small kernel takes,
    and the first elements of its tiles from the middle on."""
    n = (16 << 20) + 64 * 4096 + 77
    w = wl.WORKLOADS["mistral7b_shard16"]
    few = [oracle.bf16_rne_bits(a.view(np.uint32)) for a in wl.arrays_host(w, 0, 1 << 20)]
    return [np.resize(a, n) for a in few], [(8 << 20) + k * 4096 for k in range(64)]


def test_large_bf16_commit_at_edge_operands(bf16_state):
    """Operands at the edges of the bracketed step's ranges, one in each wave of a tile, in the
    commit's usual kernel: m' and v' at powers of two and zeros (with beta1 = beta2 = 1/2 and
    g = 0 a planted m or v is halved exactly), weights from zero to the largest, NaNs and
    infinities; then eps and step sizes on both sides of their limits."""
    (p0, g0, m0, v0), tiles = bf16_state
    p, g, m, v = (a.copy() for a in (p0, g0, m0, v0))
    plants = [  # (array, word): m', v' of half the value
        (m, 0x2080), (m, 0x207F), (m, 0xA080), (m, 0x4080), (m, 0x8000), (m, 0x0000), (m, 0x0001), (m, 0x7F7F),
        (v, 0x0000), (v, 0x1080), (v, 0x107F), (v, 0x1000), (v, 0x0FFF), (v, 0x0001), (v, 0x5FFF), (v, 0x7F7F),
        (v, 0x7F80), (v, 0xBF80), (m, 0x7F80), (m, 0x7FC1), (p, 0x0000), (p, 0x8000), (p, 0x2680), (p, 0x267F),
        (p, 0x497F), (p, 0x4980), (p, 0x7F7F), (p, 0x7F80), (p, 0xFFC0), (p, 0x0001)]
    for tile, (array, word) in zip(tiles, plants):
        for wave in range(4):
            e = tile + wave * 512 + 9
            array[e], g[e] = word, 0
    _bf16_commit(p, g, m, v, dict(H, beta1=0.5, beta2=0.5), 3, 99)
    for h, step in ((dict(H, eps=2.0 ** 100), 3), (dict(H, eps=2.0 ** 101), 3), (dict(H, eps=2.0 ** -149), 3),
                    (dict(H, lr=2.0 ** -41, weight_decay=0.0, beta1=0.0), 1), (dict(H, lr=0.0), 3),
                    (dict(H, beta2=float(np.float32(1.0) - np.float32(2.0 ** -24))), 1)):
        _bf16_commit(*(a.copy() for a in bf16_state[0]), h, step, 99)
