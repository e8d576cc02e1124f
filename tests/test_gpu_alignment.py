"""Every head, tail and misalignment that a segment can have around the vector
path, in every entry point: segments that start 0-7 elements behind an aligned
one and end anywhere in a row, a vector or a tile, among neighbours whose
elements and gaps must stay as they are.  Everything compares bit for bit."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.helpers import assert_bitwise, g_hyper, host, o_hyper

pytestmark = pytest.mark.gpu

H = wl.DEFAULT_HYPER
# below a vector, around a vector, a row of 4- and 8-element vectors, a tile, two tiles
LENGTHS = [1, 2, 3, 4, 5, 7, 8, 9, 15, 17, 1023, 1024, 1025, 1029, 2047, 2049, 2056, 3079, 4095, 4096, 4097, 4101, 4103, 5120,
           8191, 8192, 8200, 16385, 32771]


def _pk():
    import paper_2609_18178_amd as pk

    return pk


def _table(shift, lead=0):
    """Segments of all LENGTHS, behind one of `lead` elements if any; segment k starts
    `shift` + k elements (mod 8) behind an aligned element, with a gap of at least one
    before it."""
    segs, off = [(0, lead, 0)] if lead else [], lead
    for k, ln in enumerate(LENGTHS):
        off = (off + 8) // 8 * 8 + (shift + k) % 8
        segs.append((off, ln, 0))
        off += ln
    return segs, off + 3


def _arrays(n, bases, dtype):
    """Five device arrays whose first elements lie bases[k] elements behind an
    aligned address, inside buffers whose other elements are 7, host copies of
    the first four, and the buffers."""
    import torch

    rng = np.random.default_rng(n + sum(bases))
    hosts = [(rng.standard_normal(n) * s).astype(np.float32) for s in (0.02, 1e-3, 1e-4, 1e-7)]
    hosts[3] = np.abs(hosts[3])
    if dtype == torch.int16:
        hosts = [torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16) for x in hosts]
    whole = [torch.full((n + 16,), 7, dtype=dtype if k < 4 else torch.int16, device="cuda") for k in range(5)]
    dev = [w[b:b + n] for w, b in zip(whole, bases)]
    for t, x in zip(dev, hosts):
        t.copy_(torch.from_numpy(x.view(np.int16) if dtype == torch.int16 else x))
    dev[4].zero_()
    return hosts, dev, whole


def _margins_untouched(whole, bases, n):
    for w, b in zip(whole, bases):
        assert bool((w[:b] == 7).all()) and bool((w[b + n:] == 7).all())


# aligned together at every 4th element; at none (grad against the others; the copy against the fp32 arrays)
BASES = {"together": (0, 0, 0, 0, 0), "shifted": (3, 3, 3, 3, 3), "grad apart": (0, 1, 0, 0, 0), "copy apart": (0, 0, 0, 0, 2)}


def _check_binary32(bases, shift, goff, lead=0, use_workspace=True):
    import torch

    pk = _pk()
    segs, n = _table(shift, lead)
    (p, g, m, v), dev, whole = _arrays(n, BASES[bases], torch.float32)
    sh = pk.Shard(*dev, goff, segments=segs, hypers=[g_hyper(H)], use_workspace=use_workspace)
    per, total = oracle.segment_digests(p, m, v, segs, goff)
    assert pk.to_u64(pk.shard_digest(sh)) == per + [total]
    counts = [int(np.count_nonzero(g[o:o + ln].view(np.uint32))) for o, ln, _ in segs]
    assert pk.to_u64(pk.grad_guard(sh)) == counts + [sum(counts)]
    b = np.zeros(n, np.uint16)
    for step, zero in ((4, False), (5, True)):
        per, total = oracle.commit_segments(p, g, m, v, b, segs, [o_hyper(H)], step, goff)
        assert pk.to_u64(pk.adamw_commit(sh, step, zero_grad=zero)) == per + [total]
        for name, want in (("param", p), ("exp_avg", m), ("exp_avg_sq", v), ("param_bf16", b)):
            got = host(getattr(sh, name))
            assert_bitwise(name, got.view(np.uint16) if name == "param_bf16" else got, want)
    want = [oracle.bf16_digest(b[o:o + ln], goff + o) for o, ln, _ in segs]
    assert pk.to_u64(pk.bf16_digest(sh))[:-1] == want
    left = g.copy()
    for o, ln, _ in segs:
        left[o:o + ln] = 0.0
    assert_bitwise("grad", host(sh.grad), left)
    _margins_untouched(whole, BASES[bases], n)


def _check_bf16_state(bases, shift, goff, lead=0, use_workspace=True):
    import torch

    pk = _pk()
    segs, n = _table(shift, lead)
    (p, g, m, v), dev, whole = _arrays(n, BASES[bases], torch.int16)
    sh = pk.ShardBf16(*dev[:4], goff, segments=segs, hypers=[g_hyper(H)], use_workspace=use_workspace)
    want = [oracle.state_digest_bf16(p[o:o + ln], m[o:o + ln], v[o:o + ln], goff + o) for o, ln, _ in segs]
    assert pk.to_u64(pk.shard_digest_bf16(sh))[:-1] == want
    want = [oracle.commit_and_digest_bf16(p[o:o + ln], g[o:o + ln], m[o:o + ln], v[o:o + ln], o_hyper(H), 6, goff + o)
            for o, ln, _ in segs]
    assert pk.to_u64(pk.adamw_commit_bf16(sh, 6))[:-1] == want
    for name, ref in (("param", p), ("exp_avg", m), ("exp_avg_sq", v)):
        assert_bitwise(name, host(getattr(sh, name)).view(np.uint16), ref)
    _margins_untouched(whole, BASES[bases], n)


@pytest.mark.parametrize("bases", list(BASES))
@pytest.mark.parametrize("shift", [0, 1, 6])
@pytest.mark.parametrize("goff", [5, (1 << 32) - 9000])
def test_binary32_segments(bases, shift, goff):
    _check_binary32(bases, shift, goff)


@pytest.mark.parametrize("bases", ["together", "shifted", "grad apart"])
@pytest.mark.parametrize("shift", [0, 3, 7])
@pytest.mark.parametrize("goff", [5, (1 << 16) - 300])
def test_bf16_state_segments(bases, shift, goff):
    _check_bf16_state(bases, shift, goff)


@pytest.mark.parametrize("bases", list(BASES))
@pytest.mark.parametrize("shift", [0, 5])
def test_without_a_workspace(bases, shift):
    """The kernels of calls without a workspace: longer tiles, whose shares go straight
    to the result slots."""
    _check_binary32(bases, shift, (1 << 32) - 9000, use_workspace=False)
    if bases != "copy apart":
        _check_bf16_state(bases, shift, (1 << 16) - 300, use_workspace=False)
