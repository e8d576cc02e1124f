"""The result slots, which the last tile of a call writes: tile counts on both
sides of the split into lanes, one and many segments (empty ones among them),
the call that follows a workspace written to behind the state's back, and calls
that change streams.  Digests are whole numbers and compare exactly."""
import ctypes

import numpy as np
import pytest

import oracle
from tests.helpers import M64, make_shard, o_hyper
import workloads as wl

pytestmark = pytest.mark.gpu

H = wl.DEFAULT_HYPER
T = 4096  # elements of a full tile


def _pk():
    import paper_2609_18178_amd as pk

    return pk


def _state(n, seed):
    rng = np.random.default_rng(seed)
    return ((rng.standard_normal(n) * 0.02).astype(np.float32), (rng.standard_normal(n) * 1e-3).astype(np.float32),
            (rng.standard_normal(n) * 1e-4).astype(np.float32), (np.abs(rng.standard_normal(n)) * 1e-7).astype(np.float32))


def _clear(sh):
    return int(sh.workspace.count_nonzero().item()) == 0


# tiles of T elements in the guard, and of T / 4 in the state digest up to 3M
@pytest.mark.parametrize("n", [0, 1, T, 63 * T // 4, 16 * T, 16 * T + 1, 65 * T // 4 + 5, 63 * T, 64 * T, 64 * T + 1, 65 * T + 5,
                               80 * T, 1040 * T + 17])
def test_flat_slot_at_every_tile_count(n):
    pk = _pk()
    p, g, m, v = _state(n, 1)
    sh = make_shard(p, g, m, v, 12345)
    want = oracle.state_digest(p, m, v, 12345) if n else 0
    for _ in range(3):  # both sets of nodes, and the first again
        assert pk.to_u64(pk.shard_digest(sh)) == [want]
        assert pk.to_u64(pk.grad_guard(sh)) == [int(np.count_nonzero(g.view(np.uint32)))]
        assert _clear(sh)


@pytest.mark.parametrize("lengths", [[0], [0, 0, 0], [5, 0, T], [64 * T, 64 * T + 1, 0, 1], [1] * 70, [T + 1] * 33 + [0, 90 * T]])
def test_segment_slots_and_total(lengths):
    pk = _pk()
    segs, off = [], 3
    for k, ln in enumerate(lengths):
        segs.append((off, ln, 0))
        off += ln + k % 3
    n = off + 2
    p, g, m, v = _state(n, 2)
    sh = make_shard(p, g, m, v, 99, segments=segs, hypers=[H])
    per, total = oracle.segment_digests(p, m, v, segs, 99)
    for _ in range(2):
        assert pk.to_u64(pk.shard_digest(sh)) == per + [total]
        assert _clear(sh)
    b = np.zeros(n, np.uint16)
    per, total = oracle.commit_segments(p, g, m, v, b, segs, [o_hyper(H)], 4, 99)
    assert pk.to_u64(pk.adamw_commit(sh, 4)) == per + [total] and total == sum(per) & M64
    assert _clear(sh)


@pytest.mark.parametrize("n", [3 * T + 7, 70 * T])
def test_call_after_a_workspace_that_was_not_clear(n):
    """A workspace written to while its state says clear costs the digest nothing, and
    neither does one that the caller says it has written to."""
    import torch

    pk = _pk()
    p, g, m, v = _state(n, 3)
    sh = make_shard(p, g, m, v, 7)
    want = [oracle.state_digest(p, m, v, 7)]
    for _ in range(2):  # from either set
        sh.workspace.copy_(torch.randint(1, 256, sh.workspace.shape, dtype=torch.uint8, device=sh.workspace.device))
        pk.shard_digest(sh)
        assert pk.to_u64(pk.shard_digest(sh)) == want
        assert pk.to_u64(pk.shard_digest(sh)) == want
    sh.workspace.fill_(0xA5)
    sh.workspace_clean = False
    assert pk.to_u64(pk.shard_digest(sh)) == want and sh.workspace_clean


@pytest.mark.parametrize("n", [3 * T + 7, 70 * T])
def test_commit_after_a_state_that_was_wrong(n):
    """A binary32 commit goes by its state: a workspace written to while that says clear costs
    one digest, from either set, and none of the arrays."""
    import torch

    pk = _pk()
    p, g, m, v = _state(n, 9)
    sh = make_shard(p, g, m, v, 7)
    b = np.zeros(n, np.uint16)
    for first in (2, 4, 6):
        sh.workspace.copy_(torch.randint(1, 256, sh.workspace.shape, dtype=torch.uint8, device=sh.workspace.device))
        for step in range(first, first + 3):
            got = pk.to_u64(pk.adamw_commit(sh, step, pk.Hyper(**H)))
            want = oracle.commit_and_digest(p, g, m, v, b, o_hyper(H), step, 7)
            assert step == first or got == [want], step
    assert np.array_equal(sh.param.cpu().numpy().view(np.uint32), p.view(np.uint32))


def test_calls_that_change_streams_clear_first():
    """The state vouches for calls on one stream only: after a call on another
    stream the workspace is cleared by the call itself."""
    import torch

    pk = _pk()
    n = 66 * T + 3
    p, g, m, v = _state(n, 4)
    sh = make_shard(p, g, m, v, 7)
    want = [oracle.state_digest(p, m, v, 7)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for k in range(4):
        sh.workspace.fill_(0x5A)  # on the main stream, where the state vouches for nothing after a side call
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            if k == 0:
                assert sh.workspace_clean  # what the state says of the main stream
            got = pk.to_u64(pk.shard_digest(sh))
        assert got == want, k
        torch.cuda.synchronize()
        sh.workspace.fill_(0x5A)
        torch.cuda.synchronize()
        assert pk.to_u64(pk.shard_digest(sh)) == want, k


def test_digest_replays_from_a_hip_graph():
    """A captured digest, whose workspace the capture's own stream does not
    vouch for: every replay equals the eager call, with eager calls of the
    same shard between them."""
    import torch

    pk = _pk()
    n = 70 * T + 9
    p, g, m, v = _state(n, 5)
    sh = make_shard(p, g, m, v, 31)
    want = [oracle.state_digest(p, m, v, 31)]
    assert pk.to_u64(pk.shard_digest(sh)) == want
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            pk.shard_digest(sh)
    torch.cuda.current_stream().wait_stream(side)
    for k in range(3):
        sh.digest.fill_(-1)
        graph.replay()
        assert pk.to_u64(sh.digest) == want, k
        assert pk.to_u64(pk.grad_guard(sh)) == [int(np.count_nonzero(g.view(np.uint32)))]
        sh.digest.fill_(-1)
        assert pk.to_u64(pk.shard_digest(sh)) == want


def _reads(pk, sh, p, g, m, v, goff):
    """(call, its result slots) of the calls that only read a shard."""
    b = host_copy(sh)
    return [(lambda: pk.shard_digest(sh), [oracle.state_digest(p, m, v, goff)]),
            (lambda: pk.grad_guard(sh), [int(np.count_nonzero(g.view(np.uint32)))]),
            (lambda: pk.bf16_digest(sh), [oracle.bf16_digest(b, goff)])]


def host_copy(sh):
    return sh.param_bf16.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("n", [3 * T + 7, 70 * T])
@pytest.mark.parametrize("how", ["written", "written later", "replaced"])
def test_reads_after_the_caller_wrote_to_the_workspace(n, how):
    """The workspace is the caller's scratch: whatever was written to it by other
    means, without a word to the shard, the digests, the guard and the BF16
    commit are right (the slots hold something else before each call)."""
    import torch

    pk = _pk()
    p, g, m, v = _state(n, 6)

    def dirty(sh, kept):
        if how == "replaced":
            sh.workspace = torch.full_like(sh.workspace, 0x5A)
        elif how == "written":
            sh.workspace.fill_(0x5A)
        else:
            kept.fill_(0x5A)
        sh.digest.fill_(-1)

    sh = make_shard(p, g, m, v, 11)
    kept = sh.workspace
    for _ in range(2):
        for call, want in _reads(pk, sh, p, g, m, v, 11):
            dirty(sh, kept)
            assert pk.to_u64(call()) == want
            assert pk.to_u64(call()) == want
    words = [oracle.bf16_rne_bits(x.view(np.uint32)) for x in (p, g, m, v)]
    sh = pk.ShardBf16(*(torch.from_numpy(x.view(np.int16).copy()).cuda() for x in words), 11)
    kept = sh.workspace
    p, g, m, v = words
    for step in (3, 4):
        dirty(sh, kept)
        want = oracle.commit_and_digest_bf16(p, g, m, v, o_hyper(H), step, 11)
        assert pk.to_u64(pk.adamw_commit_bf16(sh, step, pk.Hyper(**H))) == [want]
        dirty(sh, kept)
        assert pk.to_u64(pk.shard_digest_bf16(sh)) == [want]


@pytest.mark.parametrize("call", ["digest", "commit"])
def test_replays_after_a_workspace_that_was_not_clear(call):
    """A call captured on the very stream the state vouches for: replays are right
    whatever the workspace holds by then."""
    import torch

    pk = _pk()
    n = 70 * T + 9
    p, g, m, v = _state(n, 7)
    sh = make_shard(p, g, m, v, 31)
    b = np.zeros(n, np.uint16)

    def go():
        return pk.shard_digest(sh) if call == "digest" else pk.adamw_commit(sh, 4, pk.Hyper(**H))

    def want():
        if call == "digest":
            return [oracle.state_digest(p, m, v, 31)]
        return [oracle.commit_and_digest(p, g, m, v, b, o_hyper(H), 4, 31)]

    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        assert pk.to_u64(go()) == want()
        with torch.cuda.graph(graph, stream=side):
            go()
        for k in range(4):
            sh.digest.fill_(-1)
            if k != 1:
                sh.workspace.fill_(0x5A)
            graph.replay()
            assert pk.to_u64(sh.digest) == want(), k
        if call == "digest":
            assert pk.to_u64(go()) == want()


def test_commits_told_that_the_workspace_is_clear():
    """PACT_COMMIT_WORKSPACE_CLEAN in call after call at one step: a workspace that
    was not clear costs no call behind the next one."""
    import torch

    pk = _pk()
    n = 70 * T + 9
    p, g, m, v = _state(n, 8)
    sh = make_shard(p, g, m, v, 31)
    b = np.zeros(n, np.uint16)
    for _ in range(2):
        sh.workspace.fill_(0x5A)
        for k in range(3):
            want = oracle.commit_and_digest(p, g, m, v, b, o_hyper(H), 4, 31)
            rc = pk._lib().pact_adamw_commit_ex(ctypes.byref(sh._c()), 4, ctypes.byref(pk.Hyper(**H)._c()),
                                                pk.PACT_COMMIT_WORKSPACE_CLEAN)
            assert rc == pk.PACT_OK
            got = pk.to_u64(sh.digest)
            assert k == 0 or got == [want], k
    torch.cuda.synchronize()
