"""What the Python calls hand to the library: the C structures as bytes, and what is
known about the workspace (no GPU)."""
import ctypes

import pytest
import torch

import paper_2609_18178_amd as pk


def _shard(monkeypatch, cls, segments, absent):
    """A shard of host tensors: nothing here launches."""
    monkeypatch.setattr(pk, "_dev_tensor", lambda t, *a: t)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 0x1234)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: type("S", (), {"cuda_stream": 0x1234}))
    n, half = 1003, torch.zeros(1003, dtype=torch.bfloat16)
    hypers = [pk.Hyper(), pk.Hyper(lr=1e-4)] if segments else None
    if cls is pk.Shard:
        p, g, m, v = (torch.zeros(n) for _ in range(4))
        return pk.Shard(p, None if absent else g, m, v, None if absent else half, (1 << 55) + 7, segments, hypers)
    p, g, m, v = (half.clone() for _ in range(4))
    return pk.ShardBf16(p, None if absent else g, m, v, 12, segments, hypers)


@pytest.mark.parametrize("cls", [pk.Shard, pk.ShardBf16])
@pytest.mark.parametrize("segments", [None, [(0, 500, 0), (500, 0, 1), (512, 491, 1)]])
@pytest.mark.parametrize("absent", [False, True])
def test_packed_bytes_are_the_structure(monkeypatch, cls, segments, absent):
    monkeypatch.setattr(pk._Workspace, "_init_workspace",
                        lambda self, nbytes: setattr(self, "workspace", torch.zeros(nbytes, dtype=torch.uint8)))
    sh = _shard(monkeypatch, cls, segments, absent)
    assert sh._packed() == bytes(sh._c())
    if cls is pk.Shard:
        assert sh._packed(workspace=False) == bytes(sh._c(workspace=False))
    sh.global_offset = -1  # wraps as in the structure (the library refuses it)
    assert sh._packed() == bytes(sh._c())


@pytest.mark.parametrize("call,cls", [(pk.shard_digest, pk.ShardBf16), (pk.shard_digest_bf16, pk.Shard),
                                      (pk.adamw_commit, pk.ShardBf16), (pk.adamw_commit_bf16, pk.Shard)])
def test_the_other_kind_of_shard_is_refused(monkeypatch, call, cls):
    monkeypatch.setattr(pk._Workspace, "_init_workspace",
                        lambda self, nbytes: (setattr(self, "workspace", None),
                                              setattr(self, "_ws_state", pk._CWorkspaceState())))
    sh = _shard(monkeypatch, cls, None, False)
    with pytest.raises(ctypes.ArgumentError):
        call(sh, 1) if "commit" in call.__name__ else call(sh)


@pytest.mark.parametrize("cls", [pk.Shard, pk.ShardBf16])
@pytest.mark.parametrize("how", ["asked for", "replaced"])
def test_a_workspace_that_others_may_write_to_is_not_taken_to_be_clear(monkeypatch, cls, how):
    """Once the caller has had the workspace, or put another in its place, only a binary32
    commit goes by what its last call left."""
    monkeypatch.setattr(pk._Workspace, "_init_workspace", lambda self, nbytes: None)
    sh = _shard(monkeypatch, cls, None, False)
    sh.workspace = torch.zeros(16 * 32 * 8, dtype=torch.uint8)
    sh._ws_shared, sh._ws_state.clear = False, 1  # as a shard that made its own
    seen = []

    def entry(shard, name, packed, *args):
        seen.append(args[-1].clear)
        args[-1].clear = 1  # as a call that ran

    monkeypatch.setattr(pk, "_enqueue", entry)
    out = torch.zeros(1, dtype=torch.int64)
    monkeypatch.setattr(pk, "_result_slots", lambda shard, o: out)
    reads = [pk.shard_digest, pk.grad_guard, pk.bf16_digest] if cls is pk.Shard else \
        [pk.shard_digest_bf16, lambda s: pk.adamw_commit_bf16(s, 1)]
    for call in reads:
        call(sh)
    assert seen == [1] * len(reads)
    if how == "asked for":
        assert sh.workspace.numel() == 16 * 32 * 8
    else:
        sh.workspace = torch.ones(16 * 32 * 8, dtype=torch.uint8)
        assert not sh.workspace_clean
    del seen[:]
    for call in reads * 2:
        call(sh)
    assert seen == [0] * 2 * len(reads)
    if cls is pk.Shard:
        pk.adamw_commit(sh, 1)
        assert seen[-1] == 1 and sh.workspace_clean
