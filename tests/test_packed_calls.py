"""The bytes the Python calls hand to the library are the C structures' (no GPU)."""
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
