"""_marshal takes a call only if every argument is exactly what the entry point wants and leaves everything else to the
ctypes path, which names the error.  Without a GPU nothing may be taken: the tensors are in host memory."""
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

from paper_2511_09323_amd import binding as B


@pytest.fixture(scope="module")
def fast():
    B.load_library()
    return B._fast


def test_host_tensors_and_other_types_are_not_taken(fast):
    x, w, ws = torch.zeros(4, 64), torch.zeros(128, 64), torch.zeros(1 << 20, dtype=torch.uint8)
    y, idx, sel = torch.zeros(4, 64), torch.zeros(4, 16, dtype=torch.int32), torch.zeros(4, 16)
    assert fast.decode(x, w, w, w, 16, y, idx, ws) == B._NOT_TAKEN
    assert fast.decode(x, w, w, w, 16, y, None, ws) == B._NOT_TAKEN
    assert fast.decode(None, w, w, w, 16, y, idx, ws) == B._NOT_TAKEN
    assert fast.decode(x, w, w, w, 16.0, y, idx, ws) == B._NOT_TAKEN
    assert fast.decode(x, w, w, w, 16, y, idx) == B._NOT_TAKEN                # wrong number of arguments
    assert fast.fwd(x, w, w, w, 16, y, idx, sel, sel, ws) == B._NOT_TAKEN
    assert fast.fwd_experts(x, [0, 4], w[None], w[None], w[None], 16, y, idx, sel, sel, ws) == B._NOT_TAKEN
    assert fast.rmsnorm(x, x[0], 1e-5, y) == B._NOT_TAKEN
    assert fast.residual_add(x, y) == B._NOT_TAKEN


def test_errors_keep_their_names(fast):
    x, w, ws = torch.zeros(4, 64), torch.zeros(128, 64), torch.zeros(1 << 20, dtype=torch.uint8)
    with pytest.raises(B.MocError, match="x must be a GPU tensor"):
        B.moc_ffn_decode(x, w, w, w, 16, ws=ws, out=(torch.zeros(4, 64), None))
    with pytest.raises(B.MocError, match="must be a GPU tensor"):
        B.moc_residual_add(x, x)


def test_tensors_without_memory_raise(fast):
    """A fake tensor says it is on the GPU and throws when asked for its address."""
    with FakeTensorMode():
        x, w = torch.empty(4, 64, device="cuda"), torch.empty(128, 64, device="cuda")
        ws, idx = torch.empty(1 << 20, dtype=torch.uint8, device="cuda"), torch.empty(4, 16, dtype=torch.int32, device="cuda")
        assert fast.decode(x, w, w, w, 16, x, idx, ws) == B._NOT_TAKEN
        assert fast.residual_add(x, x) == B._NOT_TAKEN


def test_hash_and_rebuild_cover_the_extension(tmp_path, monkeypatch):
    """The hash that tells builds apart covers marshal.cpp, and a build of single files does not leave an extension behind that is
    older than its sources."""
    import os
    import shutil

    from paper_2511_09323_amd import build as b
    csrc = tmp_path / "csrc"
    shutil.copytree(b.CSRC, csrc)
    monkeypatch.setattr(b, "CSRC", str(csrc))
    before = b.source_hash()
    with open(csrc / "marshal.cpp", "a") as f:
        f.write("// changed\n")
    assert b.source_hash() != before
    ran = []
    ext = tmp_path / "ext.so"
    monkeypatch.setattr(b, "MARSHAL", str(ext))
    monkeypatch.setattr(b, "OBJ", str(tmp_path / "obj"))
    monkeypatch.setattr(b, "_run", lambda cmd, verbose: ran.append(cmd[-3:] if "-c" in cmd else cmd))
    built = lambda: any("marshal.cpp" in a for cmd in ran for a in cmd)
    b.build(verbose=False, only=["moc_fwd.hip"])
    assert built()                                                             # missing
    ext.write_bytes(b"")
    newer = os.path.getmtime(csrc / "marshal.cpp") + 10
    os.utime(ext, (newer, newer))
    ran.clear()
    b.build(verbose=False, only=["moc_fwd.hip"])
    assert not built()
    os.utime(csrc / "marshal.cpp", (newer + 10, newer + 10))
    ran.clear()
    b.build(verbose=False, only=["moc_fwd.hip"])
    assert built()


@pytest.mark.gpu
def test_both_ways_give_the_same_call():
    x, w = torch.randn(3, 64, device="cuda").bfloat16(), [torch.randn(200, 64, device="cuda").bfloat16() for _ in range(3)]
    ws = torch.empty(B.workspace_bytes(3, 64, 200, 25, torch.bfloat16, B.OP_DECODE), dtype=torch.uint8, device="cuda")
    y, idx = torch.empty_like(x), torch.empty(3, 25, dtype=torch.int32, device="cuda")
    B.moc_ffn_decode(x, *w, 25, ws=ws, out=(y, idx))                           # taken
    y2, idx2 = B.moc_ffn_decode(x, *w, 25)                                     # allocates: ctypes
    torch.cuda.synchronize()
    assert torch.equal(y, y2) and torch.equal(idx, idx2)
    with pytest.raises(B.MocError, match="wu has shape"):
        B.moc_ffn_decode(x, w[0], w[1][:-1], w[2], 25, ws=ws, out=(y, idx))
    with pytest.raises(B.MocError, match="MOC_ERR_WORKSPACE"):
        B.moc_ffn_decode(x, *w, 25, ws=ws[:256], out=(y, idx))
    with pytest.raises(B.MocError, match="K"):
        B.moc_ffn_decode(x, *w, 201, ws=ws, out=(y, torch.empty(3, 201, dtype=torch.int32, device="cuda")))
