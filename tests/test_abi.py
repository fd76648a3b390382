"""The C-ABI library loads and exports every symbol the header declares (no compute calls)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2301_02959_amd", "libflexshard_hip.so")


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "flexshard.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(fs_[a-z_0-9]+)\s*\(", text)))


def test_header_declares_the_four_entry_points():
    names = declared_symbols()
    for must in ("fs_plan_replication", "fs_route_bucketize", "fs_seq_gather_fwd", "fs_seq_grad_bwd"):
        assert must in names


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built (run __graft_entry__.build())")
def test_library_exports_every_declared_symbol():
    lib = ctypes.CDLL(LIB)
    for name in declared_symbols():
        assert hasattr(lib, name), name
    lib.fs_version.restype = ctypes.c_int32
    lib.fs_bwd_tile.restype = ctypes.c_int32
    assert lib.fs_version() >= 1000 and lib.fs_bwd_tile() == 256


def test_binding_lists_the_same_names():
    import paper_2301_02959_amd as fs
    assert sorted(fs.EXPORTS) == declared_symbols()
    for name in fs.EXPORTS:
        assert callable(getattr(fs, name))


def test_oracle_and_library_constants_agree_by_value():
    """The two sides share no header; their constants must still mean the same."""
    import oracle
    import paper_2301_02959_amd as fs
    assert (oracle.BAD_ID, oracle.BAD_OFFSETS, oracle.BAD_PLACEMENT, oracle.COUNT_OVERFLOW, oracle.UNIQUE_OVERFLOW,
            oracle.POS_ORDER) == (fs.FS_DEV_BAD_ID, fs.FS_DEV_BAD_OFFSETS, fs.FS_DEV_BAD_PLACEMENT,
                                  fs.FS_DEV_COUNT_OVERFLOW, fs.FS_DEV_UNIQUE_OVERFLOW, fs.FS_DEV_POS_ORDER)
    assert oracle.NOT_SORTED == fs.FS_DEV_NOT_SORTED
    assert oracle.BWD_TILE == fs.FS_BWD_TILE
    assert (oracle.F32, oracle.F16, oracle.BF16) == (fs.FS_F32, fs.FS_F16, fs.FS_BF16)


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built (run __graft_entry__.build())")
def test_binding_refuses_host_tensors_and_wrong_element_types():
    """The binding passes device pointers through: a host tensor or a wrong element type never reaches the library."""
    import torch
    import paper_2301_02959_amd as fs
    host = torch.zeros(64, dtype=torch.uint8)
    with pytest.raises(TypeError):
        fs.fs_util_copy(host, host)
    w = torch.zeros(4, 8)
    with pytest.raises(TypeError):
        fs.fs_seq_gather_fwd(w, torch.zeros(1, dtype=torch.int64), torch.zeros(1, dtype=torch.int32), 0, 1, w.clone())


def test_pointers_in_native_code_and_in_python():
    """The binding's native helper is built and hands everything that is no plain CUDA tensor to the Python check: host
    tensors, subclasses, other objects raise as they do there."""
    import torch
    import paper_2301_02959_amd as fs
    from paper_2301_02959_amd import _marshal
    assert fs._ptr is _marshal.device_pointer

    class Sub(torch.Tensor):
        pass

    assert fs._ptr(None) is None and fs._ptr(None, (torch.int64,)) is None
    for bad in (torch.zeros(3), torch.zeros(3).as_subclass(Sub), torch.zeros(2, 2).t(), "text", 7):
        for dtypes in (None, (torch.float32,), (torch.int64,), [torch.float32]):
            seen = []
            for check in (fs._ptr, fs._ptr_checked):
                with pytest.raises((TypeError, AttributeError)) as e:
                    check(bad, dtypes)
                seen.append((type(e.value), str(e.value)))
            assert seen[0] == seen[1]
    with pytest.raises(TypeError):
        fs._ptr()


def test_a_native_helper_for_another_torch_is_not_used(monkeypatch):
    import torch
    import paper_2301_02959_amd as fs
    from paper_2301_02959_amd import _marshal, build
    assert _marshal.__file__ == build.MARSHAL and not os.path.exists(build.UNTAGGED)
    assert fs._native_ptr() is _marshal.device_pointer
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", "1.0.0")
        assert fs._native_ptr() is fs._ptr_checked
    with monkeypatch.context() as m:
        m.setattr(torch.version, "git_version", "of another build")
        assert fs._native_ptr() is fs._ptr_checked
    with monkeypatch.context() as m:
        m.delattr(_marshal, "built_for")                   # a helper that does not say
        assert fs._native_ptr() is fs._ptr_checked
    assert fs._native_ptr() is _marshal.device_pointer


@pytest.mark.parametrize("cxx", ["false", "/no/such/compiler"])
def test_the_build_does_without_the_native_helper(tmp_path, monkeypatch, capsys, cxx):
    """Only the HIP library has to build: without a host compiler the helper is left out, and an old one removed."""
    from paper_2301_02959_amd import build
    hipcc = tmp_path / "hipcc"                             # writes its output file, as a compiler does
    hipcc.write_text('#!/bin/sh\nwhile [ "$1" != -o ]; do shift; done\necho built > "$2"\n')
    hipcc.chmod(0o755)
    monkeypatch.setattr(build, "PKG", str(tmp_path))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "_marshal.so"))
    monkeypatch.setattr(build, "UNTAGGED", str(tmp_path / "_marshal.so"))
    (tmp_path / "_marshal.so").write_text("of another source")
    monkeypatch.setenv("HIPCC", str(hipcc))
    monkeypatch.setenv("CXX", cxx)
    assert build.build(force=True) == build.LIB
    assert (tmp_path / "lib.so").read_text() == "built\n" and not (tmp_path / "_marshal.so").exists()
    assert "check its pointers in Python" in capsys.readouterr().err
    assert not build.stale() and build.helper_stale()
    monkeypatch.setenv("HIPCC", "/no/such/compiler")
    assert build.build(force=False) == build.LIB           # the library is current, whatever the helper is
    monkeypatch.setenv("HIPCC", "false")
    with pytest.raises(RuntimeError):
        build.build(force=True)


@pytest.mark.gpu
def test_native_pointers_on_the_gpu():
    import torch
    import paper_2301_02959_amd as fs
    t = torch.zeros(8, 4, device="cuda")

    class Sub(torch.Tensor):
        pass

    for good in (t, t[3:], t.view(-1)[5:], torch.nn.Parameter(t), t.as_subclass(Sub), t[8:], t.int(), torch.zeros(0, device="cuda")):
        for dtypes in (None, (good.dtype,), (torch.uint8, good.dtype)):
            assert fs._ptr(good, dtypes) == fs._ptr_checked(good, dtypes) == good.data_ptr()
    for bad, dtypes in ((t.t(), None), (t[:, 1:], None), (t, (torch.int32,)), (t, ()), (t.cpu(), None)):
        seen = []
        for check in (fs._ptr, fs._ptr_checked):
            with pytest.raises(TypeError) as e:
                check(bad, dtypes)
            seen.append(str(e.value))
        assert seen[0] == seen[1]
    errors = []
    for check in (fs._ptr, fs._ptr_checked):                # no storage to point to: the same answer from both

        def call(x):
            check(x)
            return x

        with pytest.raises(Exception) as e:
            torch.func.vmap(call)(t)
        errors.append(type(e.value))
    assert errors[0] is errors[1]
    assert fs._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert fs._stream() == side.cuda_stream
