"""The Python binding's own logic, without a GPU: sizes that the library computes, and the stream that calls go to."""
import ctypes
import os
import shutil
import subprocess
import sys
import sysconfig

import numpy as np
import pytest
import torch

import paper_2605_28691_amd as sk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(sk._LIB_PATH):
        from paper_2605_28691_amd import build

        build.build()


def test_sizes_follow_the_value_of_their_arguments():
    """Any integer-like argument counts by its present value, also after a call with the same object or an equal number."""
    want = {8: (4, 2, 32), 16: (4, 2, 64)}
    for h, shape in want.items():
        for arg in (h, np.int64(h), np.array(h), torch.tensor(h)):
            assert sk.skiparse_lse_shape(1, 2, 2, arg, 8, 64, 2, "token") == shape
            assert sk.skiparse_bwd_workspace_bytes(1, 2, 2, arg, 8, 64, 2, "token") == 4 * int(np.prod(shape))
    t = torch.tensor(8)
    assert sk.skiparse_lse_shape(1, 2, 2, t, 8, 64, 2, "token") == want[8]
    t.fill_(16)
    assert sk.skiparse_lse_shape(1, 2, 2, t, 8, 64, 2, "token") == want[16]
    assert sk.skiparse_bwd_workspace_bytes(1, 2, 2, t, 8, 64, 2, "token") == 4 * 4 * 2 * 64


def test_sizes_refuse_what_is_no_integer():
    sk.skiparse_lse_shape(1, 2, 2, 8, 8, 64, 2, "token")
    for bad in (8.0, np.float64(8), "8", None):
        with pytest.raises(ctypes.ArgumentError):
            sk.skiparse_lse_shape(1, 2, 2, bad, 8, 64, 2, "token")
        with pytest.raises(ctypes.ArgumentError):
            sk.skiparse_bwd_workspace_bytes(1, 2, 2, bad, 8, 64, 2, "token")


@pytest.mark.parametrize("D, more", [(128, True), (64, False)])
def test_backward_without_room_for_its_faster_kernels(monkeypatch, D, more):
    """No workspace passed: where the memory for one walk is not there, the call takes what it cannot do without, as it always did."""
    at = (1, 1, 8190, 1, "token")
    q = torch.empty((1, 8190, 48, D), dtype=torch.bfloat16, device="meta")
    lse = torch.empty((1, 48, 8190), device="meta")
    least, walk = (f(1, 48, 1, 1, 8190, D, 1, "token") for f in (sk.skiparse_bwd_workspace_bytes, sk.skiparse_bwd_walk_workspace_bytes))
    assert (walk > least) == more
    used, free, empty = [], [walk], torch.empty

    def with_limit(n, **kwargs):
        if n > free[0]:
            raise torch.cuda.OutOfMemoryError(f"{n} bytes")
        return empty(n, **kwargs)

    monkeypatch.setattr(torch, "empty", with_limit)
    monkeypatch.setattr(sk, "_stream", lambda: 0)
    monkeypatch.setattr(sk, "_skiparse_attn_bwd", lambda *args: used.append(args[-3:-1]))
    for free[0], want in ((walk, walk), (walk - 1, least), (least, least)):
        if not more and free[0] < least:
            continue
        sk.skiparse_attn_bwd(q, q, q, q, q, lse, *at)
        assert used.pop()[1] == want
    free[0] = least - 1
    with pytest.raises(torch.cuda.OutOfMemoryError):
        sk.skiparse_attn_bwd(q, q, q, q, q, lse, *at)
    assert not used


def test_stream_of_a_forked_child_is_refused():
    """torch refuses the GPU in a child forked from a process that has used it; so does a call whose tensors are all there already."""
    code = """
import os, torch
torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream = (lambda: 0), (lambda device: 7)
import paper_2605_28691_amd as sk
assert sk._stream() == 7
pid = os.fork()
if pid == 0:
    torch.cuda._is_in_bad_fork = lambda: True  # what torch finds in such a child
    try:
        sk._stream()
        os._exit(3)
    except RuntimeError as e:
        os._exit(0 if "fork" in str(e) else 4)
_, status = os.waitpid(pid, 0)
assert sk._stream() == 7
raise SystemExit(os.WEXITSTATUS(status))
"""
    assert subprocess.run([sys.executable, "-c", code], cwd=ROOT).returncode == 0


@pytest.mark.parametrize("missing", ["_raw_stream", "_get_device"])
def test_stream_without_the_private_names(monkeypatch, missing):
    """A torch without the private names for the bare handle serves through its public Stream object."""

    class Stream:
        cuda_stream = 11

    monkeypatch.setattr(sk, missing, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    assert sk._stream() == 11


def test_native_marshalling_passes_on_what_is_not_plain():
    """Everything but plain tensors on the GPU, int and float goes to the general way, as it came; nothing is read from it before."""
    native = sk._marshal
    assert native is not None, "the module is built with the library"
    q = torch.zeros(1, 128, 2, 64, dtype=torch.bfloat16)
    seen = []
    native.set_up(lambda *args: seen.append(args), sk._failed)
    try:
        for name, tensors in sk._TENSORS.items():
            n = len(getattr(sk.lib(), name).argtypes)
            slots = dict(tensors)
            args = [q if i in slots else 1 for i in range(n)]
            for call in (args, args[:-1], [], [5] * n, [None] * n, [1.0] * n):
                getattr(native, name)(*call)
                assert seen.pop() == (name, *call)
    finally:
        native.set_up(sk._general, sk._failed)
    assert not seen


@pytest.mark.parametrize("bad, error", [((5,), AttributeError), ((None,), AttributeError), ((torch.zeros(1, 128, 2, 64, dtype=torch.bfloat16),), ValueError)])
def test_refused_tensors(monkeypatch, bad, error):
    monkeypatch.setattr(sk, "_stream", lambda: 0)
    good = torch.zeros(1, 128, 2, 64, dtype=torch.bfloat16)
    with pytest.raises(ValueError if error is AttributeError else error):  # q comes first, and is on the CPU
        sk.skiparse_attn_fwd(good, *bad, good, 2, 8, 8, 2, "token")
    with pytest.raises(error):
        sk._skiparse_attn_fwd(bad[0], good, good, good, 1, 2, 2, 8, 8, 64, 2, 0, 0.0, 0, 1, None, 0, 0)


def test_every_entry_point_is_marshalled_in_the_order_of_the_c_function():
    """The table of tensor arguments against the types that ctypes converts: a tensor stands exactly where the C function takes a device pointer."""
    for name, tensors in sk._TENSORS.items():
        types = getattr(sk.lib(), name).argtypes
        assert [i for i, t in enumerate(types) if t is ctypes.c_void_p] == [i for i, _ in tensors] + [len(types) - 1]


def _copy_of_package(tmp_path):
    """The built package in a folder of its own, for processes that replace its files."""
    pkg = os.path.join(tmp_path, "paper_2605_28691_amd")
    shutil.copytree(os.path.dirname(sk._LIB_PATH), pkg, ignore=shutil.ignore_patterns("csrc", "__pycache__", "*_probe.so"))
    return pkg


def test_a_library_built_after_the_import_is_the_only_one(tmp_path):
    """A process that imports the package, builds and calls runs what it has built, by every route."""
    lib = os.path.join(_copy_of_package(tmp_path), "libskiparse.so")
    code = f"""
import os, shutil
import paper_2605_28691_amd as sk
shutil.copy({lib!r}, {lib!r} + ".tmp")
os.replace({lib!r} + ".tmp", {lib!r})  # as a build does
assert sk.lib() and sk._marshal is not None and sk._skiparse_permute is sk._marshal.skiparse_permute
mapped = {{line.split(None, 5)[5].strip() for line in open("/proc/self/maps") if "libskiparse" in line}}
assert mapped == {{{lib!r}}}, mapped  # a replaced file is listed as deleted
"""
    done = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, stderr=subprocess.PIPE, text=True)
    assert done.returncode == 0, done.stderr


@pytest.mark.parametrize("change, native", [("", True), ("torch.__version__ = '0.0'", False), ("torch.version.git_version = 'another'", False)])
def test_module_is_for_one_torch(tmp_path, change, native):
    """The module reads tensors by the layout in the headers of one torch: under another one calls go through ctypes."""
    _copy_of_package(tmp_path)
    code = f"""
import torch
{change}
import paper_2605_28691_amd as sk
assert (sk._marshal is not None) == {native}
assert sk.lib() and (sk._skiparse_permute.__class__.__name__ == "partial") != {native}
"""
    assert subprocess.run([sys.executable, "-c", code], cwd=tmp_path).returncode == 0


def test_module_is_for_one_python(tmp_path):
    """Its name says which: a module without one, from another build, is taken away and never looked for."""
    from paper_2605_28691_amd import build

    assert os.path.basename(build.MARSHAL) == "_marshal" + sysconfig.get_config_var("EXT_SUFFIX") and os.path.exists(build.MARSHAL)
    assert [n for n in os.listdir(build.HERE) if n.startswith("_marshal")] == [os.path.basename(build.MARSHAL)]


def test_build_without_a_host_compiler(tmp_path, monkeypatch):
    """The library is what a build has to make; without its module calls go through ctypes.  No module of an earlier build stays beside it."""
    from paper_2605_28691_amd import build

    made = []
    for name in ("_marshal.so", os.path.basename(build.MARSHAL)):
        (tmp_path / name).write_bytes(b"old")
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / os.path.basename(build.MARSHAL)))
    monkeypatch.setattr(build, "_build_one", lambda lib, *rest: made.append((lib, sorted(p.name for p in tmp_path.iterdir()))))
    monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    with pytest.warns(UserWarning, match="ctypes"):
        assert build.build() == build.LIB
    assert made[-1] == (build.LIB, []) and not list(tmp_path.iterdir())
    monkeypatch.setenv("CXX", "false")  # one that fails
    with pytest.warns(UserWarning, match="ctypes"):
        build.build()
