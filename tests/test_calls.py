"""The kernel-level entry points through _calls.so against the same calls through ctypes: no GPU, every call is refused by the library
before anything is launched."""
import ctypes
import os
import shutil
import subprocess
import sys
import textwrap

import numpy as np
import pytest

from paper_2403_08837_amd import binding as b

# arguments of calls that the library refuses with CDP_EINVAL (a size of zero or a null pointer)
REFUSED = {"cdp_k_gemm": (0, 5, 1, 1, 4096, 4096, 4096, 0, 8, 8, 8, 8, None),
           "cdp_k_conv": (1, 0, 4096, 4096, 4096, 0, 8, 8, 8, 8, 1, 1, 0, None, 0, None),
           "cdp_k_conv_wgrad_static": (1, 4096, 4096, 4096, 0, 8, 8, 8, 8, 1, 1, 0, None),
           "cdp_k_layernorm": (0, 0, 4096, None, None, 4096, 4096, 4096, None, None, None, 0, 0, 8, None),
           "cdp_k_gelu": (0, 0, 4096, None, 4096, 0, None),
           "cdp_k_attention": (0, 0, 4096, 4096, None, 4096, 4096, 0, 0, 8, 8, 1, None)}


def _fast(name):
    getattr(b, "_" + name)(*REFUSED[name])  # loads the library and binds the entry
    return getattr(b, "_" + name)


@pytest.mark.parametrize("name", sorted(REFUSED))
def test_plain_integers_take_the_short_way(name):
    slow, fast, args = getattr(b.lib(), name), _fast(name), REFUSED[name]
    assert fast(*args) == slow(*args) == b.CDP_EINVAL
    for i, a in enumerate(args):
        if a is None:  # 0 is the null pointer too
            assert fast(*args[:i], 0, *args[i + 1:]) == b.CDP_EINVAL
    wide = tuple(a + (5 << 32) if isinstance(a, int) and a < 4096 else a for a in args)  # what does not fit an int: its low bits
    assert fast(*wide) == slow(*wide)
    assert fast(*(-1 if a == 0 else a for a in args)) == slow(*(-1 if a == 0 else a for a in args))


@pytest.mark.parametrize("name", sorted(REFUSED))
def test_other_arguments_go_through_ctypes(name):
    """Left alone by the short way, accepted or refused as before by the public function."""
    fast, args, public = _fast(name), REFUSED[name], getattr(b, name)
    given = [a or 0 for a in args]
    for i, a in enumerate(args):
        if not isinstance(a, int) or a >= 4096:
            continue
        for other in (np.int64(a), bool(a) if a < 2 else None, float(a), "8"):
            if other is None:
                continue
            call = list(args)
            call[i] = other
            assert fast(*call) is None, (i, other)
            call = list(given)
            call[i] = other
            with pytest.raises((ctypes.ArgumentError, TypeError) if isinstance(other, (float, str)) else b.CdpError):
                public(*call)
    assert fast(*args[:-1]) is None and fast(*args, 0) is None


def _in_a_copy(tmp_path, calls, program):
    """Runs `program` (b: the binding of a copy of the package in another folder, original: this one's libcdp.so), what it prints."""
    package = os.path.dirname(b.__file__)
    copy = tmp_path / "paper_2403_08837_amd"
    copy.mkdir()
    for f in os.listdir(package):
        if f.endswith(".py") or f == "libcdp.so" or f == "_calls.so" and calls is None:
            shutil.copy(os.path.join(package, f), copy / f)
    if calls:
        (copy / "_calls.so").write_bytes(calls)
    program = textwrap.dedent("""
        import os
        from paper_2403_08837_amd import binding as b
        original = %r
        copy = os.path.join(os.path.dirname(b.__file__), "libcdp.so")
        assert not os.path.samefile(copy, original)
        def refused(call, *args):
            try:
                call(*args)
            except b.CdpError as e:
                return e.code
        def mapped():
            return {l.split(None, 5)[5].strip() for l in open("/proc/self/maps") if l.rstrip().endswith("libcdp.so")}
        """) % os.path.join(package, "libcdp.so") + textwrap.dedent(program)
    env = dict(os.environ, PYTHONPATH=str(tmp_path), PYTHONSAFEPATH="1")
    return subprocess.run([sys.executable, "-c", program], cwd=str(tmp_path), env=env, check=True, capture_output=True, text=True, timeout=300).stdout


def test_calls_stay_with_the_library_beside_them(tmp_path):
    """A copied package runs its own kernels: one libcdp.so is mapped, the copy's."""
    assert os.path.exists(os.path.join(os.path.dirname(b.__file__), "_calls.so"))
    _in_a_copy(tmp_path, None, """
        assert refused(b.cdp_k_gelu, 0, 0, 4096, 0, 4096, 0) == b.CDP_EINVAL
        assert b._cdp_k_gelu(0, 0, 4096, None, 4096, 0, None) == b.CDP_EINVAL  # the short way
        assert mapped() == {os.path.realpath(copy)}, mapped()
        """)


def test_calls_stay_with_their_library_beside_another(tmp_path):
    """With the original mapped first the copy's calls still run in the copy: its last error is the one that is set."""
    _in_a_copy(tmp_path, None, """
        import ctypes
        other = ctypes.CDLL(original)
        other.cdp_last_error.argtypes, other.cdp_last_error.restype = [ctypes.c_void_p], ctypes.c_char_p
        b.lib()
        assert len(mapped()) == 2
        big = (1, 4096, 4096, 4096, 2048, 1, 1, 2048, 2048, 1, 1, 0)  # partial sums of 16 MiB a range, more than the library's own array
        assert refused(b.cdp_k_conv_wgrad_static, *big) == b.CDP_ENOMEM
        assert b._cdp_k_conv_wgrad_static(*big, None) == b.CDP_ENOMEM
        assert b"needs" in b.lib().cdp_last_error(None) and b"needs" not in (other.cdp_last_error(None) or b"")
        """)


@pytest.mark.parametrize("calls", [b"", b"not a library"])
def test_calls_without_the_short_way(tmp_path, calls):
    """No _calls.so, or one that does not load: the calls go through ctypes."""
    _in_a_copy(tmp_path, calls, """
        for _ in range(2):
            assert refused(b.cdp_k_gelu, 0, 0, 4096, 0, 4096, 0) == b.CDP_EINVAL
        assert b._cdp_k_gelu(0, 0, 4096, None, 4096, 0, None) is None
        """)


def test_build_goes_on_without_a_compiler_for_the_calls(tmp_path, monkeypatch, capsys):
    from paper_2403_08837_amd import build
    monkeypatch.setattr(build, "CALLS", str(tmp_path / "_calls.so"))
    (tmp_path / "_calls.so").write_bytes(b"of another build")
    monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    build.build_calls()
    assert not (tmp_path / "_calls.so").exists() and "ctypes" in capsys.readouterr().err
