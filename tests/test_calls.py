"""The kernel-level entry points through _calls.so against the same calls through ctypes: no GPU, every call is refused by the library
before anything is launched."""
import ctypes

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
