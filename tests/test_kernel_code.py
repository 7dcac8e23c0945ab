"""What the compiler made of inner loops whose speed hangs on it, read from the built library's own code.  No GPU."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2403_08837_amd", "libcdp.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def code_of(tmp_path_factory):
    """Instructions of a kernel, given the start of its mangled name."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    from paper_2403_08837_amd import binding
    binding.lib()  # fails here when the library has not been built
    tmp = tmp_path_factory.mktemp("code")
    shutil.copy(LIB, tmp / "libcdp.so")
    subprocess.run([OBJDUMP, "--offloading", "libcdp.so"], cwd=tmp, check=True, capture_output=True, timeout=120)
    objects = [tmp / f for f in os.listdir(tmp) if "amdgcn" in f]

    def get(name):
        for o in objects:
            names = subprocess.run([OBJDUMP, "--syms", str(o)], check=True, capture_output=True, text=True, timeout=120).stdout
            m = re.search(r"\bF \.text\s+\S+ (?:\.protected )?(%s\S*)" % name, names)
            if m:
                text = subprocess.run([OBJDUMP, "-d", "--disassemble-symbols=" + m.group(1), str(o)], check=True, capture_output=True, text=True, timeout=120).stdout
                return [l.split("//")[0].strip() for l in text.splitlines() if l.startswith("\t")]
        raise AssertionError("no kernel " + name)
    return get


def test_fp32_weight_gradient_requests_fragments_ahead_of_its_products(code_of):
    """64-row tiles: the x fragments (single LDS reads) of eight steps are requested before the first product, and none between products
    (asked for step by step, each waited for, a launch takes 5 to 13 % longer)."""
    code = [c.split()[0] for c in code_of("_ZN3cdp17conv_wgrad_kernelIfLi64E")]
    products = [i for i, c in enumerate(code) if c.startswith("v_mfma_f32_32x32x2")]
    assert len(products) == 16, len(products)  # eight steps of two
    between = [c for c in code[products[0]:products[-1]] if c == "ds_read_b32"]
    assert not between and "ds_read_b32" in code[products[0] - 12:products[0]], between
