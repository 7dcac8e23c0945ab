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
def objects(tmp_path_factory):
    """The device code of the built library."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    from paper_2403_08837_amd import binding
    binding.lib()  # fails here when the library has not been built
    tmp = tmp_path_factory.mktemp("code")
    shutil.copy(LIB, tmp / "libcdp.so")
    subprocess.run([OBJDUMP, "--offloading", "libcdp.so"], cwd=tmp, check=True, capture_output=True, timeout=120)
    return [tmp / f for f in os.listdir(tmp) if "amdgcn" in f]


@pytest.fixture(scope="module")
def code_of(objects):
    """Instructions of a kernel, given the start of its mangled name."""
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


def _scalars(operand):
    """Numbers of the scalar registers that an operand names."""
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m.group(1))} if m else set()


def _short_waits(code):
    """Buffer instructions of a kernel that read a scalar register fewer than five wait states after the vector unit wrote it (the hardware
    does not wait for that), or, loading into LDS, m0 in the very next one after its write; and how many load into LDS."""
    short, into_lds = [], 0
    for i, c in enumerate(code):
        if not c.startswith("buffer_") or " " not in c:
            continue
        read = set().union(*(_scalars(o) for o in re.split(r"[,\s]+", c)[1:]))
        lds = c.endswith(" lds")
        into_lds += lds
        states = 0
        for before in reversed(code[max(0, i - 5):i]):
            name, _, operands = before.partition(" ")
            operands = [o.strip() for o in operands.split(",")]
            if name.startswith("v_") and any(_scalars(o) & read for o in operands[:2 if "_co_" in name or "mad_" in name or "div_scale" in name else 1]):
                short.append((before, states, c))
                break
            if lds and states == 0 and operands[0] == "m0":
                short.append((before, states, c))
                break
            states += int(operands[0]) + 1 if name == "s_nop" else 1
            if states >= 5:
                break
    return short, into_lds


def test_wait_states_in_front_of_buffer_instructions(objects):
    """In particular the loads into LDS that are assembly, into which the compiler does not look.  In the kernels that have such loads no buffer
    instruction stands in a loop over the lanes' descriptors, as it does where a word of the descriptor is in a vector register."""
    kernels = 0
    for o in objects:
        text = subprocess.run([OBJDUMP, "-d", str(o)], check=True, capture_output=True, text=True, timeout=300).stdout
        for part in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            code = [l.split("//")[0].strip() for l in part.splitlines() if l.startswith("\t")]
            short, into_lds = _short_waits(code)
            assert not short, (part.split(">")[0], len(short), short[:3])
            kernels += into_lds > 0 and "conv_ge" in part.split(">")[0]
            if into_lds:
                assert not any(c.startswith("s_and_saveexec") and d.startswith("buffer_") for c, d in zip(code, code[1:])), part.split(">")[0]
    assert kernels >= 13, kernels


def test_what_counts_as_a_short_wait():
    load = "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"
    assert _short_waits(["v_readfirstlane_b32 s5, v2", "s_mov_b32 m0, s9", "s_nop 0", load]) == ([("v_readfirstlane_b32 s5, v2", 2, load)], 1)
    assert _short_waits(["v_readfirstlane_b32 s5, v2", "s_mov_b32 m0, s9", "s_nop 3", load]) == ([], 1)
    assert _short_waits(["v_readfirstlane_b32 s8, v2", "s_mov_b32 m0, s9", "s_nop 0", load]) == ([], 1)
    assert _short_waits(["s_mov_b32 s5, s20", "s_mov_b32 m0, s9", load]) == ([("s_mov_b32 m0, s9", 0, load)], 1)


def test_convolution_tiles_do_not_spill(objects):
    """Registers of the tiles that load straight into LDS, and of those in fp32: an epilogue variant that spills reloads between its stores, and a
    reload waits for them (256 x 256 tiles with a residual 276 us, without spills 248)."""
    readelf, spills = os.path.join(os.path.dirname(OBJDUMP), "llvm-readelf"), {}
    for o in objects:
        name = None
        text = subprocess.run([readelf, "--notes", str(o)], check=True, capture_output=True, text=True, timeout=120).stdout
        for key, value in re.findall(r"^\s+-?\s*\.(symbol|vgpr_spill_count):\s+(\S+)", text, flags=re.M):
            if key == "symbol":
                name = value
            elif "conv_ge" in name and ("_dl_kernel" in name or "_run_kernel" in name or "conv_gemm_kernelIf" in name):
                spills[name] = int(value)
    assert len(spills) >= 25 and not any(spills.values()), spills
