"""Rules by which launches are laid out, asked of the built library: how many ranges the reduction of a weight gradient
is cut into when it is launched on its own (conv_wgrad_splits_alone in csrc/conv_kernels.hip) and how many neighbouring tiles of it
go to one XCD (conv_wgrad_xcd_run there), which weight gradients run on the tiles of launches short of workgroups
(conv_wgrad_small_wanted in csrc/conv_wgrad_small.hip), which forward / data-gradient
launches share their reductions over workgroups and which tiles they run on (conv_launch_tile in csrc/conv256_kernels.hip), which attention passes run in
one kernel (attention_fused in csrc/attention_kernels.hip), and which products of row-contiguous operands run on the
weight-gradient tiles of the Linear launch (gemm_wgrad_tiles_wanted in csrc/kernels_api.cpp).  No GPU: the rules are host arithmetic, and the times they are held
against were measured on one."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2403_08837_amd")
F32, BF16 = 0, 1


def _asker(tmp_path_factory, name):
    """A small program that calls a rule of the library for every line of numbers it is given."""
    from paper_2403_08837_amd import binding
    binding.lib()  # fails here when the library has not been built
    exe = str(tmp_path_factory.mktemp("launch_rules") / name)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(LIB, "csrc"),
                    os.path.join(ROOT, "tests", "launch_rules", name + ".cpp"), "-o", exe, os.path.join(LIB, "libcdp.so"),
                    "-Wl,-rpath," + LIB, "-L", "/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True)

    def ask(problems):
        text = "".join(" ".join("%d" % x for x in p) + "\n" for p in problems)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        return [int(x) for x in out.split()]
    return ask


@pytest.fixture(scope="module")
def ranges(tmp_path_factory):
    return _asker(tmp_path_factory, "ranges")


@pytest.fixture(scope="module")
def runs(tmp_path_factory):
    return _asker(tmp_path_factory, "runs")


@pytest.fixture(scope="module")
def few(tmp_path_factory):
    return _asker(tmp_path_factory, "few")


@pytest.fixture(scope="module")
def fused(tmp_path_factory):
    return _asker(tmp_path_factory, "attention")


@pytest.fixture(scope="module")
def wgrad_tiles(tmp_path_factory):
    return _asker(tmp_path_factory, "gemm")


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    return _asker(tmp_path_factory, "tiles")


# dtype, M (output channels), N (taps x input channels), K (positions), {ranges: us measured, on the kernel that a launch of so many runs on};
# one count per 16 slabs or three was the rule before there was a model of the cost, and comes first
MEASURED = [
    (F32, 64, 576, 401408, {205: 329, 28: 549, 49: 502, 64: 574, 98: 389, 128: 402, 196: 340, 203: 330, 256: 317, 392: 332, 784: 339}),
    (F32, 40, 2880, 20577, {41: 93.9, 6: 216, 10: 134, 16: 127, 20: 106, 28: 103, 32: 95.4, 43: 89.8, 44: 89.4}),
    (F32, 120, 432, 107632, {128: 155, 20: 332, 32: 216, 49: 211, 64: 168, 80: 184, 98: 157, 112: 173, 121: 159, 160: 154, 196: 159}),
    (F32, 64, 3024, 10140, {20: 59.5, 5: 88.9, 10: 72.2, 12: 88.1, 14: 77.3, 16: 69.1, 23: 69.8}),
    (F32, 280, 504, 40656, {80: 175, 14: 287, 20: 208, 28: 232, 40: 168, 49: 197, 56: 178, 64: 160, 83: 176}),
    (F32, 56, 792, 39546, {78: 76.9, 16: 99.2, 32: 85.3, 40: 99.1, 49: 85.6, 56: 77.6, 64: 69.8, 69: 64.7, 81: 77.0}),
    (F32, 920, 1800, 2645, {6: 120, 1: 263, 2: 144, 3: 148, 4: 120, 5: 132, 8: 131, 9: 133}),
    (F32, 128, 576, 800, {3: 12.5, 4: 11.1, 5: 11.9}),
    (BF16, 3072, 768, 6272, {7: 75.5, 1: 120, 2: 104, 3: 78.1, 4: 74.0, 5: 68.7, 6: 76.9, 8: 73.1, 12: 83.0, 16: 86.5}),
    (BF16, 128, 1152, 25088, {25: 30.7, 6: 74.8, 12: 43.4, 20: 34.2, 28: 29.5, 32: 38.6, 40: 33.1, 49: 30.6, 53: 30.9}),
    (BF16, 64, 576, 100352, {98: 30.9, 20: 88.1, 32: 58.9, 49: 42.7, 64: 39.4, 80: 34.5, 112: 37.0, 128: 35.4, 160: 34.5, 196: 31.8, 200: 31.8}),
    (BF16, 256, 2304, 6272, {7: 29.3, 2: 54.6, 4: 36.9, 6: 32.0, 8: 36.3, 10: 34.6, 12: 32.4, 14: 29.9, 16: 32.3}),
    (BF16, 136, 19800, 15129, {4: 251, 1: 284, 2: 282, 3: 287, 6: 260, 7: 252, 8: 252, 12: 258, 16: 266, 24: 299, 33: 321}),
]


@pytest.mark.parametrize("case", MEASURED, ids=lambda c: "%s-%dx%dx%d" % ("bf16" if c[0] else "f32", *c[1:4]))
def test_count_is_no_slower_than_one_per_sixteen_slabs(ranges, case):
    """The measured count nearest to the one chosen is within 6 % of the old rule's time and 8 % of the best measured (two launches of one
    count differ by up to 3 %)."""
    dtype, m, n, k, us = case
    got = ranges([(dtype, m, n, k, k // 512 + 4)])[0]
    near = min(us, key=lambda c: abs(c - got))
    assert us[near] <= 1.06 * next(iter(us.values())) and us[near] <= 1.08 * min(us.values()), (got, near, us[near])


def test_count_stays_within_bounds(ranges):
    """Never less than one range, more than there are slabs, or more than there is room for."""
    problems = [(dt, m, n, k, room) for dt in (F32, BF16) for m in (8, 64, 128, 1000) for n in (8, 576, 20000) for k in (1, 33, 6272, 401408)
                for room in (0, 1, 3, 50, 10 ** 6)]
    for p, got in zip(problems, ranges(problems)):
        slabs = -(-p[3] // (64 if p[0] else 32))
        assert 1 <= got <= max(1, min(slabs, p[4])), (p, got)


# M, N, K, ranges, us before tiles of a range were neighbours, {neighbouring tiles on one XCD: us}; bf16 but the last
ORDER = [(648, 576, 3200, 10, 24.0, {1: 22.6, 4: 25.4, 32: 25.9}), (1984, 648, 1088, 3, 25.8, {1: 24.5, 4: 26.1, 32: 27.7}),
         (280, 1224, 4800, 11, 25.5, {1: 26.3, 4: 27.2, 32: 29.2}), (784, 7128, 300, 1, 29.6, {1: 29.6, 4: 32.0, 32: 31.0}),
         (1664, 792, 2200, 3, 36.2, {1: 34.6, 4: 35.5, 32: 37.7}), (1832, 896, 1104, 3, 26.6, {1: 26.2, 4: 26.1, 32: 28.4}),
         (104, 5688, 2048, 7, 21.8, {1: 21.9, 4: 22.0, 32: 24.3}), (104, 1368, 15552, 27, 28.0, {1: 27.9, 4: 27.7, 32: 29.4}),
         (40, 8424, 2448, 8, 22.0, {1: 18.6, 4: 18.6, 32: 20.8}), (80, 2400, 13950, 20, 33.3, {1: 30.3, 4: 30.4, 32: 31.9}),
         (776, 120, 85050, 103, 82.3, {1: 78.8, 4: 54.4, 32: 54.1}), (272, 368, 18432, 36, 26.5, {1: 29.7, 4: 27.4, 32: 27.5}),
         (928, 18400, 98, 1, 48.5, {1: 48.4, 4: 51.3, 32: 49.3}), (96, 6192, 1331, 5, 37.9, {1: 38.1, 4: 38.1, 32: 39.4})]


def test_order_of_weight_gradient_tiles(runs):
    """Within 6 % of the order before (two launches of one order differ by up to 3 %)."""
    for (m, n, k, s, before, us), run in zip(ORDER, runs([c[:4] for c in ORDER])):
        assert us[run] <= 1.06 * before, (m, n, k, run)


# dtype, M, N, K, ranges, us on conv_wgrad_kernel, us on the tiles of launches short of workgroups
FEW = [(F32, 104, 7056, 25, 1, 10.6, 13.7), (F32, 32, 7128, 98, 4, 10.3, 13.7), (F32, 112, 2016, 128, 4, 9.8, 13.1), (F32, 48, 4032, 243, 4, 11.5, 13.1),
       (F32, 104, 1584, 200, 4, 12.7, 13.1), (F32, 40, 3312, 98, 4, 10.0, 12.2), (F32, 64, 5112, 49, 2, 10.4, 10.2), (F32, 48, 2808, 128, 4, 10.2, 9.7),
       (F32, 728, 504, 49, 2, 13.3, 10.3), (F32, 880, 1008, 32, 1, 13.6, 13.8), (F32, 216, 1080, 200, 4, 16.9, 13.3), (F32, 256, 1296, 169, 3, 17.3, 14.2),
       (F32, 64, 1656, 2450, 8, 28.5, 21.8), (F32, 40, 2600, 1250, 6, 22.3, 18.8), (F32, 512, 4608, 98, 1, 26.6, 27.6), (F32, 128, 1152, 25088, 53, 90, 147),
       (BF16, 744, 5112, 25, 1, 18.3, 18.8), (BF16, 56, 5688, 2800, 9, 20.9, 19.5), (BF16, 232, 1400, 6845, 11, 27.4, 25.1), (BF16, 24, 2880, 10368, 21, 21.0, 19.1),
       (BF16, 256, 2304, 6272, 14, 30.2, 32.3), (BF16, 64, 576, 100352, 196, 31.9, 34.0)]


def test_launches_short_of_workgroups(few):
    """The faster of the two kernels; in bf16 only where both operands are 16-byte aligned."""
    for (dt, m, n, k, s, other, here), on in zip(FEW, few([c[:5] + (0,) for c in FEW])):
        assert (here if on else other) <= 1.03 * min(here, other), (dt, m, n, k, s, on)
    assert not any(few([c[:5] + (1,) for c in FEW if c[0] == BF16]))


# Cout, taps x Cin, positions: what the library's own array holds at one range per 16 slabs or three, some of it only just
SCRATCH = 16 << 20
SHAPES = [(64, 288, 1024), (128, 1152, 25088), (256, 2304, 6272), (192, 1728, 6272), (512, 1024, 1568), (64, 576, 401408), (512, 2304, 6272),
          (1024, 1024, 6272), (40, 200, 100000), (512, 4608, 25088), (512, 4608, 40), (2048, 2048, 40)]


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_count_depends_on_the_shape_alone(ranges, dtype):
    """cdp_k_conv with the workspace its header asks for, with a larger one, and the entry point with the library's own array cut the
    reduction alike; what that entry point took when the count was one per 16 slabs or three it still takes."""
    for m, n, k in SHAPES:
        recommended, larger = ranges([(dtype, m, n, k, k // 512 + 4), (dtype, m, n, k, 2 ** 31 - 1)])
        assert recommended == larger, (m, n, k)
        slabs, tiles = -(-k // (64 if dtype else 32)), -(-m // (128 if m >= 128 else 64)) * -(-n // 128)
        old = max(1, min(slabs, max(3, min(-(-slabs // 16), -(-1024 // tiles)))))
        if 4 * m * n * old <= SCRATCH:
            assert 4 * m * n * recommended <= SCRATCH, (m, n, k)


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_refusal_names_the_bytes_of_the_launch(ranges, dtype):
    """The entry point with the library's own array refuses what its partial sums do not fit, and says how many bytes those are."""
    import torch
    if torch.cuda.device_count():
        pytest.skip("made-up addresses: a call that is not refused may only fail for want of a GPU")
    from paper_2403_08837_amd import binding as b
    refused = 0
    for m, n, k in SHAPES:
        need = 4 * m * n * ranges([(dtype, m, n, k, 2 ** 31 - 1)])[0]
        if need <= SCRATCH:
            continue
        refused += 1
        width = 32 if k % 32 == 0 else k
        with pytest.raises(b.CdpError) as e:
            b.cdp_k_conv_wgrad_static(dtype, 64, 64, 64, k // width, 1, width, n, m, 1, 1, 0)
        assert e.value.code == b.CDP_ENOMEM and "needs %d bytes" % need in str(e.value), str(e.value)
    assert refused >= 2


# M, N, K, us with the reduction shared over workgroups, us as one chain per tile
SHARED = [(49, 512, 4608, 10.9, 22.5), (392, 512, 4608, 13.4, 22.6), (784, 512, 4608, 17.8, 22.7), (1568, 512, 4608, 24.4, 22.8),
          (98, 1024, 9216, 15.2, 40.5), (392, 1024, 9216, 26.5, 40.8), (196, 256, 2304, 9.3, 13.4), (784, 256, 2304, 11.5, 13.5),
          (1568, 256, 2304, 14.3, 13.4), (3136, 256, 2304, 17.5, 14.0), (49, 512, 2048, 8.2, 11.6), (392, 512, 2048, 10.0, 11.7),
          (784, 512, 2048, 15.0, 11.7), (64, 64, 1024, 7.1, 7.7), (784, 512, 1024, 8.7, 7.7), (784, 128, 1152, 8.4, 8.9),
          (3136, 128, 1152, 10.3, 9.0), (98, 512, 512, 7.2, 5.9), (256, 64, 576, 7.9, 6.4)]


def test_long_reductions_of_few_tiles_are_shared(tiles):
    """Where a workspace is there, the faster of the two; without one, never."""
    got = tiles([(m, n, k, 1, 0) for m, n, k, _, _ in SHARED])
    for (m, n, k, shared_us, chain_us), tile in zip(SHARED, got):
        assert (shared_us if tile == 0 else chain_us) <= 1.03 * min(shared_us, chain_us), (m, n, k, tile)
    assert all(t != 0 for t in tiles([(m, n, k, 0, 0) for m, n, k, _, _ in SHARED]))


# M, N, K, us: conv_gemm_kernel, direct-to-LDS tiles of 64 x 64 with slabs of 64, of 32
NARROW = [(34848, 64, 5184, 58.2, 54.9, 67.2), (40328, 64, 5184, 62.5, 57.3, 68.9), (48672, 64, 5184, 71.2, 64.3, 74.5),
          (28800, 64, 9216, 87.6, 73.0, 81.8), (34848, 64, 9216, 99.8, 108.7, 123.0), (40328, 40, 9216, 103.9, 108.8, 116.9),
          (12800, 64, 5184, 38.2, 25.4, 27.4), (28800, 64, 576, 9.8, 8.0, 7.9), (45000, 64, 1024, 17.5, 16.9, 18.7)]


def test_narrow_launches_take_the_fastest_tile(tiles):
    for (m, n, k, *us), tile in zip(NARROW, tiles([(m, n, k, 0, 0) for m, n, k, *_ in NARROW])):
        assert us[{0: 0, 4: 1, 5: 2}[tile]] <= 1.03 * min(us), (m, n, k, tile)


# M, N, K, us: conv_gemm_kernel, tiles of 256 x 128, 192 x 128, 128 x 128 (None: not measured)
ROUNDS = [(25088, 128, 1152, 24.9, 21.9, 18.0, 14.6), (8503, 344, 3072, 45.1, 43.7, 34.5, 27.5), (2725, 928, 128, 7.8, 8.3, 7.3, 6.2),
          (3457, 984, 1536, 26.3, 25.8, 21.3, 17.7), (6272, 768, 3072, 54.2, 44.3, 37.3, 53.2), (6272, 768, 768, 19.9, 17.1, 14.2, 19.4),
          (20091, 256, 128, 9.8, 9.2, 8.1, 10.4), (5684, 768, 2304, 43.4, 36.0, 29.7, 42.1), (12544, 512, 1024, 24.5, 21.3, 30.8, 23.3),
          (161728, 120, 1152, 68.2, 74.5, 78.2, None), (66517, 824, 1024, 162.5, 176.0, 176.3, None), (23232, 2088, 1152, 157.1, 170.1, 175.1, None),
          (68436, 360, 1216, 93.7, 100.7, 100.7, None), (103394, 200, 1088, 85.7, 91.7, 92.1, None), (80515, 248, 1664, 102.3, 109.0, 115.2, None),
          (38108, 1984, 1024, 205.8, 216.6, 226.1, None), (92500, 616, 1152, 179.0, 188.2, 189.7, None), (16735, 1944, 1344, 126.5, 132.1, 127.4, None)]


def test_launches_in_rounds_take_the_fastest_tile(tiles):
    """One round, two, and, where the epilogue reads beside the tile, long reductions past that; lines at 150, 256 and 512 tiles of 128 x 128, 256 of
    192 x 128, and K = 1024."""
    for (m, n, k, *us), tile in zip(ROUNDS, tiles([c[:3] + (0, 2) for c in ROUNDS])):
        assert us[{0: 0, 2: 1, 6: 2, 3: 3}[tile]] <= 1.03 * min(u for u in us if u), (m, n, k, tile)
    #  256 x 128: 2, 128 x 128: 3, 64 x 64: 4, 192 x 128: 6, conv_gemm_kernel: 0
    lines = {(149 * 128, 128, 1024): 4, (150 * 128, 128, 1024): 3, (128 * 128, 256, 1024): 3, (128 * 128 + 1, 256, 1024): 6,
             (128 * 192, 256, 1024): 6, (128 * 192 + 1, 256, 1024): 2, (511 * 128, 128, 512): 2, (512 * 128, 128, 512): 0,
             (512 * 128, 128, 1024): 2, (512 * 128, 128, 960): 0, (512 * 192, 128, 4096): 6, (512 * 192 + 1, 128, 4096): 2,
             (4001 * 128, 128, 1024): 0, (4000 * 128, 128, 4096): 2}
    for beside in (1, 2, 3, 4, 5, 6):  # whatever it is that the epilogue reads
        assert {c: t for c, t in zip(lines, tiles([c + (0, beside) for c in lines]))} == lines, beside


# M, N, K, us: conv_gemm_kernel, tiles of 256 x 256, 256 x 128, 192 x 128, 128 x 128 walked by resident workgroups; epilogues that read nothing
MANY = [(100352, 256, 64, 15.7, 19.4, 24.0, 24.6, 18.5), (16035, 584, 64, 8.77, 10.66, 12.65, 11.63, 10.90), (5031, 2504, 64, 11.36, 12.03, 14.06, 16.14, 13.70),
        (14028, 1656, 128, 16.8, 21.3, 22.8, 23.7, 20.5), (25088, 512, 128, 12.92, 12.03, 14.86, 16.75, 14.92), (412926, 112, 128, 35.1, 51.2, 42.5, 44.6, 35.4),
        (17073, 1304, 192, 19.4, 23.9, 25.1, 25.5, 22.3), (18618, 704, 192, 14.70, 13.51, 16.25, 18.70, 16.01), (43667, 376, 192, 15.85, 22.13, 22.58, 20.43, 17.11),
        (19929, 592, 256, 16.7, 14.4, 16.4, 18.4, 16.4), (55962, 296, 320, 24.2, 27.9, 26.5, 26.3, 25.0), (32203, 784, 384, 32.0, 34.5, 35.9, 35.5, 30.2),
        (39821, 312, 384, 20.8, 28.0, 21.5, 22.5, 20.2), (183644, 72, 448, 35.0, 44.4, 38.0, 39.0, 33.5), (11607, 1344, 512, 25.6, 34.1, 26.1, 26.8, 24.4),
        (6272, 3072, 768, 45.7, 46.9, 47.3, 51.1, 40.2), (66517, 824, 1024, 151.4, 150.8, 142.2, 137.0, 132.3), (38108, 1984, 1024, 175.5, 145.4, 172.5, 172.7, 162.6),
        (23232, 2088, 1152, 137.3, 124.8, 132.5, 132.8, 122.4), (68436, 360, 1216, 79.7, 93.8, 79.6, 78.3, 70.2), (113066, 496, 1600, 222, 189, 207, 229, 236),
        (24534, 456, 2048, 61.3, 50.1, 60.6, 52.1, 54.0), (36029, 1672, 2304, 346, 250, 294, 304, 305), (7163, 2384, 2560, 113, 115, 108, 88, 100)]


def test_launches_of_many_tiles_take_the_fastest(tiles):
    """512 tiles of 128 x 128 and more: within 6 % of the fastest (the rule is a model of rms 7 to 10 %); lines at a reduction of 350, at one round of
    256 x 256, at 640."""
    for (m, n, k, *us), tile in zip(MANY, tiles([c[:3] + (0, 0) for c in MANY])):
        assert us[{0: 0, 1: 1, 2: 2, 6: 3, 7: 4}[tile]] <= 1.06 * min(us), (m, n, k, tile)
    #  256 x 256: 1, walked: 7
    lines = {(511 * 128, 128, 384): 2, (512 * 128, 128, 384): 7, (600 * 128, 128, 320): 0, (600 * 128, 128, 384): 7, (200 * 256, 256, 128): 1, (180 * 256, 256, 64): 0,
             (256 * 256, 256, 576): 1, (257 * 256, 256, 576): 7, (300 * 256, 256, 576): 7, (500 * 256, 256, 1024): 1}
    assert {c: t for c, t in zip(lines, tiles([c + (0, 0) for c in lines]))} == lines
    # walked only where nothing is read, and never one slab
    assert all(t != 7 for beside in (1, 2, 3, 4, 5, 6) for t in tiles([c[:3] + (0, beside) for c in MANY]))
    assert all(t != 7 for t in tiles([(m, n, 64, 0, 0) for m, n, *_ in MANY]))


def test_gelu_epilogue_refuses_what_it_cannot_store():
    """The second tensor moves in 16-byte pieces: misaligned, missing or short ones are refused before anything is launched, and so are
    fp32, 64 columns and fewer, and channel counts that are not whole pieces (made-up addresses, every call is refused)."""
    from paper_2403_08837_amd import binding as b
    ok = dict(dtype=BF16, rows=512, cin=128, cout=128, ws=4096, bytes=512 * 128 * 2)
    for which in (10, 11):
        for bad in (dict(ws=4104), dict(ws=4098), dict(ws=0), dict(bytes=512 * 128 * 2 - 1), dict(bytes=0), dict(dtype=F32), dict(cin=64, cout=64),
                    dict(cin=100, cout=100)):
            c = dict(ok, **bad)
            with pytest.raises(b.CdpError) as e:
                b.cdp_k_conv(c["dtype"], which, 256, 256, 256, 1, 1, c["rows"], c["cin"], c["cout"], 1, 1, 0, ws_ptr=c["ws"], ws_bytes=c["bytes"])
            assert e.value.code == b.CDP_EINVAL, bad
    with pytest.raises(b.CdpError) as e:
        b.cdp_k_conv(BF16, 12, 256, 256, 256, 1, 1, 512, 128, 128, 1, 1, 0)
    assert e.value.code == b.CDP_EINVAL


# bf16 backward; samples, tokens, heads, width of a head, us in separate kernels, us in the fused ones
ATTENTION = [(6, 416, 12, 48, 87.5, 123.8), (4, 656, 12, 48, 152.7, 199.2), (8, 500, 12, 48, 140.8, 156.1), (64, 416, 8, 48, 518.3, 598.0),
             (8, 624, 8, 48, 156.4, 191.8), (1, 656, 12, 48, 78.1, 85.8), (6, 416, 12, 80, 123.6, 137.3), (1, 384, 4, 80, 45.2, 46.9),
             (8, 416, 8, 80, 119.9, 72.2), (64, 300, 4, 80, 218.8, 159.0), (8, 577, 8, 48, 263.1, 225.5), (8, 577, 8, 64, 268.8, 165.8),
             (8, 624, 8, 64, 158.8, 128.9), (64, 261, 4, 48, 178.5, 112.9), (8, 300, 8, 48, 63.3, 41.7), (32, 196, 12, 64, 101.0, 52.0)]


def test_attention_backward_takes_the_faster_kernels(fused):
    for (b, t, h, dh, apart, together), one in zip(ATTENTION, fused([(1, BF16, b, t, h * dh, h) for b, t, h, dh, _, _ in ATTENTION])):
        assert (together if one else apart) <= 1.02 * min(apart, together), (b, t, h, dh)


# fp32, 128 x 128 tile asked for; M, N, K, us on the generic kernel, us on the weight-gradient tiles
ROW_CONTIGUOUS = [(4001, 3003, 1, 28.1, 38.1), (4001, 3003, 16, 29.0, 39.6), (4001, 3003, 2000, 830, 945), (4672, 2321, 12, 24.8, 38.4),
                  (4673, 2320, 32, 35.3, 40.1), (3001, 7001, 200, 219, 238), (2601, 3101, 16, 27.7, 35.0), (4672, 2320, 12, 23.9, 28.2),
                  (4672, 2320, 17, 34.7, 28.2), (4672, 2320, 64, 45.4, 29.5), (40000, 300, 12, 40.1, 46.7), (20000, 600, 8, 38.6, 42.5),
                  (20000, 600, 24, 54.2, 42.9), (4096, 4096, 8, 39.5, 30.0), (600, 20000, 8, 41.4, 29.0), (2004, 2004, 8, 19.5, 12.5),
                  (1001, 2003, 8, 21.0, 10.0), (1000, 2000, 1, 19.5, 11.0), (64, 64, 8, 17.0, 7.0)]


def test_row_contiguous_products_take_the_faster_kernel(wgrad_tiles):
    got = wgrad_tiles([(0, m, n, k, m, n, F32) for m, n, k, _, _ in ROW_CONTIGUOUS])
    for (m, n, k, generic, tiles_us), on_tiles in zip(ROW_CONTIGUOUS, got):
        assert (tiles_us if on_tiles else generic) <= 1.02 * min(generic, tiles_us), (m, n, k)
    # the other tiles of the generic kernel, and bf16, never were faster
    assert all(wgrad_tiles([(s, m, n, k, m, n, dt) for m, n, k, _, _ in ROW_CONTIGUOUS for s, dt in ((1, F32), (2, F32), (0, BF16))]))
