"""The host's choices between ways of doing the same work (csrc/rules.h), asked on the CPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2608_11919_amd", "csrc")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "rules_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-o",
                    exe, os.path.join(HERE, "rules_driver.cpp")], check=True)

    def run(*requests):
        """One answer per request, as a list of whole numbers."""
        p = subprocess.run([exe], input="\n".join(requests) + "\n", capture_output=True,
                           text=True, check=True)
        return [[int(x) for x in line.split()] for line in p.stdout.splitlines()]
    return run


@pytest.mark.parametrize("flags,takes", [
    (0x0, 1),                        # the default kind
    (0x40000000, 1),                 # coherent
    (0x40000001, 1),                 # coherent, portable
    (0x80000000, 0),                 # non-coherent
    (0xC0000000, 0),                 # both
    (0x1, 0), (0x4, 0),              # portable, write-combined: the kind is not stated
])
def test_copy_kernel_takes_memory_the_gpu_does_not_cache(ask, flags, takes):
    assert ask(f"pinned {flags}") == [[takes]]


@pytest.mark.parametrize("K,longest,geom", [
    (0, 0, [1, 4]), (9, 1024, [1, 4]), (64, 1025, [4, 1]), (1, 40000, [4, 1]),
    (65, 4096, [1, 16]), (325, 2752, [1, 16]), (65, 4097, [4, 4]), (325, 38000, [4, 4]),
])
def test_finish_takes_more_waves_for_few_long_tensors(ask, K, longest, geom):
    assert ask(f"finish {K} {longest}") == [geom]


LINEAR, DYNAMIC = 0, 1


def test_many_tiny_tensors_are_a_small_step(ask):
    """13000 tensors of 64 elements fill 13000 work units of up to 8192 elements, and move
    832000 elements: they keep every workgroup that fits."""
    for B in (1024, 4096):
        for code_map in (LINEAR, DYNAMIC):
            assert ask(f"percu {B} {code_map} 64x13000") == [[0, 0]]
    assert ask("percu 1024 0 100000000 64x13000") == [[2, 2]]


@pytest.mark.parametrize("B", [64, 128, 256, 512, 1024, 4096])
def test_streaming_steps_keep_two_workgroups_per_cu(ask, B):
    assert ask(f"percu {B} 0 {48 << 20}", f"percu {B} 0 {64 << 20}", f"percu {B} 0 {462 << 20}") \
        == [[0, 0], [2, 2], [2, 2]]
    assert ask(f"percu {B} 0 {54 << 20}") == ([[0, 0]] if B == 4096 else [[2, 2]])


def test_streaming_steps_with_the_dynamic_map(ask):
    n = 462 << 20
    assert ask(*[f"percu {B} 1 {n}" for B in (1024, 2048, 4096, 8192)], f"percu 8192 0 {n}") == \
        [[2, 2], [3, 2], [3, 2], [0, 0], [2, 2]]


M = 1 << 20
OTHER_BLOCKS = [B for B in range(64, 65536 + 1, 64) if B & (B - 1) or B > 8192]


def test_every_geometry_holds_its_unit(ask):
    """A unit's elements fit its lanes' granules, its blocks the kernel's LDS words, and the
    kernel is one of those compiled, for every block size over lists of every kind."""
    lists = ["1", "64", "5000", "300x700", "1000x300", "6000x300", "9000x300", "1500x20000",
             f"{M}", f"{5 * M}", f"{13 * M}", f"{33 * M}", f"{50 * M}", f"{200 * M}"]
    requests = [(B, m, l) for B in OTHER_BLOCKS for m in (LINEAR, DYNAMIC) for l in lists]
    answers = ask(*[f"geom {B} {m} {l}" for B, m, l in requests])
    assert len(answers) == len(requests)
    for (B, m, l), (waves, granules, blocks) in zip(requests, answers):
        where = (B, m, l, waves, granules, blocks)
        if waves == 0:
            assert B > 2048 and blocks == 1, where
            continue
        assert B <= 16384, where
        assert (waves, granules) in {(1, 2), (1, 4), (4, 1), (4, 2), (4, 3), (8, 2), (16, 2)}, where
        assert 1 <= blocks <= 16 and (waves == 1 or blocks == 1), where
        assert blocks * B <= 512 * waves * granules, where


@pytest.mark.parametrize("B,code_map,sizes,geom", [
    # few blocks: a workgroup each
    (768, LINEAR, f"{3 * M // 10}", [4, 1, 1]), (384, LINEAR, f"{M // 5}", [4, 1, 1]),
    (192, DYNAMIC, "100000", [4, 1, 1]),
    # small lists: two granules per lane
    (768, LINEAR, f"{M}", [1, 2, 1]), (384, LINEAR, f"{20 * M}", [1, 2, 2]),
    (576, LINEAR, f"{M}", [1, 2, 1]), (640, DYNAMIC, f"{4 * M}", [1, 2, 1]),
    (832, LINEAR, f"{200 * M}", [1, 2, 1]), (192, LINEAR, f"{200 * M}", [1, 2, 5]),
    # large ones, as before
    (768, LINEAR, f"{138 * M}", [1, 4, 2]), (384, LINEAR, f"{138 * M}", [1, 4, 5]),
    (576, DYNAMIC, f"{20 * M}", [1, 4, 3]), (768, DYNAMIC, f"{138 * M}", [1, 2, 1]),
    (1536, LINEAR, "100", [4, 1, 1]), (3072, LINEAR, f"{M}", [4, 2, 1]),
    (5120, DYNAMIC, f"{M}", [4, 3, 1]), (8128, LINEAR, f"{M}", [8, 2, 1]),
    # many short tensors
    (3072, LINEAR, "350x288", [0, 0, 1]), (8128, DYNAMIC, "1000x288", [0, 0, 1]),
    (3072, LINEAR, "1500x9000", [4, 2, 1]), (5120, LINEAR, "3600x288", [4, 3, 1]),
    (12288, LINEAR, "7000x288", [0, 0, 1]), (16384, DYNAMIC, "350x288", [0, 0, 1]),
    (16384, DYNAMIC, "11000x288", [16, 2, 1]), (12288, LINEAR, "6000x100", [16, 2, 1]),
    # block sizes that leave many lanes of sixteen waves idle
    (8256, LINEAR, f"{M}", [16, 2, 1]), (8256, LINEAR, f"{20 * M}", [0, 0, 1]),
    (8256, LINEAR, f"{92 * M}", [16, 2, 1]), (8256, DYNAMIC, f"{92 * M}", [0, 0, 1]),
    (10240, DYNAMIC, f"{32 * M}", [0, 0, 1]), (12288, DYNAMIC, f"{32 * M}", [0, 0, 1]),
    (12288, DYNAMIC, f"{4 * M}", [16, 2, 1]), (12288, DYNAMIC, f"{138 * M}", [16, 2, 1]),
    (12288, LINEAR, f"{138 * M}", [16, 2, 1]), (16384, LINEAR, f"{32 * M}", [16, 2, 1]),
    (16448, LINEAR, f"{32 * M}", [0, 0, 1]),
])
def test_kernels_of_other_block_sizes(ask, B, code_map, sizes, geom):
    assert ask(f"geom {B} {code_map} {sizes}") == [geom]


def test_streaming_fp32_state_steps_keep_three_workgroups_per_cu(ask):
    assert ask("percu32 1000", f"percu32 {20 * M}", f"percu32 {32 * M}", "percu32 3000000000") == \
        [[0], [0], [3], [3]]


def test_other_blocks_are_those_the_power_kernel_does_not_take(ask):
    """Lists of 300 short tensors: the rules for block sizes that are no power of two, or
    above 8192, see their blocks."""
    assert ask("geom 16384 0 350x300", "geom 3072 0 350x300", "geom 192 0 350x300") == \
        [[0, 0, 1], [0, 0, 1], [4, 1, 1]]
