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


def test_streaming_steps_with_the_dynamic_map(ask):
    n = 462 << 20
    assert ask(*[f"percu {B} 1 {n}" for B in (1024, 2048, 4096, 8192)], f"percu 8192 0 {n}") == \
        [[2, 2], [3, 2], [3, 2], [0, 0], [2, 2]]
