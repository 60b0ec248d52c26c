"""The rules that send products of 33 to 256 rows to the kernel with a wave per 32 rows, compiled from the library's source for the host: every product that
they take has an instance, every instance is reached, and the limits lie where they were measured."""
import ctypes
import os
import re
import subprocess

import pytest

import paper_2511_16665_amd

SRC = open(os.path.join(os.path.dirname(paper_2511_16665_amd.__file__), "csrc", "gemm.hip")).read()


def _function(name):
    return re.search(rf"^static [\w ]+ {name}\([^)]*\) {{\n.*?^}}\n", SRC, re.M | re.S).group(0)


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    names = {"mid_glu_width": "int, int, int", "mid_glu_four": "int, int, int", "mid_split_plan": "int, int, int, int, int, int*", "few_glu_width": "int, int, int"}
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text("\n".join(_function(n) for n in names) + 'extern "C" {\n' + "\n".join(
        f"int x_{n}({', '.join(f'{t.strip()} a{i}' for i, t in enumerate(ts.split(',')))}) {{ return {n}({', '.join(f'a{i}' for i in range(len(ts.split(','))))}); }}"
        for n, ts in names.items()) + "\n}\n")
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-o", str(d / "r.so"), str(d / "r.cpp")], check=True)
    return ctypes.CDLL(str(d / "r.so"))


def _glu_instances():
    """{(four sums, waves, blocks)} of launch_mid_glu."""
    body = _function("launch_mid_glu")
    four, one = body.split("#undef TLT_MID")[:2]
    return {(f, int(a), int(b)) for f, part in ((True, four), (False, one)) for a, b in re.findall(r"TLT_MID\((\d), (\d)\)", part)}


KS = [64, 128, 448, 512, 576, 960, 1024, 1088, 2496, 2560, 2624, 3584, 8192]


def test_gate_up_every_product_has_an_instance_and_every_instance_a_product(rules):
    reached = set()
    for N in range(128, 32768, 128):
        for K in KS:
            for M in (1, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256, 257):
                wtn = rules.x_mid_glu_width(M, N, K)
                if wtn:
                    assert 32 < M <= 256 and -(-N // (16 * wtn)) <= 256
                    reached.add((bool(rules.x_mid_glu_four(M, wtn, K)), (M + 31) // 32, wtn))
    assert reached == _glu_instances()


@pytest.mark.parametrize("M,N,K,wtn,four", [
    (33, 8192, 64, 2, 1), (64, 8192, 64, 2, 1), (65, 8192, 960, 0, 0), (65, 8192, 1024, 2, 0), (128, 8192, 1024, 2, 0), (129, 8192, 4096, 0, 0),
    (64, 12288, 960, 0, 0), (64, 12288, 1024, 3, 1), (65, 12288, 1024, 3, 0), (129, 12288, 448, 0, 0), (256, 12288, 512, 3, 0), (257, 12288, 512, 0, 0),
    (33, 16384, 1024, 0, 0), (64, 16384, 8192, 0, 0), (65, 16384, 448, 0, 0), (65, 16384, 512, 4, 1), (128, 16384, 512, 4, 1), (129, 16384, 512, 4, 0),
    (33, 20480, 64, 5, 0), (64, 20480, 960, 5, 0), (64, 20480, 1024, 5, 1), (65, 20480, 2496, 5, 0), (128, 20480, 2560, 5, 1), (224, 20480, 2560, 5, 0),
    (225, 20480, 2560, 0, 0), (64, 24576, 1024, 6, 1), (128, 24576, 2560, 6, 1), (224, 24576, 64, 6, 0), (225, 24576, 64, 0, 0),
    (33, 28672, 128, 0, 0), (64, 28672, 2496, 0, 0), (64, 28672, 2560, 7, 1), (65, 28672, 64, 7, 0), (128, 28672, 2560, 7, 0), (192, 28672, 2560, 7, 0),
    (193, 28672, 2560, 0, 0), (64, 28800, 2560, 0, 0),
])
def test_gate_up_limits(rules, M, N, K, wtn, four):
    assert rules.x_mid_glu_width(M, N, K) == wtn
    if wtn:
        assert bool(rules.x_mid_glu_four(M, wtn, K)) == bool(four)


def test_cuts_along_k_fit_the_chip_the_buffer_and_the_ring(rules):
    """Cuts of six K steps at least, one workgroup per CU at most, no more slices than the caller has room for."""
    cuts, taken = ctypes.c_int(), 0
    for N in range(128, 16384, 128):
        for K in KS + [18944, 28672]:
            for M in (32, 33, 128, 129, 224, 225, 256, 257):
                for general in (1, 2, 4, 9, 12):
                    for room in (1, 2, 5, 12):
                        cuts.value = -1
                        if not rules.x_mid_split_plan(M, N, K, general, room, ctypes.byref(cuts)):
                            continue
                        taken += 1
                        tiles = N // (64 if M <= 128 else 128)
                        assert 32 < M <= 256 and 2 <= cuts.value <= room and 200 <= tiles * cuts.value <= 256 and K // 64 // cuts.value >= 6
    assert taken > 1000


def test_every_gate_up_instance_is_run_by_the_product_tests(rules):
    """By the cases that compare products of random operands, from their parameters."""
    test_gpu_mid_rows, test_gpu_few_rows = (pytest.importorskip(m) for m in ("test_gpu_mid_rows", "test_gpu_few_rows"))
    run = set()
    for f in (test_gpu_mid_rows.test_bf16_gate_up, test_gpu_few_rows.test_bf16_gate_up):
        for M, N, K in f.pytestmark[0].args[1]:
            wtn = rules.x_mid_glu_width(M, N, K)
            if wtn:
                run.add((bool(rules.x_mid_glu_four(M, wtn, K)), (M + 31) // 32, wtn))
    assert run == _glu_instances()


def test_the_gate_up_cases_are_told_apart_by_their_sums(rules):
    """The cases that are compared bit for bit with one chain are those that have one."""
    m = pytest.importorskip("test_gpu_mid_rows")
    for M, N, K in m.test_bf16_gate_up.pytestmark[0].args[1]:
        wtn = rules.x_mid_glu_width(M, N, K)
        assert ((M, N, K) in m.FOUR_SUMS) == bool(wtn and rules.x_mid_glu_four(M, wtn, K)), (M, N, K)
