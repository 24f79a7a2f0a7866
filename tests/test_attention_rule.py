"""Which kernels the attention score takes (csrc/attention_rule.hpp, host code): the choice at sizes where all of them were measured."""
import os
import shutil
import subprocess

import pytest

import test_gpu_attention as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NUM_CU = 256


@pytest.fixture(scope="module")
def owners(tmp_path_factory):
    """owners(d, causal, heads, T): tokens per block in units of 64 (0 for the narrow pair) and wavefronts of a workgroup"""
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("rule")
    src, exe = d / "rule.cpp", d / "rule"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "attention_rule.hpp"\n'
                   'int main(int, char** a) { auto c = dymoe::attn_choice((atoi(a[4]) + 31) / 32, atoi(a[3]), atoi(a[2]), atoi(a[1]), '
                   'atoi(a[5])); std::printf("%d %d\\n", c.owners, c.waves); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2603_19172_amd", "csrc"), str(src), "-o", str(exe)], check=True)

    def ask(d_, causal, heads, T, num_cu=NUM_CU):
        out = subprocess.run([str(exe)] + [str(int(v)) for v in (d_, causal, heads, T, num_cu)], check=True, capture_output=True,
                             text=True).stdout
        return tuple(int(v) for v in out.split())
    return ask


FORMS = {128: [(0, 4), (2, 8), (4, 8), (2, 4)], 64: [(0, 4), (2, 8), (2, 4)]}

# us of the whole score: head size, causal, heads, tokens; the forms in this order
MEASURED = [
    (128, 1, 16, 320, 14.1, 18.1, 22.4, 17.7), (128, 0, 16, 257, 13.9, 15.9, 19.1, 15.6), (128, 1, 20, 512, 26.1, 19.3, 28.1, 20.8),
    (128, 0, 20, 512, 27.0, 18.1, 24.7, 18.6), (128, 0, 8, 1200, 44.7, 30.4, 45.4, 34.7), (128, 0, 24, 400, 23.5, 17.5, 22.8, 18.1),
    (128, 1, 4, 2500, 72.2, 50.8, 84.0, 60.7), (128, 0, 1, 5000, 100.3, 88.5, 150.2, 108.3), (128, 1, 16, 4096, 292.0, 93.8, 128.2, 101.3),
    (128, 1, 24, 5000, 609.3, 205.6, 187.5, 193.7), (128, 0, 16, 5000, 719.4, 272.5, 313.4, 265.0), (128, 0, 32, 3500, 712.4, 275.0, 231.7, 246.1),
    (128, 1, 64, 2048, 311.9, 112.4, 94.8, 91.7), (128, 0, 24, 2048, 189.9, 81.8, 69.5, 73.2), (128, 1, 44, 1600, None, 66.1, 60.8, 53.6),
    (128, 0, 44, 1600, None, 110.0, 110.7, 92.2), (128, 1, 32, 4096, 549.8, 182.7, 159.8, 166.3), (128, 0, 80, 1600, None, 179.3, 168.8, 145.9),
    (128, 1, 96, 512, 53.4, 31.2, 29.9, 24.6), (128, 0, 96, 512, 63.0, 34.0, 26.4, 26.5),
    (64, 1, 48, 320, 13.8, 17.0, 16.3), (64, 0, 4, 1700, 23.6, 32.0, 35.5), (64, 0, 8, 2048, 38.6, 34.4, 38.9),
    (64, 1, 8, 2048, 31.6, 35.7, 40.6), (64, 0, 8, 2500, 64.4, 41.0, 46.9), (64, 1, 24, 700, 18.3, 21.2, 22.2),
    (64, 0, 24, 700, 25.7, 20.1, 20.6), (64, 1, 20, 1000, 32.5, 24.3, 26.2), (64, 1, 8, 3000, 52.8, 48.0, 56.3),
    (64, 1, 4, 6000, 99.4, 82.4, 99.0), (64, 0, 2, 8000, 122.8, 105.0, 127.0), (64, 1, 24, 2048, 74.4, 39.8, 42.0),
    (64, 1, 64, 2500, 234.4, 127.9, 89.1), (64, 1, 64, 3000, 319.2, 169.9, 120.1), (64, 1, 48, 3000, 247.1, 134.2, 95.3),
    (64, 1, 32, 6000, 579.5, 271.0, 210.9), (64, 0, 48, 2048, 193.5, 98.1, 79.5), (64, 0, 32, 1400, 72.9, 50.6, 42.7),
    (64, 0, 24, 1400, 62.0, 50.7, 43.0), (64, 0, 32, 4096, 487.2, 225.8, 193.7)]


@pytest.mark.parametrize("measured", MEASURED, ids=lambda m: "d%d-causal%d-%dx%d" % (m[0], m[1], m[3], m[2]))
def test_the_form_taken_is_the_fastest_measured(owners, measured):
    us = {form: t for form, t in zip(FORMS[measured[0]], measured[4:]) if t is not None}
    taken = owners(*measured[:4])
    assert us[taken] <= 1.05 * min(us.values())


@pytest.mark.parametrize("num_cu", [1, 7, 32, 256, 304, 2000])
def test_any_chip_and_any_size_has_an_answer(owners, num_cu):
    for d in (64, 128):
        for causal in (0, 1):
            for heads, T in ((1, 1), (65535, 33), (3, 300), (8, 300), (24, 1400), (48, 7000), (1, 2 ** 31 - 1 - 31)):
                assert owners(d, causal, heads, T, num_cu) in FORMS[d]


def test_the_gpu_tests_take_the_forms_they_name(owners):
    for T, heads, _, d in G.THREE_ON_A_UNIT:
        assert owners(d, 1, heads, T) == owners(d, 0, heads, T) == (2, 4)
    for T, heads, _, causal in G.TWO_ON_A_UNIT:
        assert owners(128, causal, heads, T) == (2, 4)
    for T, heads, _, causal in G.BLOCKS_OF_256:
        assert owners(128, causal, heads, T) == (4, 8)
    for d, causal, heads, _, T, form, behind in G.AROUND_THE_LINES:
        assert (owners(d, causal, heads, T), owners(d, causal, heads, T + 1)) == (form, behind)
    assert (owners(128, 1, 64, 900), owners(128, 0, 64, 900), owners(64, 1, 64, 900)) == ((2, 4), (4, 8), (2, 4))
