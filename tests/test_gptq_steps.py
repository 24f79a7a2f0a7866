"""How the factorisation's tiles are divided over its launches (csrc/gptq_steps.hpp, host code)."""
import os
import shutil
import subprocess

import pytest

import test_gpu_gptq as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "gptq_steps.hpp"
using namespace dymoe;
int main(int n, char** a)
{
    if (n == 4) {       // workgroups behind each panel of 256 columns, negative: the small ones
        const long N = atol(a[1]), K = atol(a[2]);
        for (long base = 0; base < K; base += 256) {
            const GqBehindGrid g = gq_behind_grid(N, K, base, base + 256 < K ? base + 256 : K, atol(a[3]));
            std::printf("%ld ", g.small ? -g.workgroups : g.workgroups);
        }
        return 0;
    }
    const long num_cu = atol(a[1]);
    for (long nb = 1; nb <= 1024; nb += nb < 300 ? 1 : 61) {
        for (long q = 0; 2 * q + 2 < nb; q++) {
            const long k = 2 * q + 2;
            const GqWide even = gq_wide(nb, k, num_cu), odd = gq_wide(nb, k + 1, num_cu);
            const long rest = even.first + even.later;
            if (k + 1 < nb && k + 2 < nb && (odd.first != even.first || odd.later != even.later || odd.near != even.near)) return 1;
            if (even.first < 0 || even.later < 0 || (k + 2 >= nb && k + 1 < nb && even.later)) return 2;
            if (k + 2 >= nb) continue;
            const long first = gq_wide_blocks(even, k), second = gq_wide_blocks(odd, k + 1), all = first + second;
            if (first < 0 || second < 0) return 3;
            // not longer than in halves, or as near to halves as the tiles allow
            long half = (all / 2 - (first - 2 * even.first)) / 2;
            half = half < 0 ? 0 : half > rest ? rest : half;
            const long f = first - 2 * even.first + 2 * half;
            if (gq_launch_length(nb, num_cu, first) + gq_launch_length(nb, num_cu, second) >
                gq_launch_length(nb, num_cu, f) + gq_launch_length(nb, num_cu, all - f)) return 4;
            for (const long blocks : {first, second}) {
                const long w = gq_workers(nb, num_cu, blocks);
                if (w < 0 || w > num_cu || (blocks > 0 && w == 0)) return 5;
            }
        }
    }
    // 8192 columns on 256 compute units: equal halves take 1010.6 blocks' time
    double split = 0.0;
    for (long k = 2; k < 128; k++) split += gq_launch_length(128, 256, gq_wide_blocks(gq_wide(128, k, 256), k));
    std::printf("%.1f\n", split);
    if (split > 975.0) return 6;
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("steps")
    src, exe = d / "steps.cpp", d / "steps"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2603_19172_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("num_cu", [256, 304, 64, 8])
def test_a_panels_launches_take_all_tiles_in_the_fewest_rounds(program, num_cu):
    r = subprocess.run([program, str(num_cu)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    print(r.stdout)


def test_the_gpu_tests_reach_both_kernels_of_the_columns_behind(program):
    for kind, sizes in G.CORRECTIONS.items():
        for N, K, _ in sizes:
            r = subprocess.run([program, str(N), str(K), "256"], check=True, capture_output=True, text=True)
            launches = [int(v) for v in r.stdout.split()]
            assert {"small": min(launches) < 0, "large": max(launches) > 0, "none": not any(launches)}[kind], (N, K, launches)
            # the large kernel's values: of the matrix behind the second panel, of the working copy behind later ones
            if (N, K) == (12353, 960):
                assert launches[1] > 0 and launches[2] > 0
