"""Which bf16 batches take the few-row kernels (csrc/ffn_thin.hip), asked of the built library on the host."""
import os
import shutil
import subprocess

import pytest

from paper_2503_05066_amd import build, capmoe

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm/include"
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM), reason="g++ and the HIP headers are needed")

HARNESS = r"""
#include <stdio.h>
#include "common.h"
int main() {
    int n, e, k, d, h, mode, dtype;
    double gamma;
    while (scanf("%d %d %d %d %d %d %lf %d", &n, &e, &k, &d, &h, &mode, &gamma, &dtype) == 8) {
        moe_desc_t desc{};
        desc.n_tokens = n, desc.d_model = d, desc.n_experts = e, desc.top_k = k, desc.d_hidden = h, desc.device_groups = 1;
        desc.mode = mode, desc.capacity_scope = 1, desc.gamma = gamma, desc.dtype = dtype;
        if (capmoe::validate(&desc) != 0) { puts("refused"); continue; }
        puts(capmoe::ffn_is_thin(desc, capmoe::derive(desc)) ? "few" : "wide");
    }
}
"""

NONE, TOKEN = capmoe.MODE_NONE, capmoe.MODE_TOKEN_DROP
CASES = [  # tokens, experts, k, d, h, mode, gamma -> kernels
    # no expert can have more than 64 rows: by the average alone
    ((1, 64, 8, 2048, 1024, NONE, 1.0), "few"),
    ((64, 8, 2, 4096, 14336, NONE, 1.0), "few"),
    ((64, 64, 6, 4096, 1408, NONE, 1.0), "few"),
    ((128, 64, 8, 2048, 1024, TOKEN, 1.0), "few"),        # a capacity of 16 rows
    ((256, 32, 2, 2048, 1024, TOKEN, 4.0), "few"),        # of 64
    # an expert may have more
    ((65, 32, 1, 2048, 1024, NONE, 1.0), "few"),
    ((256, 32, 1, 2048, 4096, NONE, 1.0), "few"),         # 256 rows, 8 on average, 2^23 weights of a kind
    ((257, 64, 1, 1024, 1024, NONE, 1.0), "wide"),
    ((256, 31, 1, 1024, 1024, NONE, 1.0), "wide"),
    ((256, 32, 1, 2048, 4224, NONE, 1.0), "wide"),
    ((256, 32, 1, 4096, 14336, NONE, 1.0), "wide"),
    ((128, 16, 1, 4096, 4096, NONE, 1.0), "wide"),
    ((128, 128, 8, 4096, 2048, NONE, 1.0), "wide"),
    ((128, 64, 2, 2048, 2048, NONE, 1.0), "few"),
    ((128, 64, 2, 2048, 2176, NONE, 1.0), "wide"),
    ((129, 64, 2, 1024, 1024, NONE, 1.0), "wide"),
    ((160, 64, 3, 2048, 1024, NONE, 1.0), "wide"),
    ((256, 32, 1, 8192, 1024, NONE, 1.0), "wide"),        # the wide blocks split K there
    ((256, 32, 1, 1024, 8192, NONE, 1.0), "wide"),
    ((256, 32, 1, 8064, 1024, NONE, 1.0), "few"),
    ((256, 32, 1, 4096, 4096, TOKEN, 16.0), "wide"),      # a capacity of 128 rows: no more than all tokens' rows either
]


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    folder = tmp_path_factory.mktemp("rule")
    (folder / "main.cpp").write_text(HARNESS)
    capmoe.load()
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM, "-I", os.path.join(ROOT, "include"), "-I", build.CSRC,
                    str(folder / "main.cpp"), "-o", str(folder / "main"), build.LIB, "-Wl,-rpath," + os.path.dirname(build.LIB),
                    "-Wl,--allow-shlib-undefined"], check=True)
    asked = "".join(" ".join(map(str, c)) + " 1\n" for c, _ in CASES) + "1 8 2 128 128 0 1.0 0\n"
    return subprocess.run([str(folder / "main")], input=asked, capture_output=True, text=True, check=True).stdout.split()


@pytest.mark.parametrize("at", range(len(CASES)), ids=lambda i: "-".join(map(str, CASES[i][0])))
def test_kernels_of_a_batch(answers, at):
    assert answers[at] == CASES[at][1]


def test_fp32_has_none(answers):
    assert answers[-1] == "wide"
