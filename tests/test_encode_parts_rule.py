"""How many workgroups share a plaintext's limbs (encode_parts in csrc/encode.hpp),
on the CPU: one where more of them only queue on the same CUs, several where CUs
would idle, never more than there are limbs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include <cstdio>
#include <cstdlib>
#include "encode.hpp"
int main(int argc, char** argv) {
  for (int i = 1; i + 2 < argc; i += 3)
    std::printf("%d\\n", pvfl::encode_parts(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoi(argv[i + 2])));
}
"""


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    d = tmp_path_factory.mktemp("parts")
    (d / "parts.hip").write_text(SRC)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-w", "-I",
                    os.path.join(ROOT, "paper_2405_00482_amd", "csrc"), str(d / "parts.hip"), "-o", str(d / "parts")],
                   check=True, capture_output=True)

    def run(cases):
        args = [str(x) for c in cases for x in c]
        out = subprocess.run([str(d / "parts"), *args], check=True, capture_output=True, text=True).stdout
        return [int(x) for x in out.split()]
    return run


def test_workgroups_that_would_queue_are_not_made(parts):
    # (log N, plaintexts, limbs): every CU has a workgroup, or the last limbs' share would be a second round
    cases = [(13, 192, 3), (13, 224, 3), (13, 256, 3), (13, 160, 2), (12, 512, 2), (14, 160, 4), (15, 512, 8), (14, 4096, 5)]
    assert parts(cases) == [1] * len(cases)


def test_idle_cus_are_used(parts):
    cases = [(12, 1, 2), (13, 1, 3), (13, 64, 3), (13, 128, 2), (14, 1, 4), (14, 64, 4), (14, 128, 4), (15, 16, 8)]
    assert parts(cases) == [2, 3, 3, 2, 4, 4, 2, 8]


def test_never_more_than_the_limbs(parts):
    cases = [(n, c, l) for n in (12, 13, 14, 15) for c in (1, 7, 100, 255, 257, 1000) for l in (1, 2, 5, 17)]
    got = parts(cases)
    assert all(1 <= p <= l for p, (_, _, l) in zip(got, cases))
