"""How graph replay cuts a run of blocks into launches
(paper_2509_04390_amd/csrc/batch.hpp), built for the host with g++: every
block once, in order, 16 at most, and no batch of fewer than three (three
launches where one or two blocks take one or two)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_runs_are_cut_into_whole_batches_and_single_blocks(tmp_path):
    exe = str(tmp_path / "batch_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2509_04390_amd", "csrc"),
                    os.path.join(ROOT, "tests", "batch_driver.cpp"), "-o", exe], check=True)
    asked = [(b, n) for b in (0, 1) for n in range(1, 70)]
    out = subprocess.run([exe], input="".join("%d %d\n" % a for a in asked), capture_output=True,
                         text=True, check=True).stdout.splitlines()
    for (b, n), line in zip(asked, out):
        parts = [int(v) for v in line.split()]
        assert sum(parts) == n and max(parts) <= 16
        if not b:
            assert parts == [1] * n
        else:
            assert all(p == 1 or p >= 3 for p in parts)
            assert parts == [16] * (n // 16) + ([n % 16] if n % 16 >= 3 else [1] * (n % 16))
