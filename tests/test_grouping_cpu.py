"""The one-wave grouping of few pairs (App. A), the kernel's own text compiled for
the CPU (grouping_cpu.cpp): indices in range, and union-find's groups, offsets
and members, whatever the order of the lanes between the wave's waits."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "..", "paper_1404_2324_amd", "csrc", "massive.hip")


def test_group_few_on_the_cpu(tmp_path):
    src = open(SRC).read()
    a = src.index("constexpr int kFewU")
    b = src.index("// The grouping of ne_all encounter pairs by one workgroup", a)
    text = src[a:b]
    assert text.count("int* gm") == 1
    (tmp_path / "group_few.inc").write_text(text.replace("int* gm", "Ptr gm"))
    exe = str(tmp_path / "grouping")
    subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-Wno-unknown-pragmas", "-I",
                    str(tmp_path), os.path.join(HERE, "grouping_cpu.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
