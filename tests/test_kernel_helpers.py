"""Helpers that the kernels share with the host code, compiled here for the host:
what a plan kernel reads off a sort key, over every width of the agent ids."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(tmp_path, body):
    src = tmp_path / "t.cpp"
    src.write_text('#include <cstdio>\n#include <cstring>\n#include "ss_internal.h"\n'
                   "using namespace ss;\nint main() {\n" + body + "\nreturn 0;\n}\n")
    exe = tmp_path / "t"
    subprocess.run(["g++", "-std=c++17", "-O3", "-Wall", "-Wno-attributes", "-Wno-unused-result",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2601_21473_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)


def test_distance_of_a_key(tmp_path):
    """Every distance comes back from its key whatever the id's width (31 bits:
    more than 2^30 agents), with a tag where one fits and without."""
    r = run(tmp_path, """
    const unsigned ds[] = {0u, 1u, 1023u, 0x3FFFFFFFu, 0x40000000u, 0x7FFFFFFFu, 0x80000000u,
                           0xC0000001u, 0xFFFFFFFEu, 0xFFFFFFFFu};
    for (unsigned b = 1; b <= 31; ++b)
        for (unsigned d : ds)
            for (u64 id : {0ull, (1ull << b) - 1})
                for (u64 tag : {0ull, kTagL, kTagC}) {
                    if (tag && b + 32 > kTagShift) continue;
                    const u64 key = ((u64)d << b) | id | tag;
                    if (key_distance(key, b) != d) { printf("bits %u distance %u\\n", b, d); return 1; }
                }
    """)
    assert r.returncode == 0, r.stdout
