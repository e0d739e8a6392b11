"""Helpers that the kernels share with the host code, compiled here for the host:
what a plan kernel reads off a sort key, over every width of the agent ids, and
the words of a plan's result."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(tmp_path, body):
    src = tmp_path / "t.cpp"
    src.write_text('#include <cstdio>\n#include <cstring>\n#include "ss_internal.h"\n'
                   "using namespace ss;\nint main() {\n" + body + "\nreturn 0;\n}\n")
    exe = tmp_path / "t"
    subprocess.run(["g++", "-std=c++17", "-O3", "-Wall", "-Wstrict-aliasing=1",
                    "-Werror=strict-aliasing", "-Wno-attributes", "-Wno-unused-result",
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


def test_words_of_a_result(tmp_path):
    """The words hold what was last stored in the members, also where the
    compiler may assume that members and words don't alias."""
    r = run(tmp_path, """
    for (unsigned k = 1; k < 1000; ++k) {
        PlanResult r = {};
        r.status = -(int)k;
        r.n_victims = k; r.n_loads = 2 * k; r.n_demand = 3 * k; r.n_demand_victims = 4 * k;
        r.units_out = 5ull * k; r.units_written = ~0ull - k;
        u64 w[sizeof(PlanResult) / 8];
        words_of(r, w);
        r.n_victims = 7;
        PlanResult back;
        memcpy(&back, w, sizeof back);
        if (back.status != -(int)k || back.n_victims != k || back.n_loads != 2 * k ||
            back.n_demand != 3 * k || back.n_demand_victims != 4 * k ||
            back.units_out != 5ull * k || back.units_written != ~0ull - k) return 1;
    }
    """)
    assert r.returncode == 0
