"""The table of resident workgroups that the weight-stationary kernel's shape
choice reads (csrc/resident_table.h), in a CPU build: every (device, shape, LDS
size) is queried once, however many others are in use, and a failed query is
not kept.
"""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "resident_table.h"
using namespace sl;
static ResidentTable<3, 7, 160 * 1024> table;
int main()
{
    int queries = 0, bad = 0;
    for (int pass = 0; pass < 3; ++pass)
        for (int d = 0; d < 3; ++d)
            for (int s = 0; s < 7; ++s)
                for (size_t lds = 0; lds <= 160 * 1024; lds += 256) {
                    const int want = (int)(lds / 256 * 3 + s * 11 + d) % 8193;
                    int got = -1;
                    const sl_status st = table.get(d, s, lds, &got, [&](int *out) {
                        ++queries;
                        *out = want;
                        return SL_OK;
                    });
                    bad += st != SL_OK || got != want;
                }
    printf("%d %d ", queries, bad);
    // a failure is passed on and asked again; sizes off the table's step and
    // devices past its end are asked each time
    static ResidentTable<1, 1, 1024> t;
    int calls = 0, out = 0;
    auto fail = [&](int *) { ++calls; return SL_ERR_HIP; };
    auto ok = [&](int *o) { ++calls; *o = 5; return SL_OK; };
    bad = t.get(0, 0, 512, &out, fail) != SL_ERR_HIP;
    bad += t.get(0, 0, 512, &out, ok) != SL_OK || out != 5;
    bad += t.get(0, 0, 512, &out, fail) != SL_OK || out != 5;
    for (int i = 0; i < 2; ++i) bad += t.get(0, 0, 100, &out, ok) != SL_OK || t.get(1, 0, 512, &out, ok) != SL_OK;
    printf("%d %d\n", calls, bad);
}
"""


def test_each_pair_is_queried_once(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2211_07715_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()
    assert out == [str(3 * 7 * 641), "0", "6", "0"], out
