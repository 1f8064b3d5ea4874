"""CPU test of what the launchers ask of the runtime once per GPU (a kernel's largest dynamic LDS): every device
is asked, none twice, a failure again."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include "hgf_once.h"
int main()
{
    static hgf::OncePerDevice once;
    int asked[80] = {};
    for (int round = 0; round < 3; ++round)
        for (int d = 0; d < 80; ++d)
            if (once(d, [&] { return ++asked[d] == 1 && d == 5 ? 7 : 0; }) != (round == 0 && d == 5 ? 7 : 0)) return 1;
    for (int d = 0; d < 80; ++d)
        if (asked[d] != (d >= 64 ? 3 : (d == 5 ? 2 : 1))) return 2;
    return 0;
}
"""


def test_every_device_is_asked_once(tmp_path):
    src, exe = tmp_path / "once.cpp", tmp_path / "once"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2602_05269_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
    # ... and the launchers keep no answer for the whole process
    for name in ("hgf_short.hip", "hgf_batch.hip", "hgf_decode.hip"):
        text = open(os.path.join(ROOT, "paper_2602_05269_amd", "csrc", name)).read()
        assert "static const hipError_t" not in text, name
