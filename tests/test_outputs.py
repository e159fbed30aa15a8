"""Which outputs the mask gather stores itself (csrc/outputs.h), checked on the host with
g++: aligned memory of the context's own device, and no other; the rest is copied."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "outputs.h"
#include <cstdio>
using namespace gss;
int main() {
    for (int device = 0; device < 8; ++device)
        for (int at = -1; at < 8; ++at)
            for (int mem = 0; mem < 2; ++mem)
                for (uintptr_t a = 4096; a < 4112; ++a) {
                    OutputPlace p;
                    p.device = mem;
                    p.ordinal = at;
                    p.address = a;
                    const bool want = mem == 1 && at == device && a % 8 == 0;
                    if (stores_directly(p, device) != want) { std::printf("%d %d %d %d\n", device, at, mem, (int)(a % 16)); return 1; }
                }
    if (stores_directly(OutputPlace{}, 0)) { std::printf("nowhere\n"); return 1; }
    std::printf("ok\n");
    return 0;
}
"""


def test_direct_stores_are_local(tmp_path):
    src = tmp_path / "outputs_check.cpp"
    exe = tmp_path / "outputs_check"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2012_03119_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
