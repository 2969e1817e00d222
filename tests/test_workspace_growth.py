"""How much the library-owned workspace grows by, in a host program of its own (no device)."""
import os
import subprocess


def test_the_workspace_falls_back_to_what_is_needed(tmp_path):
    """The library-owned workspace grows in steps of 32 MB, and by what a call needs where such a step does not fit."""
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_08192_amd", "csrc")
    src = tmp_path / "grow.cpp"
    src.write_text("""
#include <stdio.h>
#include <initializer_list>
#include "ta_params.h"
static size_t room, asked;
static void *take(size_t n) { asked += 1; return n <= room ? &room : nullptr; }
int main()
{
    const size_t MB = 1 << 20;
    for (size_t r : {100 * MB, 40 * MB, 31 * MB, 3 * MB, 2 * MB})
        for (size_t need : {100000 * (size_t)1, 3 * MB, 32 * MB, 33 * MB}) {
            void *p = nullptr;
            room = r; asked = 0;
            const size_t got = ta_host_grow(need, take, &p);
            const size_t fit = (need + 32 * MB - 1) / (32 * MB) * 32 * MB, least = (need + MB - 1) / MB * MB;
            const size_t want = fit <= r ? fit : least <= r ? least : 0;
            if (got != want || (got != 0) != (p != nullptr) || asked > 2) { printf("%zu %zu %zu %zu", r, need, got, want); return 1; }
        }
    return 0;
}
""")
    exe = str(tmp_path / "grow")
    out = subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-I" + csrc, str(src), os.path.join(csrc, "ta_host.cpp"),
                          "-o", exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert out.returncode == 0, out.stdout
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert out.returncode == 0, out.stdout
