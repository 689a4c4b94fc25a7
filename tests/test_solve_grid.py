"""The choice of a solve's kernel and grid (solve_grid in csrc/p2m_host.hpp) over every
small pair of resident counts: the grid never exceeds what its own kernel holds at once
(its barriers would wait for workgroups that cannot start), no tile is left without a
workgroup, and the streaming kernel runs exactly where the resident one does not fit.
Host compiler, CPU only."""
import shutil
import subprocess

import pytest

from test_host_sanitizers import ROOT

SRC = """
#include <cstdio>
#include "paper_1610_05258_amd/csrc/p2m_host.hpp"
int main() {
    int bad = 0;
    for (int held = -1; held <= 12; ++held)
        for (int hs = -1; hs <= 12; ++hs)
            for (int nt = 0; nt <= 30; ++nt) {
                const p2m::SolveGrid g = p2m::solve_grid(held, hs, nt);
                const int own = g.stream ? hs : held;
                const bool runs = nt > 0 && (nt <= held || hs > 0);
                bool ok = runs ? g.groups >= 1 && g.groups <= own && g.groups <= nt : g.groups == 0;
                if (runs) ok = ok && g.stream == (nt > held) && (g.stream || g.groups == nt);
                if (!ok) ++bad, std::printf("held %d stream %d tiles %d -> %d %d\\n", held, hs, nt, g.groups, (int)g.stream);
            }
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_solve_grid(tmp_path):
    src = tmp_path / "grid.cpp"
    src.write_text(SRC)
    exe = tmp_path / "grid"
    r = subprocess.run(["g++", "-std=c++17", "-I", ROOT, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
