"""16-byte vectors of a chunk: every vector loaded as a whole lies inside the row, and the others' entries are covered."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "chunk_vectors.hpp"
using specvlm::ChunkVectors;
int main() {
    const int threads = 1024;
    for (int vec : {8, 4})
        for (int V : {65537, 65538, 66559, 66560, 66561, 99254, 131071, 131072, 131073, 152064})
            for (int off = 0; off < vec; ++off) {
                const int bytes = 16 / vec, chunk = (V + threads - 1) / threads;
                const uintptr_t row = 0x100000 + static_cast<uintptr_t>(off) * bytes;
                for (int t = 0; t < threads; ++t) {
                    const int v0 = t * chunk < V ? t * chunk : V, v1 = v0 + chunk < V ? v0 + chunk : V;
                    if (v0 >= v1) continue;
                    const ChunkVectors c(row, v0, v1, V, vec);
                    const int first = v0 - c.lead;
                    if ((row + static_cast<intptr_t>(first) * bytes) % 16) return printf("not on a boundary\n"), 1;
                    if (first + c.count * vec < v1 || first + (c.count - 1) * vec >= v1) return printf("count\n"), 1;
                    for (int k = 0; k < c.count + 3; ++k) {               // as the kernel asks: clamped
                        const int at = (k > c.lo ? k : c.lo) < c.hi ? (k > c.lo ? k : c.lo) : c.hi;
                        const int e = first + at * vec;
                        if (e < 0 || e + vec > V) return printf("V %d off %d thread %d: vector %d at entry %d\n", V, off, t, k, e), 1;
                        const bool inside = first + k * vec >= 0 && first + (k + 1) * vec <= V;
                        if (k < c.count && (k >= c.lo && k <= c.hi) != inside) return printf("V %d off %d thread %d: vector %d\n", V, off, t, k), 1;
                    }
                }
            }
    return 0;
}
"""


def test_whole_vectors_lie_inside_the_row(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2509_11815_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
