"""The LDS of consecutive work items of the persistent batch kernel, on the
CPU: stencil_item, as it stands in the source, runs with stand-ins that record
what a block does.  A brick ends with reads of its LDS and a marching tile
begins with writes to LDS that overlays it, so a barrier has to lie between a
brick and whatever item follows."""
import itertools
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2603_19371_amd", "csrc")

HARNESS = r"""
#include <algorithm>
#include <cstdio>
#define __device__
#define __forceinline__ inline
using std::min;
constexpr int kT3 = 8, kTY = 8;
struct Geom { int nz = 1; };
struct Tiling { int cz = 1; };
struct BatchPair { Geom g; Tiling t; int bricks; };
struct Pol { struct Local {}; };
static void __syncthreads() { putchar('|'); }
template <int S> void brick_origin(const Geom&, int, int&, int&, int&) {}
void tile_origin(const Tiling&, int, int, int& x, int& y, int& z) { x = y = z = 0; }
template <int R, class... A> void stencil_cube(A&&...) { putchar('b'); }
template <int R, int TY, bool FENCE = true, class... A> void stencil_tile(A&&...) { putchar('t'); }
%s
int main(int, char** argv) {
  int lm = 0, lb = 0;
  Pol::Local loc;
  for (const char* c = argv[1]; *c; ++c) {
    BatchPair P;
    P.bricks = *c == 'b';
    stencil_item<3, 2>(Pol(), P, 0, loc, lm, lb);
  }
}
"""


def test_a_barrier_follows_every_brick(tmp_path):
    src = open(os.path.join(CSRC, "batch_attempt.h")).read()
    item = re.search(r"template <int R, int FORM, class Pol, class LM, class LB>\n"
                     r"__device__ __forceinline__ void stencil_item\(.*?\n}\n", src, re.S).group(0)
    cpp, exe = tmp_path / "order.cpp", tmp_path / "order"
    cpp.write_text(HARNESS.replace("%s", item))
    subprocess.run(["g++", "-std=c++17", "-o", exe, cpp], check=True)
    for seq in map("".join, itertools.product("bt", repeat=3)):
        got = subprocess.run([exe, seq], capture_output=True, text=True, check=True).stdout
        assert got.replace("|", "") == seq, got
        assert not re.search("b[bt]", got), (seq, got)
