"""The GEMM dispatch rule (csrc/gemm_route.hpp) compiled for the host."""

from __future__ import annotations

import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2508_02343_amd", "csrc", "gemm_route.hpp")
MAIN = """
#include <cstdio>
#include "%s"
int main() {
  long long m, n;
  mm::GemmSizes z;
  while (scanf("%%lld %%lld %%d %%d %%d %%d", &m, &n, &z.steps[0], &z.steps[1], &z.steps[2], &z.cus) == 6) {
    z.m = m;
    z.n = n;
    const mm::GemmRoute r = mm::gemm_route(z);
    int tn = 8, tm = 4;
    const char* name = "direct";
    if (r.kernel == mm::GemmKernel::kTiled128) name = "tiled";
    if (r.kernel == mm::GemmKernel::kTiled256) { name = "tiled"; tm = 8; }
    if (r.kernel == mm::GemmKernel::kSplit) {
      name = "split";
      tn = mm::kSplitShapes[r.shape].tn;
      tm = mm::kSplitShapes[r.shape].tm;
    }
    const mm::DirectPlan p = r.kernel == mm::GemmKernel::kDirect ? mm::direct_plan(m, n, z.cus) : mm::DirectPlan{0, 0};
    printf("%%s %%dx%%d %%lld %%d\\n", name, 32 * tn, 32 * tm, (long long)mm::tile_count(n, m, tn, tm), p.rows);
  }
}
"""


@functools.lru_cache(maxsize=None)
def _program() -> str:
    d = tempfile.mkdtemp(prefix="mm_route_")
    src, exe = os.path.join(d, "route.cpp"), os.path.join(d, "route")
    with open(src, "w") as f:
        f.write(MAIN % HEADER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe, src], check=True)
    return exe


@functools.lru_cache(maxsize=None)
def _run(M: int, N: int, split, cus: int) -> list[str]:
    steps = [-(-(p // 32) // 4) for p in split]
    line = " ".join(str(v) for v in (M, N, *steps, cus))
    return subprocess.run([_program()], input=line, check=True, capture_output=True, text=True).stdout.split()


def route(M: int, N: int, split, cus: int = 256) -> tuple[str, int]:
    """("direct" | "split 64x32" | "tiled 256x128" ..., tiles) of an [M, K] x [N, K]
    product with this split (tiles without a meaning for "direct")."""
    out = _run(M, N, tuple(split), cus)
    return out[0] if out[0] == "direct" else f"{out[0]} {out[1]}", int(out[2])


def kernel(M: int, N: int, split, cus: int = 256) -> str:
    """The compiled kernel such a product takes: as route(), the decode kernel with
    its activation tiles and the weight rows of a strip ("direct 2 tiles 24 rows")."""
    name, _ = route(M, N, split, cus)
    tiles = 1 if M <= 16 else (2 if M <= 32 else 4)
    return f"direct {tiles} tiles {_run(M, N, tuple(split), cus)[3]} rows" if name == "direct" else name
