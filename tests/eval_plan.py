"""The launches of an evaluation, as eval_plan() of the built library cuts them (on the host, no GPU): a small program linked
against it, built once per process."""
import functools
import os
import shutil
import subprocess
import tempfile

import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1804_10574_amd")
STEM, IDENT, DOWN = 0, 1, 2

SOURCE = r"""
#include <hip/hip_runtime.h>
#include "ddg_kernels.h"
#include <cstdio>
#include <cstdlib>
using namespace ddg;
int main(int n, char** v) {      // images, height = width, bf16, then kind, input channels and stride of every block
  std::vector<EvalBlockShape> b;
  for (int i = 4; i + 2 < n; i += 3) b.push_back({atoi(v[i]), atoi(v[i + 1]), atoi(v[i + 2])});
  EvalPlan p;
  if (!eval_plan(b.data(), (int)b.size(), atoi(v[1]), atoi(v[2]), atoi(v[2]), atoi(v[3]) ? BF16 : F32, &p)) return 1;
  for (const EvalLaunch& l : p.launches) printf("%d %d %d %zu\n", l.count, l.strips, l.gap, l.lds);
  return 0;
}
"""


@functools.lru_cache(maxsize=None)
def _program():
    from paper_1804_10574_amd.build import FLAGS, HIPCC
    if not shutil.which(HIPCC) or not os.path.exists(os.path.join(PKG, "libddg.so")):
        pytest.skip("needs hipcc and the built library")
    d = tempfile.TemporaryDirectory(prefix="eval_plan")
    src, exe = os.path.join(d.name, "main.cpp"), os.path.join(d.name, "plan")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([HIPCC] + FLAGS + ["-I", os.path.join(PKG, "csrc"), src, f"-L{PKG}", "-l:libddg.so", f"-Wl,-rpath,{PKG}", "-o", exe],
                   check=True, capture_output=True)
    return d, exe


def launches(blocks, n, hw, bf16=True):
    """[(blocks, strips, bytes between pixels, LDS bytes)]; None: the per-layer kernels. blocks: (kind, input channels, stride)."""
    r = subprocess.run([_program()[1], str(n), str(hw), str(int(bf16))] + [str(v) for b in blocks for v in b],
                       capture_output=True, text=True, timeout=60)
    return [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()] if r.returncode == 0 else None


def shapes(blocks):
    """Blocks of a module description (kind, cin, cmid, cout, stride, projection) as launches() takes them; no head."""
    import workloads as wk
    return [(STEM if b[0] == wk.BLOCK_STEM else DOWN if b[4] == 2 else IDENT, b[1], b[4]) for b in blocks if b[0] != wk.BLOCK_HEAD]
