"""Where the prefill finds a key tile in the K8 (V8) blocks of a sequence, at
lengths past 2^24 tokens, whose blocks take more than 2^31 bytes: the kernel's
own function, evaluated by the compiler (a pass over such a sequence takes
minutes on the GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

DRIVER = """
#include "turbo_common.h"
#include "attn_prefill.hip"
using turbo::tile_span;
// the tiles of nb blocks of 8192 bytes, in turn, with kH blocks to a tile
constexpr bool covers(int nb, int kH, int from) {
  const int tiles = (nb + kH - 1) / kH;
  for (int j = from; j < tiles; ++j) {
    const int blocks = nb - j * kH < kH ? nb - j * kH : kH;
    if (tile_span(nb, kH, j).offset != 8192L * kH * j) return false;
    if (tile_span(nb, kH, j).bytes != 8192 * blocks) return false;
  }
  return true;
}
%s
"""


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
def test_key_tiles_past_2_31_bytes(tmp_path):
    checks = []
    for kH in (1, 2):
        for nb in (1, 2, 3, 65, (1 << 18) - 1, (1 << 18) + 1, (1 << 19) + 1, (1 << 20) - 1):
            first = max(0, (nb + kH - 1) // kH - 64)  # the last 64 tiles
            checks.append(f"static_assert(covers({nb}, {kH}, {first}), \"nb={nb} kH={kH}\");")
    src = tmp_path / "tiles.hip"
    src.write_text(DRIVER % "\n".join(checks))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-fsyntax-only",
                        "-std=c++17", "-Wno-everything", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(ROOT, "paper_2412_08585_amd", "csrc"), str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
