"""The push pass's packed heights keep every height that a frame of 2^28 pixels can have, in order and
apart from "no way to the sink", whatever the direction bits (checked by the compiler)."""
import os
import subprocess

from paper_1008_0502_amd import build

PROBE = """
#include "sp_internal.h"
constexpr bool in_order(int32_t a, int32_t b) { return (cut_pack(a) | 7u) < cut_pack(b); }
constexpr bool kept(int32_t h) {
  return cut_unpack(cut_pack(h)) == h && cut_unpack(cut_pack(h) | 7u) == h && (cut_pack(h) | 7u) < SP_CUT_HINF;
}
static_assert(kept(0) && kept(1) && kept((1 << 26) - 1) && kept(1 << 26) && kept(1 << 27) && kept(1 << 28), "kept");
static_assert(in_order(0, 1) && in_order((1 << 26) - 1, 1 << 26) && in_order((1 << 27) - 1, 1 << 27) &&
              in_order((1 << 28) - 1, 1 << 28) && in_order(1 << 28, SP_CUT_INF), "in order");
static_assert(cut_unpack(cut_pack(SP_CUT_INF)) == SP_CUT_INF, "no way to the sink");
"""


def test_every_height_is_kept(tmp_path):
    src = tmp_path / "heights.hip"
    src.write_text(PROBE)
    r = subprocess.run([build._hipcc(), *build.HIP_FLAGS, "-I", build.INCLUDE, "-I", build.CSRC, "-x", "hip",
                        "-fsyntax-only", str(src)], capture_output=True, text=True, env=os.environ)
    assert r.returncode == 0, r.stderr
