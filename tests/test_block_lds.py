"""The workgroup solver's LDS request covers everything that its panel steps read (checked by the
compiler, no GPU needed): they take 16 consecutive entries of a row from a panel's first column on,
also in a last panel of fewer columns, so the last row's reach past the matrix array."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = """
#include "block_tron.hpp"
using S = mt::BlockTron<2, 8, false>;
constexpr bool covered(int n)
{
    const int ld = (n + 1) | 1, panel = (n - 1) / 16 * 16;
    return sizeof(double) * (size_t)(S::oU + (n - 1) * ld + panel + 16) <= S::lds_bytes(n);
}
constexpr bool all(int n) { return n > 128 || (covered(n) && all(n + 1)); }
static_assert(all(1), "a panel's reads end inside the workgroup's LDS");
static_assert(S::lds_bytes(128) <= 160 * 1024, "the largest request fits a CU");
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_panel_reads_stay_inside_the_request(tmp_path):
    src = tmp_path / "reach.hip"
    src.write_text(SOURCE)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "--cuda-host-only", "-fsyntax-only",
                        "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2106_14995_amd", "csrc"),
                        str(src)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
