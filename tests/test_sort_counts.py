"""Where the coherence sort's first pass keeps its counters, on the host, for every batch size that takes
the pass: at a 16-byte boundary, past the keys, and before the arrays that the pass writes."""
import os
import shutil
import subprocess

import pytest

from paper_2504_21627_amd import build as B

COUNTS = r"""
#include <cstdio>
#include "lsnif_launch.hpp"
using namespace lsnif;
int main()
{
    for (uint32_t n = 2u * kRadixTile; n <= kGroupMax; ++n) {
        const size_t at = group_counts_at(n), words = (size_t)((n + kRadixTile - 1u) / kRadixTile) * kGroupDigits;
        if (at % 4u || at < n || at + words > 2u * (size_t)n) return std::printf("n %u: at %zu\n", n, at), 1;
    }
    std::printf("ok\n");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="hipcc not available")
def test_first_counters_are_aligned_and_apart(tmp_path):
    src, exe = tmp_path / "counts.hip", tmp_path / "counts"
    src.write_text(COUNTS)
    csrc = os.path.join(os.path.dirname(B.__file__), "csrc")
    subprocess.run([B.HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)], check=True,
                   capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
