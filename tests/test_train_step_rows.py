"""Which weight rows the training step's kernel reads, on the host: for every object it accepts, the
first layer's product stays inside the packed weights, whatever the tile's longest list."""
import os
import shutil
import subprocess

import pytest

from paper_2504_21627_amd import build as B

ROWS = r"""
#include <cstdio>
#include "lsnif_train.hpp"
using namespace lsnif;
int main()
{
    unsigned long long shapes = 0, tails = 0;
    for (uint32_t width : {64u, 128u})
        for (uint32_t nh = 1; nh <= 6; ++nh)
            for (uint32_t H = 2; H <= 64; H += 2)
                for (uint32_t L = 1; L <= 32; ++L)
                    for (uint32_t F : {2u, 3u}) {
                        const uint32_t in0 = H * L * F;
                        if (!step_takes(in0, H, nh, width, 1u << 24)) continue;
                        ++shapes;
                        // rows of `width` floats in the packed weights: layer 0, the others, the head of 16 columns
                        const uint32_t held = in0 + (nh - 1u) * width + kMaxOut;
                        if (held < 16u) return std::printf("first rows: %u %u %u %u %u\n", width, nh, H, L, F), 1;
                        for (uint32_t most = 1; most <= H / 2u; ++most) {
                            const uint32_t K1 = 2u * most * L * F, K = K1 / 16u * 16u;
                            if (K < K1 && K + 16u > (K1 + 31u) / 32u * 32u) return std::printf("inputs not zeroed\n"), 1;
                            tails += K < K1;
                            for (uint32_t row = K; K < K1 && row < K + 16u; ++row)
                                if (step_weight_row(row, K1) >= in0 || (row < K1 && step_weight_row(row, K1) != row))
                                    return std::printf("row %u: %u %u %u %u %u\n", row, width, nh, H, L, F), 1;
                        }
                    }
    std::printf("ok %llu %llu\n", shapes, tails);
    return shapes > 200 && tails > 200 ? 0 : 1;
}
"""


@pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="hipcc not available")
def test_first_layer_rows_stay_in_the_weights(tmp_path):
    src, exe = tmp_path / "rows.hip", tmp_path / "rows"
    src.write_text(ROWS)
    csrc = os.path.join(os.path.dirname(B.__file__), "csrc")
    subprocess.run([B.HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)], check=True,
                   capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
