"""What the loads of the fp32 kernel for 3x3 filters in KCRS order span (csrc/conv_f32_kcrs33.h), compiled for the host: of the blocks that exist every scalar
offset lies inside the tensor with what the lanes add to it, and beyond the last block, which the loads run ahead of, buffer and scalar offset are empty."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_04728_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "conv_f32_kcrs33.h"
int main()
{
    int N, C, H, W, K;
    while (scanf("%d %d %d %d %d", &N, &C, &H, &W, &K) == 5) {
        const int blocks = C / dr::KCRS33_CB, HW = H * W;
        const long w_bytes = 9l * K * C * 4, x_bytes = (long)N * C * HW * 4;
        int wrong = 0, read = 0;
        for (int blk = 0; blk < blocks + 2; ++blk) {           // filters: two blocks ahead; activations: one
            // a lane adds up to the last filter's row and its last 16 bytes of the block
            const dr::LoadRange f = dr::kcrs33_filters(blk, blocks, (int)w_bytes);
            const long lane = ((long)(K - 1) * C * 9 + dr::KCRS33_ROW - 4) * 4;
            wrong += f.scalar < 0 || f.scalar > f.bytes || (blk < blocks ? f.scalar != blk * 72 * 4 || f.scalar + lane + 16 > f.bytes : f.bytes != 0);
            for (int j = 0; blk < blocks + 1 && j < 4; ++j)
                for (int group = 0; group < 2; ++group) {      // two groups of four channels
                    const dr::LoadRange p = dr::kcrs33_plane(blk, blocks, j, HW, (int)x_bytes);
                    const long at = (((long)(N - 1) * C + group * 4) * HW + HW - 1) * 4;
                    wrong += p.scalar < 0 || p.scalar > p.bytes || (blk < blocks ? p.scalar + at + 4 > p.bytes : p.bytes != 0);
                    read += p.bytes != 0;
                }
        }
        printf("%d %d\n", wrong, read == blocks * 8);
    }
}
"""


def test_every_load_lies_inside_its_buffer(tmp_path):
    (tmp_path / "loads.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(tmp_path / "loads.cpp"), "-o", str(tmp_path / "loads")])
    cases = [(1, 16, 1, 1, 1), (1, 16, 3, 3, 64), (2, 32, 13, 9, 64), (32, 64, 56, 56, 192), (1, 512, 30, 28, 32), (3, 48, 1000, 2000, 5),
             (1, 16, 5000, 6710, 8), (7, 4096, 4, 4, 14560)]      # ... inputs and filters just below 2 GiB
    out = subprocess.run([str(tmp_path / "loads")], input="\n".join("%d %d %d %d %d" % c for c in cases), capture_output=True, text=True, check=True).stdout
    assert out.split("\n")[:-1] == ["0 1"] * len(cases)
