"""The first entry of the zone's tile list that a block of an extrapolation
launch reads lies in the list, whatever the grid and the number of blocks (256
for one context; a batch launches as many per member as its largest member
has tiles), and is the block's own where the list has one for it.  The
library's own function, in host code."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = r"""
#include "paper_2402_12696_amd/csrc/lbrmt_internal.h"
#include <cstdio>
using namespace lbrmt;
int main()
{
    for (int nx = 8; nx <= 700; nx += nx < 130 ? 1 : 37)
        for (int ny = 8; ny <= 700; ny += ny < 130 ? 1 : 41) {
            const long long room = fused_tiles(nx, ny);
            for (int b = 0; b < FF_BLOCKS; b++) {
                const int at = ff_first(b, nx, ny);
                if (at < 0 || at >= room || (b < room && at != b)) {
                    printf("%d x %d, block %d: entry %d of %lld\n", nx, ny, b, at, room);
                    return 1;
                }
            }
        }
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_a_blocks_first_entry_lies_in_the_list(tmp_path):
    src, exe = tmp_path / "list.hip", tmp_path / "list"
    src.write_text(SOURCE)
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-I", ROOT, str(src), "-o",
                    str(exe)], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    out = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert out.returncode == 0, out.stdout
