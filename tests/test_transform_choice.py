"""A transform pass that is chosen for a size takes it: the rules the host chooses by and the launchers' own checks (host, no GPU)."""
import subprocess
from pathlib import Path

from paper_2604_22808_amd import binding as B
from paper_2604_22808_amd.build import hipcc

ROOT = Path(__file__).resolve().parent.parent

PROGRAM = r"""
#include <cstdio>
#include "ctx.h"
using namespace fa;
int main() {   // lines "direction W d chosen refused"; launches of no slices: the launcher checks the sizes and starts nothing
  for (int W : {16, 64, 112, 128})
    for (int64_t d = 64; d <= 32768 * 64; d = d < 16384 + 640 ? d + 64 : d * 2) {
      WhPassArgs a{};
      a.T = 128; a.d = (int)d; a.rows = a.out_rows = a.ldh = 64; a.cols = a.out_cols = a.ldw = W;
      int slots[3];
      std::printf("f %d %d %d %d\n", W, a.d, (int)wh_fits(a.T, a.d, 64, W, 64, W), launch_wh_pass(&a, 1, 256, nullptr, slots) != hipSuccess);
      std::printf("i %d %d %d %d\n", W, a.d, (int)hw_fits(a), launch_hw_inverse(&a, 1, 256, nullptr) != hipSuccess);
    }
}
"""


def test_what_the_one_pass_transforms_are_chosen_for_they_take(tmp_path):
    (tmp_path / "t.cpp").write_text(PROGRAM)
    lib = Path(B.LIB_PATH).parent
    subprocess.check_call([hipcc(), "-std=c++17", "--offload-host-only", f"-I{ROOT / 'include'}", f"-I{lib / 'csrc'}", str(tmp_path / "t.cpp"),
                           "-o", str(tmp_path / "t"), f"-L{lib}", "-lfreqattn", f"-Wl,-rpath,{lib}"])
    lines = [line.split() for line in subprocess.check_output([str(tmp_path / "t")], text=True).splitlines()]
    took = {"f": {}, "i": {}}
    for way, w, d, chosen, refused in lines:
        assert not (chosen == "1" and refused == "1"), (way, w, d)
        took[way].setdefault(int(w), {})[int(d)] = chosen == "1"
    # eight rows of 128 x W x d 16-bit values in 32 bits, less the 128 bytes of a row's piece: what an axis at a time takes as well
    for w, t in took["f"].items():
        for d, chosen in t.items():
            assert chosen == (128 * w * d * 16 + 128 < 2 ** 32), (w, d)
    assert took["f"][128][8192] and took["f"][128][16320] and not took["f"][128][16384] and took["f"][112][9408]
