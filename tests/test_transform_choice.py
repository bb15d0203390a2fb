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


def _run(program, tmp_path):
    (tmp_path / "t.cpp").write_text(program)
    lib = Path(B.LIB_PATH).parent
    subprocess.check_call([hipcc(), "-std=c++17", "--offload-host-only", f"-I{ROOT / 'include'}", f"-I{lib / 'csrc'}", str(tmp_path / "t.cpp"),
                           "-o", str(tmp_path / "t"), f"-L{lib}", "-lfreqattn", f"-Wl,-rpath,{lib}"])
    return [line.split() for line in subprocess.check_output([str(tmp_path / "t")], text=True).splitlines()]


# rows (kt, h) in LDS that the H axis of the generic T + H pass reads for `KT` rows kt: lane group g takes rows g R .. g R + R - 1 of each kt
PAIR_PROGRAM = r"""
#include <cstdio>
#include "ctx.h"
using namespace fa;
int main() {
  for (int T = 1; T <= 16; ++T)
    for (int H = 1; H <= 64; ++H)
      for (int KT = 0; KT <= T; ++KT) {
        const int R = (H + 3) / 4, ldh = (H + 15) / 16 * 16, made = th_rows(T, H, KT);
        bool ok = made >= KT && made <= T;
        for (int kt = 0; kt < KT; ++kt)
          for (int j = 0; j < 4 * R; ++j) {
            const int row = kt * H + j;
            ok = ok && (row < T * H ? row / H < made : (row + 1 - T * H) * 64 <= ldh * (ldh + 4));   // (made, or of the matrix behind)
          }
        if (!ok) std::printf("%d %d %d\n", T, H, KT);
      }
}
"""


def test_rows_that_the_generic_pair_of_axes_reads_are_made(tmp_path):
    assert _run(PAIR_PROGRAM, tmp_path) == []


# T passes of a few slices, of the boxes that low (a quarter) and mid (half) bands keep beside the whole grid: forward (k) and inverse (i)
SHARE_PROGRAM = r"""
#include <cstdio>
#include "ctx.h"
using namespace fa;
int main() {
  for (int T = 16; T <= 128; T += 16) {
    DctPassArgs p[3][2];   // [low, mid, whole][forward, inverse]
    for (int k = 0; k < 3; ++k) {
      const int box = k == 2 ? T : T * (k + 1) / 4, side = k == 2 ? 16 : 4 * (k + 1);
      for (DctPassArgs& a : p[k]) { a = DctPassArgs{}; a.inner = side * 64; a.nslab = 6 * side; }
      p[k][0].n = T; p[k][0].n_out = box;
      p[k][1].n = (box + 15) / 16 * 16; p[k][1].n_out = T; p[k][1].perm_in = (const int32_t*)1; p[k][1].delta = k < 2;
    }
    for (int way = 0; way < 2; ++way)
      for (int lead = 1; lead < 3; ++lead)
        for (int k = 0; k < lead; ++k)
          if (!dct_passes_share(p[lead][way], p[k][way], 256)) std::printf("%d %d %d %d\n", T, way, lead, k);
    // a gather that selects reads its own rows only, and a launch has no tiles beyond its lead's
    DctPassArgs s = p[0][1];
    s.delta = 0;
    if (s.n < T && dct_passes_share(p[2][1], s, 256)) std::printf("%d selects\n", T);
    if (T > 32 && dct_passes_share(p[0][0], p[2][0], 256)) std::printf("%d keeps more\n", T);
  }
}
"""


def test_small_t_passes_share_a_launch_whatever_they_keep(tmp_path):
    assert _run(SHARE_PROGRAM, tmp_path) == []


def test_what_the_one_pass_transforms_are_chosen_for_they_take(tmp_path):
    lines = _run(PROGRAM, tmp_path)
    took = {"f": {}, "i": {}}
    for way, w, d, chosen, refused in lines:
        assert not (chosen == "1" and refused == "1"), (way, w, d)
        took[way].setdefault(int(w), {})[int(d)] = chosen == "1"
    # eight rows of 128 x W x d 16-bit values in 32 bits, less the 128 bytes of a row's piece: what an axis at a time takes as well
    for w, t in took["f"].items():
        for d, chosen in t.items():
            assert chosen == (128 * w * d * 16 + 128 < 2 ** 32), (w, d)
    assert took["f"][128][8192] and took["f"][128][16320] and not took["f"][128][16384] and took["f"][112][9408]
