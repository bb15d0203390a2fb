"""Kernel settings that belong to a device are made on every device, and again where they failed (host, no GPU)."""
import subprocess
from pathlib import Path

CSRC = Path(__file__).resolve().parent.parent / "paper_2604_22808_amd" / "csrc"

PROGRAM = r"""
#include "per_device.h"
#include <cstdio>
#include <initializer_list>
int main() {
  fa::OncePerDevice once;
  int calls[70] = {0}, fail = 1;
  auto run = [&](int dev) { return once.run(dev, [&] { ++calls[dev]; return dev == 3 && fail-- > 0 ? 7 : 0; }); };
  const int first = run(3);   // fails, and is tried again
  for (int rep = 0; rep < 3; ++rep)
    for (int dev : {0, 3, 63, 65}) if (run(dev) != 0) return 1;
  std::printf("%d %d %d %d %d %d", first, calls[0], calls[1], calls[3], calls[63], calls[65]);
}
"""


def test_once_per_device(tmp_path):
    (tmp_path / "t.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", f"-I{CSRC}", str(tmp_path / "t.cpp"), "-o", str(tmp_path / "t")])
    assert subprocess.check_output([str(tmp_path / "t")], text=True) == "7 1 0 2 1 3"


def test_no_kernel_setting_is_made_once_per_process():
    """Every place that raises a kernel's limit goes through the helper."""
    users = [p.name for p in CSRC.iterdir() if "hipFuncSetAttribute" in p.read_text()]
    assert users == ["ctx.h"], users
