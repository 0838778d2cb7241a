"""What has to be done once per device (csrc/per_device.h), compiled with the host compiler."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_09547_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "per_device.h"
int main() {
  qgtc::OncePerDevice once;
  int calls = 0;
  bool works = true;
  auto set = [&] { ++calls; return works; };
  auto expect = [&](int dev, bool ok, int n) {
    const bool r = once(dev, set);
    if (r != ok || calls != n) { std::printf("device %d: %d, %d calls\n", dev, r, calls); return false; }
    return true;
  };
  bool good = expect(0, true, 1) && expect(0, true, 1);      // once
  good = good && expect(1, true, 2) && expect(1, true, 2);   // on every device
  works = false;
  good = good && expect(2, false, 3) && expect(2, false, 4); // a failure is reported and not kept
  works = true;
  good = good && expect(2, true, 5) && expect(2, true, 5) && expect(63, true, 6) && expect(0, true, 6);
  good = good && expect(64, true, 7) && expect(64, true, 8) && expect(-1, false, 8);
  return good ? 0 : 1;
}
"""


def test_once_on_every_device(tmp_path):
    src = tmp_path / "once.cpp"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(tmp_path / "once")], check=True)
    r = subprocess.run([str(tmp_path / "once")], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout


def test_kernels_ask_per_device():
    """Every kernel that takes more LDS than a launch gets unasked goes through it."""
    for name in os.listdir(CSRC):
        text = open(os.path.join(CSRC, name)).read() if name.endswith((".h", ".hip")) else ""
        assert "hipFuncSetAttribute" not in text or name == "qgtc_internal.h", name
