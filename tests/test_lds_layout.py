"""The LDS of a STREAM tile with several vectors, computed on the host by the
function the kernels use: every part on its alignment, none over the next, and
no tile's parts past what is launched for the largest."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = r"""
#include <cstdio>
#include "tiles.h"
using namespace ffx;
template <class AR, int S>
static int check() {
  const uint32_t nrs[] = {1, 2, 3, 5, 63, 64, 65, 127, 255, 256}, nes[] = {0, 1, 3, 4, 5, 255, 256, 257, 2047, 2048, 4095, 4096};
  for (uint32_t nr : nrs)
    for (uint32_t ne : nes) {
      const StreamLds l = stream_b_lds<AR, S>(nr, ne);
      const bool ok = l.rps % 4 == 0 && l.words % 16 == 0 && l.values % 16 == 0 && l.rps >= nr * S * sizeof(typename AR::Acc) &&
                      l.words >= l.rps + (nr + 1) * 4 && l.values >= l.words + ne * 4 && l.bytes >= l.values + ne * 4 &&
                      l.words - l.rps < (nr + 1) * 4 + 16 && l.bytes <= tiles_lds_bytes<AR>(256, 4096, S);
      if (!ok) {
        printf("accumulator of %zu bytes, S = %d, %u rows, %u entries: %u %u %u %u\n", sizeof(typename AR::Acc), S, nr, ne, l.rps,
               l.words, l.values, l.bytes);
        return 1;
      }
    }
  return 0;
}
template <class AR>
static int widths() { return check<AR, 2>() || check<AR, 4>() || check<AR, 8>() || check<AR, 16>(); }
int main() {
  return widths<ArSmall>() || widths<ArM31>() || widths<ArGF2>() || widths<ArF32<true>>() || widths<ArF64<uint32_t, false>>();
}
"""


LIMITS = r"""
#include <cstdio>
#include "launch.h"
using namespace ffx;
int main() {
  LdsLimits l;
  int calls = 0, a, b;
  auto raise = [&](int dev, const void* k, int bytes, hipError_t result) {
    return l.raise(dev, k, bytes, [&] { ++calls; return result; });
  };
  bool ok = raise(0, &a, 70000, hipSuccess) == hipSuccess && calls == 1;
  ok = ok && raise(0, &a, 70000, hipSuccess) == hipSuccess && raise(0, &a, 66000, hipSuccess) == hipSuccess && calls == 1;
  ok = ok && raise(0, &a, 150000, hipSuccess) == hipSuccess && calls == 2;  // more than was granted
  ok = ok && raise(1, &a, 70000, hipSuccess) == hipSuccess && calls == 3;   // another device
  ok = ok && raise(0, &b, 70000, hipErrorInvalidValue) != hipSuccess && calls == 4;
  ok = ok && raise(0, &b, 70000, hipSuccess) == hipSuccess && calls == 5;   // a refused call granted nothing
  printf("%d calls\n", calls);
  return ok ? 0 : 1;
}
"""


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no hipcc")
@pytest.mark.parametrize("name,source", [("layout", SOURCE), ("limits", LIMITS)])
def test_on_the_host(tmp_path, name, source):
    """`limits`: a kernel's limit is raised again when a launch needs more than was granted."""
    src, exe = tmp_path / (name + ".hip"), tmp_path / name
    src.write_text(source)
    csrc = os.path.join(ROOT, "paper_1004_3719_amd", "csrc")
    # the host's half only: no device code is built, and nothing of it is called
    r = subprocess.run([HIPCC, "--cuda-host-only", "-O0", "-fPIC", "-std=c++17", "-I" + csrc, "-I" + os.path.join(ROOT, "include"),
                        "-c", str(src), "-o", str(exe) + ".o"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run(["g++", str(exe) + ".o", "-o", str(exe), "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
