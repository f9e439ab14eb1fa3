"""Which calls take the digit sort at once after a bucket outgrew its block: those of the same sizes, no others."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_07331_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include "host.hpp"
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\\n", __LINE__, #x); return 1; } } while (0)
int main() {
  hlc::OverflowNotes n;
  CHECK(!n.take(1000, 2000));
  n.add(1000, 2000);
  CHECK(!n.take(2000, 1000) && !n.take(1000, -1));       // other sizes keep the buckets
  int k = 0;
  while (n.take(1000, 2000)) ++k;
  CHECK(k == hlc::OverflowNotes::FIRST);
  CHECK(!n.take(1000, 2000));                             // tried again once
  long tried = 0, calls = 0;
  for (; calls < 100000; ++calls)
    if (!n.take(1000, 2000)) { ++tried; n.add(1000, 2000); }
  CHECK(tried < 110);                                     // always crowded: rarely tried
  for (int j = 0; j < hlc::OverflowNotes::KEPT; ++j) n.add(j, -1);
  CHECK(!n.take(1000, 2000));                             // the oldest note makes room
  for (int j = 0; j < hlc::OverflowNotes::KEPT; ++j) CHECK(n.take(j, -1));
  return 0;
}
"""


def test_overflow_notes(tmp_path):
    from paper_2301_07331_amd import build_lib
    src, exe = tmp_path / "notes.hip", tmp_path / "notes"
    src.write_text(PROGRAM)
    subprocess.run([build_lib.HIPCC, *build_lib.FLAGS, "--cuda-host-only", "-I", CSRC, "-c", str(src), "-o",
                    str(exe) + ".o"], check=True)
    subprocess.run([build_lib.HIPCC, str(exe) + ".o", "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
