"""The entry test of the pivoted QR's launches, on the CPU: within a launch it
has one answer before and after the stop that the launch itself stores, since
its wavefronts make it at any time; later launches leave at once."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "cpqr.hpp"
int main() {
  for (int kmax = 1; kmax <= 40; ++kmax)
    for (int at = 0; at < kmax; ++at) {  // the step that stops
      lsh::CpqrState st{kmax, 0, 0.0};
      for (int j = 0; j < kmax; ++j) {
        const bool early = st.over(j);
        if (j == at) st.stop(j);
        const bool late = st.over(j);
        if (early != late) return 1;
        if (early != (j > at)) return 2;
      }
      if (st.k != at || !st.done) return 3;
    }
  return 0;
}
"""


def test_one_answer_for_every_wavefront_of_a_launch(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2007_12718_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
