"""The append's ring slots on the host: over every accepted combination of past length, chunk, window, initial
tokens and ring of a small range (rings shorter than the window among them), each slot lies in the ring, and a
token that has scores is read from the slot that holds it; and the chunk's keys are read only where the call has to
give them."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "ring_slot.h"
using namespace infllm;
int main() {
  long cases = 0, shorter = 0;
  for (int ring = 2; ring <= 14; ++ring)
    for (int n_q = 1; n_q < ring; ++n_q)
      for (int n_local = 1; n_local <= 20; ++n_local)
        for (int n_init = 0; n_init <= 9; n_init += 3)
          for (int past = 0; past <= 40; ++past) {
            // as infllm_append checks its arguments
            const int t_lo = std::max(n_init, past - n_local), t_hi = past + n_q - n_local;
            if (t_hi > t_lo && t_lo + ring < past + n_q) continue;
            ++cases;
            shorter += ring <= n_local;
            const bool need_k = t_hi > t_lo && t_hi > past;  // the chunk's keys may be absent otherwise
            for (int i = 0; i < n_q; ++i) {
              const int sp = ring_slot(past % ring, i, ring), st = leaving_slot(past + i, n_local, n_init, sp, ring);
              const int t = past + i - n_local;
              if (sp != (past + i) % ring || st < 0 || st >= ring || (t >= n_init && st != t % ring)) {
                std::printf("ring %d n_q %d l_L %d l_I %d past %d i %d: %d %d\n", ring, n_q, n_local, n_init, past, i, sp, st);
                return 1;
              }
              const bool chunk = leaving_key_in_chunk(past, t, n_init);
              if ((chunk && !need_k) || (t >= n_init && chunk != (t >= past)) || t >= past + n_q) {
                std::printf("key: n_q %d l_L %d l_I %d past %d i %d\n", n_q, n_local, n_init, past, i);
                return 1;
              }
            }
          }
  std::printf("%ld %ld\n", cases, shorter);
  return cases > 10000 && shorter > 1000 ? 0 : 2;
}
"""


def test_ring_slots(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    (tmp_path / "slots.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "slots")
    subprocess.run([cxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2402_04617_amd", "csrc"), str(tmp_path / "slots.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
