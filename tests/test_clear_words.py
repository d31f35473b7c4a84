"""The words that the attention kernels clear on the way, computed on the host for the places of threads in small and in
the largest grids (csrc/hb_internal.h, compiled for the host alone): nothing outside them is written."""
import os
import subprocess

from paper_2509_18824_amd import build as B

SOURCE = r"""
#include <stdio.h>
#include "hb_internal.h"
int main() {
  using hb::clear_words;
  unsigned long long guarded[3000];
  // no words at no address, the plain call of every grid: the last places of 2^23 to 2^24 - 1 workgroups of 256 threads
  for (uint32_t groups : {1u, 1000u, 1u << 23, (1u << 23) + 5u, (1u << 24) - 1u})
    for (uint32_t group : {0u, groups / 2, groups - 1u})
      for (uint32_t thread : {0u, 255u}) {
        clear_words({nullptr, 0}, group, groups, thread, 256);
        for (auto &w : guarded) w = 7;
        clear_words({guarded + 1000, 1000}, group, groups, thread, 256);
        const unsigned long long first = (unsigned long long)group * 256 + thread, step = (unsigned long long)groups * 256;
        for (unsigned long long i = 0; i < 3000; ++i) {
          const bool mine = i >= 1000 && i < 2000 && i - 1000 >= first && (i - 1000 - first) % step == 0;
          if (guarded[i] != (mine ? 0ull : 7ull)) return printf("word %lld of group %u of %u\n", (long long)i - 1000, group, groups), 1;
        }
      }
  // all threads together clear every word
  for (auto &w : guarded) w = 7;
  for (uint32_t group = 0; group < 3; ++group)
    for (uint32_t thread = 0; thread < 256; ++thread) clear_words({guarded, 3000}, group, 3, thread, 256);
  for (auto w : guarded)
    if (w) return puts("a word is left"), 1;
  return puts("cleared"), 0;
}
"""


def test_no_word_outside_is_cleared_whatever_the_grid(tmp_path):
    src, exe = tmp_path / "clear_words.hip", tmp_path / "clear_words"
    src.write_text(SOURCE)
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-O3", "-fno-gpu-rdc") and not f.startswith("--offload")]
    flags = [f for i, f in enumerate(flags) if f not in ("-Xclang", "-target-feature", "-packed-fp32-ops")]
    subprocess.run([B.HIPCC, *flags, "-O1", "--cuda-host-only", str(src), "-o", str(exe)], check=True, capture_output=True, timeout=300)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout == "cleared\n", run.stdout
