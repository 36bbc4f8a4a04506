"""The workspaces that the library keeps (csrc/workspace_cache.h, host code without GPU calls), with an allocator that refuses blocks above a limit."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_22137_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "workspace_cache.h"
int main() {
  prism::WorkspaceCache cache;
  static char memory[64];
  int asked = 0;
  size_t limit = 100;
  auto alloc = [&](size_t n) -> void* { ++asked; return n <= limit ? memory + asked : nullptr; };
  int one, two;
  // a call that would like 150 and can do with 80
  auto call = [&](const void* owner, size_t wish, size_t least) -> size_t {
    if (cache.get(0, owner, wish, true, alloc)) return wish;
    return cache.get(0, owner, least, false, alloc) ? least : 0;
  };
  auto show = [&](size_t got) { std::printf("%zu %d\n", got, asked); };
  show(call(&one, 150, 80));      // 80: asked for 150 and 80
  show(call(&one, 150, 80));      // again: nothing is asked for
  show(call(&one, 200, 80));      // more than what was refused: nor here
  show(call(&one, 95, 80));       // less: there is such a block
  show(call(&two, 150, 120));     // neither: 0, both asked for
  show(call(&two, 150, 120));     // what the call needs at least is always asked for
  limit = 300;
  show(call(&two, 150, 120));     // 120: memory has come free, the wish stays refused
  show(call(&one, 90, 90));       // there
  cache.blocks.clear();           // released
  show(call(&one, 150, 80));      // 150
  std::printf("%zu\n", cache.blocks.size());
}
"""


def test_a_refused_size_is_not_asked_for_again(tmp_path):
    src, exe = tmp_path / "cache.cpp", tmp_path / "cache"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I" + CSRC, str(src), "-o", str(exe)])
    got = [tuple(int(v) for v in line.split()) for line in subprocess.check_output([str(exe)], text=True).splitlines()]
    assert got == [(80, 2), (80, 2), (80, 2), (95, 3), (0, 5), (0, 6), (120, 7), (90, 7), (150, 8), (1,)]
