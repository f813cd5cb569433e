"""The rules on sizes that choose between kernels (csrc/dispatch_rules.h), compiled for the host, at sizes where one side was measured to be faster."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROBE = r'''
#include "dispatch_rules.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
int main(int argc, char** argv) {
  long long v[8] = {};
  for (int i = 2; i < argc; ++i) v[i - 2] = atoll(argv[i]);
  bool r = false;
  if (!strcmp(argv[1], "few")) r = moqe::few_rows_kernel(v[0], v[1], v[2], int(v[3]), v[4] != 0, v[5] != 0);
  else if (!strcmp(argv[1], "nlp")) r = moqe::nlp_whole_rows(v[0], v[1], v[2], v[3]);
  else return 1;
  printf("%d\n", int(r));
  return 0;
}
'''


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "probe.cpp", d / "probe"
    src.write_text(PROBE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2508_09204_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    return lambda *a: subprocess.run([str(exe)] + [str(int(x)) if not isinstance(x, str) else x for x in a], check=True,
                                     capture_output=True, text=True).stdout.strip() == "1"


# n, k, rows, experts that can have rows, gate/up, experts of unequal weight bytes
@pytest.mark.parametrize("args,few", [
    ((4096, 11008, 1, 1, False, False), True), ((4096, 11008, 16, 1, False, False), True), ((4096, 4096, 16, 1, False, True), True),
    ((8192, 4096, 8, 1, False, False), True), ((8192, 4096, 16, 1, False, False), False), ((8192, 2048, 16, 1, False, False), True),
    ((16384, 512, 2, 1, False, False), True), ((16384, 512, 16, 1, False, False), False), ((16384, 4096, 16, 1, False, False), False),
    ((32768, 4096, 1, 1, False, False), False), ((4096, 4096, 16, 4, False, False), False), ((8192, 4096, 16, 8, False, True), False),
    ((4096, 512, 16, 8, False, True), True), ((4096, 11008, 8, 4, False, True), True), ((4096, 11008, 8, 4, False, False), False),
    ((11008, 4096, 1, 1, True, False), True), ((11008, 4096, 16, 1, True, False), False), ((11008, 4096, 16, 4, True, True), True),
    ((16384, 4096, 16, 4, True, False), False), ((18944, 3584, 16, 8, True, True), True), ((32768, 512, 16, 1, True, False), True),
    ((256, 256, 16, 3, True, True), True), ((16, 128, 1, 1, False, False), True),
    ((11008, 4096, 16, 16, True, False), False), ((8192, 8192, 16, 16, True, False), True), ((4096, 11008, 16, 16, False, True), True),
    ((2048, 2048, 16, 16, False, False), True), ((8192, 2048, 16, 16, False, False), False), ((4096, 4096, 4, 4, False, False), True),
    ((16, 128, 17, 1, False, False), False), ((16, 128, 17, 1, True, False), False),      # what the kernel can hold
])
def test_launches_of_few_rows(rule, args, few):
    assert rule("few", *args) is few


# token rows, d, width, feed-forward
@pytest.mark.parametrize("args,whole", [
    ((32768, 3584, 384, 1536), True), ((513, 64, 128, 128), True), ((512, 64, 128, 128), False), ((513, 3584, 512, 2048), False), ((600, 64, 256, 640), False),
    ((528, 1024, 384, 12288), False), ((2048, 1024, 384, 12288), False), ((4112, 1024, 384, 12288), True), ((528, 1024, 384, 24576), False),
    ((528, 1024, 384, 6144), True), ((528, 1024, 256, 32768), False), ((528, 1024, 256, 8192), True), ((528, 1024, 128, 16384), True),
    ((32768, 24576, 384, 1536), True), ((8192, 32768, 384, 1536), False), ((4096, 65536, 384, 1536), False), ((1024, 65536, 384, 1536), True),
    ((1024, 131072, 384, 1536), False), ((12288, 65536, 256, 1024), False), ((4096, 65536, 256, 1024), True), ((16384, 65536, 128, 512), True),
    ((1 << 20, 1 << 22, 256, 256), False),      # operand copies past 32-bit offsets
])
def test_whole_rows_of_the_nlp_router(rule, args, whole):
    assert rule("nlp", *args) is whole
