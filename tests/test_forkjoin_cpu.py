"""Two streams of one call (csrc/ff_forkjoin.hpp): whichever step fails, the
second stream is joined back once it was forked, and the first error returns."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "ff_forkjoin.hpp"
enum Status { OK = 0, FORK = 1, FIRST = 2, SECOND = 3, JOIN = 4 };
int main(int argc, char** argv) {
  auto step = [&](const char* name, Status s) {
    std::printf("%s ", name);
    for (int i = 1; i < argc; ++i)
      if (std::strcmp(argv[i], name) == 0) return s;
    return OK;
  };
  const Status rc = ff::fork_join([&] { return step("fork", FORK); }, [&] { return step("first", FIRST); },
                                  [&] { return step("second", SECOND); }, [&] { return step("join", JOIN); });
  std::printf("%d\n", (int)rc);
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("forkjoin")
    src, exe = d / "t.cpp", d / "t"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-I", os.path.join(ROOT, "paper_2609_14706_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("failing,want", [
    ([], "fork first second join 0"), (["fork"], "fork 1"), (["first"], "fork first join 2"),
    (["second"], "fork first second join 3"), (["join"], "fork first second join 4"),
    (["second", "join"], "fork first second join 3")])
def test_the_join_always_follows_the_fork(program, failing, want):
    out = subprocess.run([program, *failing], check=True, capture_output=True, text=True).stdout
    assert out.split() == want.split()


def test_the_engine_orders_its_streams_through_it():
    """No other place in the engine makes one stream wait for another."""
    text = open(os.path.join(ROOT, "paper_2609_14706_amd", "csrc", "ff_engine.hip")).read()
    assert text.count("hipStreamWaitEvent") == 1 and text.count("fork_join(") == 2
