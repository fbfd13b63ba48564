"""Slices on host threads: every slice runs, and a failure to start a thread
(no memory for its state) is reported with the started ones ended, not
thrown."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>
#include "host_slices.h"
static std::atomic<int> left{-1};  // allocations until one fails; < 0: none does
void* operator new(std::size_t n) {
  if (left.load() >= 0 && left.fetch_sub(1) == 0) throw std::bad_alloc();
  void* p = std::malloc(n);
  if (!p) std::abort();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
int main(int, char** argv) {
  if (argv[1][0] == 'n') return std::printf("%d\n", finger::copy_slices(std::strtoull(argv[2], nullptr, 10))), 0;
  std::atomic<int> ran{0}, sum{0};
  left = std::atoi(argv[1]);
  const bool all = finger::run_sliced(std::atoi(argv[2]), [&](int i) { ++ran; sum += i; });
  left = -1;
  std::printf("%d %d %d\n", (int)all, ran.load(), sum.load());
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("slices")
    (d / "slices.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_2206_11408_amd", "csrc"),
                    str(d / "slices.cpp"), "-o", str(d / "slices")], check=True)
    return lambda *a: subprocess.run([str(d / "slices"), *map(str, a)], capture_output=True, text=True)


def test_every_slice_runs(program):
    for n in (0, 1, 4, 8):
        assert program(-1, n).stdout.split() == ["1", str(n), str(n * (n - 1) // 2)]


@pytest.mark.parametrize("fail_at", [0, 1, 2, 3])
def test_no_memory_for_a_thread(program, fail_at):
    r = program(fail_at, 4)
    assert r.returncode == 0, r.stderr
    all_ran, ran, _ = map(int, r.stdout.split())
    assert all_ran == 0 and ran < 4


def test_slices_only_where_they_pay(program):
    mb = 1 << 20
    got = [int(program("n", b).stdout) for b in (0, 10 * mb, 41 * mb, 64 * mb - 1, 64 * mb, 1 << 33)]
    assert got == [1, 1, 1, 1, 4, 4]
