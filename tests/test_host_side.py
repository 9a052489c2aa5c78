"""Host code of the library that no call reaches without a GPU, compiled on its own with the host
compiler: the split of a launch over the grid's dimensions, and what is kept of ended handles' device
memory (with a device of the test's own in place of HIP's); and what the compiler makes of kernels that
no result shows."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _compile(folder, source):
    """A C++ program that sees the library's headers and links nothing of HIP."""
    src, exe = folder / "prog.cpp", folder / "prog"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2604_18556_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    return str(exe)


def _lines(exe, *args):
    return subprocess.run([exe, *args], check=True, capture_output=True, text=True).stdout.splitlines()


SPLIT = r"""
#include "gsq_internal.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2) {
    const gsq::RowSplit s = gsq::split_rows(std::atoll(argv[i]), std::atoll(argv[i + 1]));
    std::printf("%d %u %u\n", s.rows_x, s.gx, s.gy);
  }
}
"""
EDGE = (1 << 24) - 1   # workgroups of 256 threads in one dimension: 2^32 - 256 threads


def test_rows_split_over_the_grid(tmp_path):
    """(rows, workgroups per row): every row has its place (y rows_x + x / cols covers 0 .. rows - 1,
    each once), and no dimension holds 2^32 threads; layers that fit one dimension keep one."""
    cases = [(1, 1), (7, 3), (EDGE, 1), (EDGE + 1, 1), (1 << 24, 2), (17_000_015, 1), (1 << 30, 1),
             (EDGE // 2, 2), (EDGE // 2 + 1, 2), (5, EDGE // 5), (6, EDGE // 5), (70_000, 256),
             (1, 65536), (255, 65536), (256, 65536), (2000, 65536)]
    lines = _lines(_compile(tmp_path, SPLIT), *(str(x) for c in cases for x in c))
    assert len(lines) == len(cases)
    for (rows, cols), line in zip(cases, lines):
        rows_x, gx, gy = map(int, line.split())
        assert gx == rows_x * cols and 0 < gx <= EDGE, (rows, cols, line)
        assert (gy - 1) * rows_x < rows <= gy * rows_x and 0 < gy <= 65535, (rows, cols, line)
        assert gy == 1 or (rows_x + 1) * cols > EDGE, (rows, cols, line)


# A device of 1600 bytes, of which a sixteenth (100) may be kept and an eighth (200) must be free.
POOL = r"""
#include "gsq_pool.h"
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
static std::map<void*, size_t> live;
static size_t total = 1600, others = 0;
static bool refuse = false;
static size_t in_use() {
  size_t n = others;
  for (auto& b : live) n += b.second;
  return n;
}
extern "C" hipError_t hipMalloc(void** p, size_t n) {
  if (refuse) return hipErrorStreamCaptureUnsupported;
  if (in_use() + n > total) return hipErrorOutOfMemory;
  live[*p = std::malloc(n)] = n;
  return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) {
  if (!live.erase(p)) std::puts("freed twice");
  return hipSuccess;   // the address is not used again: each stays told apart
}
extern "C" hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *t = total;
  *f = total - in_use();
  return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

// words: a<dev>:<bytes> take a block, n<dev>:<bytes> a new one, g give the oldest one held back,
// o<bytes> what others use, c<0|1> refuse allocations as in a stream capture, r<dev> release
int main(int argc, char** argv) {
  static gsq::DevicePool pool;
  struct Held { int dev; void* p; size_t n; };
  std::map<int, Held> held;
  int first = 0, next = 0;
  for (int i = 1; i < argc; ++i) {
    const char* w = argv[i] + 1;
    if (argv[i][0] == 'a' || argv[i][0] == 'n') {
      Held h{std::atoi(w), nullptr, 0};
      const size_t n = std::atoi(std::string(w).substr(std::string(w).find(':') + 1).c_str());
      const hipError_t e = argv[i][0] == 'a' ? pool.take(h.dev, n, &h.p, &h.n)
                                             : pool.take_new(h.dev, h.n = n, &h.p);
      if (e == hipSuccess) held[next++] = h; else std::printf("none ");
    } else if (argv[i][0] == 'g') {
      const Held h = held[first];
      held.erase(first++);
      pool.give(h.dev, h.p, h.n, gsq::DevicePool::limit());
    } else if (argv[i][0] == 'o') {
      others = std::atoi(w);
    } else if (argv[i][0] == 'c') {
      refuse = *w == '1';
    } else {
      pool.release(std::atoi(w));
    }
    size_t kept = in_use() - others;
    for (auto& h : held) kept -= h.second.n;
    std::printf("%zu ", kept);
  }
  std::puts("");
}
"""


@pytest.fixture(scope="module")
def pool(tmp_path_factory):
    return _compile(tmp_path_factory.mktemp("pool"), POOL)


@pytest.mark.parametrize("words,kept", [
    # kept, and taken again where at most a quarter is wasted
    ("a0:40 g a0:40 g a0:33 g a0:31", "0 40 0 40 0 40 40"),
    # never more than a sixteenth: the oldest goes, a block above it is not kept
    ("a0:40 a0:50 a0:30 g g g", "0 0 0 40 90 80"),
    ("a0:40 a0:101 g g", "0 0 40 40"),
    # an eighth must be free (the ended handle's own block not counted): else all of the device's goes
    ("a0:40 a0:20 g o1400 g", "0 0 40 40 0"),
    ("a0:40 a0:101 g o1400 g", "0 0 40 40 0"),
    ("a0:40 a0:20 g o1341 g", "0 0 40 40 0"),
    ("a0:40 a0:20 g o1340 g", "0 0 40 40 60"),
    # another device's blocks are not this one's
    ("a1:40 a0:30 a0:20 g g o1400 g", "0 0 0 40 70 70 40"),
    # an allocation that does not fit takes what is kept on its device, once
    ("a0:40 g o1500 a0:90 a0:90", "0 40 40 0 none 0"),
    ("a0:40 a1:30 g g r0 r-1", "0 0 40 70 30 0"),
    # nor does a new one, and one that is refused for another reason leaves it
    ("a0:40 g n0:20 n0:20 g", "0 40 40 40 60"),
    ("a0:40 g o1599 n0:1 o1560 n0:4", "0 40 40 0 0 0"),
    ("a0:40 g c1 n0:4 a0:90 a0:40 c0 n0:4", "0 40 40 none 40 none 40 0 0 0"),
])
def test_kept_memory_policy(pool, words, kept):
    """Bytes kept after each word of the program above."""
    line, = _lines(pool, *words.split())
    assert line.split() == kept.split()


def test_every_allocation_is_one_that_kept_memory_makes_room_for():
    csrc = os.path.join(ROOT, "paper_2604_18556_amd", "csrc")
    assert [n for n in sorted(os.listdir(csrc)) if "hipMalloc(" in open(os.path.join(csrc, n)).read()] \
        == ["gsq_pool.h"]


def test_fp64_kernels_keep_their_values_in_registers(tmp_path):
    """The LDS and scratch of the fp64 kernels as compiled for gfx950: the local shift's window table
    (512 bytes) and eight wavefront sums (64) at most, so that no array of a thread's own has been put
    into either."""
    from paper_2604_18556_amd import build
    try:
        cc = build.hipcc()
    except RuntimeError as e:
        pytest.skip(str(e))
    r = subprocess.run([cc, *build.FLAGS, "--offload-device-only", "-Rpass-analysis=kernel-resource-usage",
                        "-c", os.path.join(build.CSRC, "gsq_elem64.hip"), "-o", str(tmp_path / "x.o")],
                       check=True, capture_output=True, text=True)
    used = {}
    for line in r.stderr.splitlines():
        m = re.search(r"(Function Name|ScratchSize|LDS Size)[^:]*: (\S+)", line)
        if m and m[1] == "Function Name":
            used[m[2]] = name = {}
        elif m:
            name[m[1]] = int(m[2])
    used = {n: u for n, u in used.items() if "ward_f64" in n}
    assert len(used) == 9 + 9 * 8   # seven grids, shift, ternary; scales, samples, optimiser
    for n, u in used.items():
        assert u["ScratchSize"] == 0 and u["LDS Size"] <= 512 + 64, (n, u)
