"""Host logic of the copies of a call, on the CPU: pieces of the sources compiled with g++ and stand-ins
for what they call."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2503_04424_amd", "csrc")


def source_of(file, head):
    """The function (with its template line) whose definition matches `head`, by its braces."""
    text = open(os.path.join(CSRC, file)).read()
    at = re.search(head, text)
    assert at, head
    depth = 0
    for k in range(text.index("{", at.end()), len(text)):
        depth += {"{": 1, "}": -1}.get(text[k], 0)
        if depth == 0:
            return text[at.start():k + 1]


def run(tmp_path, program):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(program)
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", str(exe), str(src)], check=True, capture_output=True, timeout=300)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, (out.returncode, out.stdout, out.stderr)


def test_results_for_another_device_are_not_written_by_a_kernel(tmp_path):
    """Memory of this device only; what belongs to another one, host and managed memory, and addresses that
    the runtime does not know go through the runtime's copy."""
    run(tmp_path, """
#include <cstdio>
enum hipError_t { hipSuccess, hipErrorInvalidValue };
enum hipMemoryType { hipMemoryTypeUnregistered, hipMemoryTypeHost, hipMemoryTypeDevice, hipMemoryTypeManaged };
struct hipPointerAttribute_t { hipMemoryType type; int device; };
static hipPointerAttribute_t known;
static int current = 0;
static hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  if (!p) return hipErrorInvalidValue;
  *a = known;
  return hipSuccess;
}
static hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
static hipError_t hipGetLastError() { return hipSuccess; }
""" + source_of("memdet.hip", r"static bool device_memory\(") + """
int main() {
  int x, bad = 0;
  for (current = 0; current < 3; ++current)
    for (int type = 0; type < 4; ++type)
      for (int device = 0; device < 3; ++device) {
        known = {(hipMemoryType)type, device};
        if (device_memory(&x) != (type == hipMemoryTypeDevice && device == current)) {
          std::printf("type %d of device %d, current %d\\n", type, device, current);
          ++bad;
        }
      }
  return bad + (device_memory(nullptr) ? 1 : 0);
}
""")


def test_copies_read_no_further_than_the_last_entry(tmp_path):
    """A matrix whose last entry is the last one of its memory (rows longer than the order: a view of some
    columns): behind it lies a page that cannot be read.  Rows of pieces of 16 bytes, orders around them and
    around leaves; what arrives is the lower part up to the end of each row's leaf on the diagonal."""
    run(tmp_path, """
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include <sys/mman.h>
#define __global__
#define __launch_bounds__(x)
#define __restrict__
struct Index { unsigned x; };
static Index blockIdx, threadIdx;
struct f64x2 { double v[2]; };
struct f32x4 { float v[4]; };
""" + source_of("kernels_reduce.h", r"template <[^>]*>\n__global__[^\n]*\bcopy_lower_kernel\(") + """
template <typename T, typename E>
int check(int64_t n, int64_t ld) {
  const size_t page = 4096, bytes = ((n - 1) * ld + n) * sizeof(T), room = (bytes + page - 1) / page * page;
  char* base = (char*)mmap(nullptr, room + page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  if (base == MAP_FAILED || mprotect(base + room, page, PROT_NONE)) return 1;
  T* src = (T*)(base + room - bytes);
  for (int64_t i = 0; i < n; ++i)
    for (int64_t j = 0; j < n; ++j) src[i * ld + j] = T(1 + i * n + j);
  const int64_t ldd = (n + 31) / 32 * 32;
  std::vector<T> dst((size_t)(n * ldd), T(-1));
  std::printf("n %ld ld %ld size %zu\\n", (long)n, (long)ld, sizeof(T));
  std::fflush(stdout);
  for (blockIdx.x = 0; blockIdx.x < n; ++blockIdx.x)
    for (threadIdx.x = 0; threadIdx.x < 256; ++threadIdx.x) copy_lower_kernel<T, E>(src, ld, dst.data(), ldd, n);
  int bad = 0;
  for (int64_t i = 0; i < n; ++i)
    for (int64_t j = 0; j < n && j < (i / 64 + 1) * 64; ++j) bad += dst[i * ldd + j] != T(1 + i * n + j);
  munmap(base, room + page);
  return bad;
}
int main() {
  int bad = 0;
  for (int64_t n : {1, 2, 3, 5, 63, 64, 65, 66, 127, 129, 130, 131, 257}) {
    bad += check<double, f64x2>(n, (n + 1) / 2 * 2) + check<double, f64x2>(n, (n + 1) / 2 * 2 + 2) + check<double, double>(n, n);
    bad += check<float, f32x4>(n, (n + 3) / 4 * 4) + check<float, f32x4>(n, (n + 3) / 4 * 4 + 4) + check<float, float>(n, n);
  }
  return bad != 0;
}
""")


def test_scaled_copy_that_was_asked_for_goes_before_long_rows():
    """A budget with room for the pivot-scaled copies beside a copy of the matrix with its shortest rows holds
    them; more room, and the rows start on 128-byte lines."""
    import paper_2503_04424_amd as M
    M.load()
    for n, dtype, bs in [(323, "f64", 64), (323, "f32", 64), (1000, "f32", 128), (1001, "f64", 256)]:
        ask = lambda budget, flags=M.FLAG_SCALED_COPY: M.mdet_workspace_query(n, dtype, bs, budget, False, flags, True)[0]
        scaled = ask(0) - ask(0, 0)
        low, high = 0, ask(0, 0)
        while high - low > 1:
            mid = (low + high) // 2
            try:
                ask(mid, 0)
                high = mid
            except M.MemdetError:
                low = mid
        assert scaled > 0 and high < ask(0, 0)
        assert ask(high + scaled) == high + scaled and ask(ask(0)) == ask(0) and ask(ask(0) - 1) == high + scaled
        assert ask(high) == high and ask(high + scaled - 1) <= high + scaled - 1
