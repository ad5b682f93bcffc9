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
