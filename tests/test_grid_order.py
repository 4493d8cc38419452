"""Host logic of csrc/one_grid.hpp, the order between launches whose workgroups wait for each other,
compiled by the host compiler against stand-ins for the HIP calls it makes: no GPU, every failure forced."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PROGRAM = r'''
#include "one_grid.hpp"
#include <cstdio>
#include <cstring>
#include <string>
static std::string failing, calls;
static hipError_t call(const char *name) {
  calls += name; calls += " ";
  return failing == name ? hipErrorUnknown : hipSuccess;
}
static bool capturing = false;
extern "C" {
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return call("capturing");
}
hipError_t hipGetDevice(int *d) { *d = 0; return call("device"); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)0x10; return call("create"); }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return call("wait"); }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return call("record"); }
hipError_t hipStreamSynchronize(hipStream_t) { return call("synchronize"); }
hipError_t hipGetLastError(void) { return call("clear"); }
}
static void grid(const char *what, const char *fail, bool captured = false, bool wanted = true) {
  failing = fail; capturing = captured; calls.clear();
  bool ordered;
  {
    snn::OneGridAtATime order(nullptr, wanted);
    ordered = order.ordered();
    calls += "| ";
  }
  printf("%s: %d %s\n", what, (int)ordered, calls.c_str());
}
int main() {
  grid("unwanted", "", false, false);
  grid("create", "create");
  grid("first", "");
  grid("second", "");
  grid("captured", "", true);
  for (const char *f : {"capturing", "device", "wait", "record"}) grid(f, f);
  grid("last", "");          // no lock is left behind
}
'''

EXPECTED = {
    "unwanted": "0 |",
    "create": "0 capturing device create clear |",
    "first": "1 capturing device create | record",
    "second": "1 capturing device wait | record",
    "captured": "0 capturing clear |",
    "capturing": "0 capturing clear |",
    "device": "0 capturing device clear |",
    "wait": "0 capturing device wait clear |",
    "record": "1 capturing device wait | record clear synchronize",
    "last": "1 capturing device wait | record",
}


@pytest.fixture(scope="module")
def outcome(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid_order")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    f"-I{ROOT}/paper_2402_18994_amd/csrc", "-o", str(d / "main"), str(d / "main.cpp"), "-lpthread"], check=True)
    out = subprocess.run([str(d / "main")], check=True, capture_output=True, text=True, timeout=20).stdout
    return {k: v.strip() for k, v in (line.split(": ", 1) for line in out.splitlines())}


@pytest.mark.parametrize("case", list(EXPECTED))
def test_a_grid_that_could_not_be_ordered_is_not_called_ordered(outcome, case):
    """`0`: the caller launches a step at a time.  `1`: the launch is behind the grid before it, and the
    next one behind it - through the event, or because the host has waited for the stream."""
    assert outcome[case] == EXPECTED[case]
