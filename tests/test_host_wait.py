"""The host's wait for a kernel's publication (`wait_tag` in csrc/prims.hip),
compiled for the host with g++ from the library source over a stand-in for the
stream: a word that is set soon is seen without a wait on the stream, a long
wait sleeps in the stream's own (so it honours the device's scheduling flag)
instead of holding a core, and a stream that fails or ends without the
publication ends the wait."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_1904_08553_amd", "csrc", "prims.hip")

HARNESS = r"""
#include <time.h>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <stdexcept>
#include <thread>
using hipError_t = int;
constexpr int hipSuccess = 0, hipErrorNotReady = 600, hipErrorUnknown = 999;
struct Stream {  // a stream that ends some time from now
  std::mutex mu;
  std::condition_variable cv;
  bool ended = false;
  int status = hipSuccess, waits = 0;
  void end(int s) {
    std::lock_guard<std::mutex> lk(mu);
    ended = true;
    status = s;
    cv.notify_all();
  }
};
using hipStream_t = Stream*;
static hipError_t hipStreamQuery(hipStream_t s) {
  std::lock_guard<std::mutex> lk(s->mu);
  return s->ended ? s->status : hipErrorNotReady;
}
static hipError_t hipStreamSynchronize(hipStream_t s) {
  std::unique_lock<std::mutex> lk(s->mu);
  ++s->waits;
  s->cv.wait(lk, [&] { return s->ended; });
  return s->status;
}
struct DeviceError : std::runtime_error {
  using std::runtime_error::runtime_error;
};
#define DC_HIP(x)                                    \
  do {                                               \
    if ((x) != hipSuccess) throw DeviceError("hip"); \
  } while (0)
struct HostTag {
  uint32_t* host;
  uint32_t* dev;
  uint32_t value;
};
%s
static double cpu_ms() {
  timespec t;
  clock_gettime(CLOCK_THREAD_CPUTIME_ID, &t);
  return t.tv_sec * 1e3 + t.tv_nsec * 1e-6;
}
enum Outcome { SEEN, DEVICE, NO_PUBLICATION };
// The wait for a word set (publish) and a stream ended (status) after us.
static Outcome wait(int us, bool publish, int status, int* waits, double* cpu) {
  uint32_t word = 0;
  Stream s;
  HostTag tag{&word, nullptr, 7};
  std::thread gpu([&] {
    std::this_thread::sleep_for(std::chrono::microseconds(us));
    if (publish) __atomic_store_n(&word, 7u, __ATOMIC_RELEASE);
    s.end(status);
  });
  Outcome o = SEEN;
  const double t0 = cpu_ms();
  try {
    wait_tag(tag, &s);
  } catch (const DeviceError&) {
    o = DEVICE;
  } catch (const std::runtime_error&) {
    o = NO_PUBLICATION;
  }
  *cpu = cpu_ms() - t0;
  gpu.join();
  *waits = s.waits;
  return o;
}
int main() {
  int waits, bad = 0;
  double cpu;
  {  // already there: no call into the runtime at all
    uint32_t word = 7;
    Stream s;
    HostTag tag{&word, nullptr, 7};
    wait_tag(tag, &s);
    bad += s.waits != 0;
  }
  bad += wait(100000, true, hipSuccess, &waits, &cpu) != SEEN;
  printf("a wait of 100 ms: %%.1f ms of the thread's time, %%d waits\n", cpu, waits);
  bad += cpu > 20 || waits != 1;
  bad += wait(2000, false, hipSuccess, &waits, &cpu) != NO_PUBLICATION;
  bad += wait(2000, false, hipErrorUnknown, &waits, &cpu) != DEVICE;
  printf("bad %%d\n", bad);
  return bad != 0;
}
"""


def _source():
    text = open(SRC).read()
    m = re.search(r"^(constexpr int SPIN_US = [^;]*;\n)?void wait_tag\(.*?\n\}\n", text, re.S | re.M)
    assert m, "wait_tag not found in prims.hip"
    return m.group(0)


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_host_wait(tmp_path):
    src, exe = tmp_path / "host_wait.cpp", tmp_path / "host_wait"
    src.write_text(HARNESS % _source())
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
