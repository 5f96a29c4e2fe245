"""The block pool of a context is looked at under its lock: an allocation that
failed and wants the pool's blocks back waits while another thread holds the
pool (a grid freed meanwhile), instead of reading its table beside it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2410_15227_amd")

PROGRAM = r"""
#include <atomic>
#include <chrono>
#include <thread>
#include "common.hpp"
using namespace sphmap;
int main() {
  BlockPool pool;
  auto refused = [&] {  // no device holds 2^60 bytes
    Arena a;
    a.spare = &pool;
    try { a.get("x", (size_t)1 << 60); } catch (const Error &e) { return e.code == SPHMAP_ENOMEM; }
    return false;
  };
  if (!refused()) return 2;
  std::atomic<bool> done{false};
  pool.mu.lock();
  std::thread t([&] { if (refused()) done = true; });
  std::this_thread::sleep_for(std::chrono::milliseconds(700));
  const bool early = done;
  pool.mu.unlock();
  t.join();
  return early ? 3 : done ? 0 : 4;
}
"""


def test_failed_allocation_waits_for_the_pool(tmp_path):
    lib = os.path.join(PKG, "libsphmap.so")
    if not os.path.exists(lib):
        from paper_2410_15227_amd import build
        build.build()
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(PKG, "csrc"), str(src), lib, "-L/opt/rocm/lib", "-lamdhip64", "-lpthread",
                    "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib", "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], timeout=60).returncode == 0
