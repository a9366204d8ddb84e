"""The address arithmetic of the CG updates over whatever their state holds.

The update kernels load the residual from a ring slot before they look at
whether the system updates at all, and the state lives in the caller's
uninitialised workspace.  The slot of a system that does not update must lie in
the ring for any bytes in the fields that only an iteration writes.  Checked on
the host: the function is the kernels' own, compiled for the host.
"""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1801_01473_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

MAIN = r"""
#include <cstdio>
#include <cstring>
#include "sysred.h"
using namespace lqcd;
int main() {
  static SysState S;
  const int its[] = {-1, -2, -31, -32, int(0x80000000), int(0xC3C3C3C3), 0x7FFFFFFF, 0x3F3F3F3F, 0, 30, 31};
  for (int it : its)
    for (int R = 1; R <= kMaxWin + 1; ++R) {
      std::memset(&S, 0, sizeof(S));
      S.iter_k = it;  // left by whoever used the workspace before
      for (bool fused : {true, false}) {
        const BaseStep u = base_step(S, 0, fused);
        if (u.go || u.slot % R < 0 || u.slot % R >= R) {
          std::printf("iter_k %d R %d fused %d: slot %d\n", it, R, int(fused), u.slot % R);
          return 1;
        }
      }
      if (it >= 0 && it < 0x7FFFFFFF) {  // a system that updates: the slot after iteration it
        S.upd_any = 1;
        if (base_step(S, 0, true).slot != it + 1) return 2;
      }
    }
  return 0;
}
"""


def test_ring_slot_of_finished_systems(tmp_path):
    src, exe = tmp_path / "slots.hip", tmp_path / "slots"
    src.write_text(MAIN)
    res = subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-I", CSRC, str(src),
                          "-o", str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
