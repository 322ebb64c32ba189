"""The schedules that the autotuner times include the built-in policy, so a
tuned batch is never left with a slower schedule than an untuned one.  The list
is made on the host: a small program linked against the library prints it."""
import os
import shutil
import subprocess

import pytest

from paper_1704_08897_amd import bhx, build as B

PROGRAM = r"""
#include <cstdio>
#include "bhx_runtime.h"
int main() {
  const bhx::Schedule d;
  for (int transform : {0, 1, 2})
    for (int eligible : {0, 1}) {
      bhx_opts o;
      bhx_default_opts(&o);
      o.transform = transform;
      const bhx::Resolved R = bhx::resolve_opts(&o);
      for (const bhx::Schedule& s : bhx::autotune_candidates(R, eligible, 24))
        std::printf("%d %d %d\n", transform, eligible,
                    s.rows_cap == d.rows_cap && s.occ_s == d.occ_s && s.occ_r == d.occ_r &&
                        s.occ_c == d.occ_c && s.occ_d == d.occ_d && s.transform == transform);
    }
}
"""


def test_built_in_policy_is_a_candidate(tmp_path):
    if shutil.which(B.HIPCC) is None:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "main.hip", tmp_path / "main"
    src.write_text(PROGRAM)
    flags = [f for f in B.FLAGS if f not in ("-shared", "-O3")]
    r = subprocess.run([B.HIPCC, *flags, "-O0", "-I", B.CSRC, "-I", os.path.dirname(bhx.HEADER_PATH),
                        str(src), "-L", B.HERE, "-l:libbhx.so", f"-Wl,-rpath,{B.HERE}", "-o",
                        str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    rows = [tuple(map(int, l.split())) for l in r.stdout.splitlines()]
    for transform in (0, 1, 2):
        for eligible in (0, 1):
            assert (transform, eligible, 1) in rows
