"""The LDS stages of the update bodies, in the code the compiler makes of them.

A stage is filled again by direct-to-LDS loads as soon as the workgroup has
passed the barrier behind its last use, so at every barrier of these bodies
each wave's LDS reads have to be complete, not only issued: another wave's
load may overwrite what a read in flight has yet to fetch.  The bodies are
compiled alone for gfx950 and every path through their assembly is followed:
between an LDS read and the next barrier there is a wait for all of them.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_11937_amd import build

SRC = """
#include "tile_ops.h"
#include "tile_ops_lp.h"
union alignas(512) Smem {
  TcUpdSmem upd;
  TcPotrfSmem potrf;
};
extern "C" __global__ __launch_bounds__(TC_THREADS, 2) void k_syrk(double* C, const double* P, int64_t lda, int kd) {
  __shared__ Smem sm;
  (void)tc_syrk_block<false, false>(C, P, lda, kd, sm.upd, sm.potrf);
}
extern "C" __global__ __launch_bounds__(TC_THREADS, 2) void k_syrk_potrf(double* C, const double* P, int64_t lda, int kd,
                                                                         int* bad) {
  __shared__ Smem sm;
  *bad = tc_syrk_block<true, false>(C, P, lda, kd, sm.upd, sm.potrf);
}
extern "C" __global__ __launch_bounds__(TC_THREADS, 2) void k_update(double* C, const double* P, int64_t lda, int mr,
                                                                     int mc, int kd) {
  __shared__ TcUpdSmem sm;
  tc_update_block<false>(C, P, P, lda, mr, mc, kd, false, sm);
}
extern "C" __global__ __launch_bounds__(TC_THREADS, 2) void k_update_lp(double* C, const float* P, int64_t lda, int mr,
                                                                        int mc, int kd) {
  __shared__ TcUpdSmem sm;
  tc_update_block_lp<TC_PREC_FP32, false>(C, P, P, lda, lda, mr, mc, kd, false, sm);
}
"""


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("waits")
    (d / "k.hip").write_text(SRC)
    r = subprocess.run(["hipcc", *build.HIPFLAGS, "-I", build.CSRC, "-x", "hip", "-S", "--cuda-device-only",
                        str(d / "k.hip"), "-o", str(d / "k.s")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return (d / "k.s").read_text().splitlines()


def body(listing, name):
    start = next(i for i, l in enumerate(listing) if l.startswith(name + ":"))
    end = next(i for i in range(start, len(listing)) if listing[i].startswith(".Lfunc_end"))
    ops = [l.split(";")[0].strip() for l in listing[start + 1:end]]
    return [o for o in ops if o and (not o.startswith(".") or o.endswith(":"))]


@pytest.mark.parametrize("kernel", ["k_syrk", "k_syrk_potrf", "k_update", "k_update_lp"])
def test_reads_complete_at_barriers(listing, kernel):
    ops = body(listing, kernel)
    at = {o[:-1]: i for i, o in enumerate(ops) if o.endswith(":")}
    assert sum(o.startswith("ds_read") for o in ops) > 8 and sum(o.startswith("s_barrier") for o in ops) > 1
    # over every path: before instruction i, may a read be in flight
    work, seen = [(0, False)], set()
    while work:
        i, pending = work.pop()
        if i >= len(ops) or (i, pending) in seen:
            continue
        seen.add((i, pending))
        op = ops[i]
        if op.startswith("ds_read"):
            pending = True
        elif op.startswith("s_waitcnt") and re.search(r"lgkmcnt\(0\)", op):
            pending = False
        elif op.startswith("s_barrier"):
            assert not pending, f"{kernel}: a read may be in flight at the barrier of line {i}: {ops[i - 4:i + 1]}"
        branch = re.match(r"s_c?branch\w*\s+(\S+)", op)
        if branch:
            work.append((at[branch.group(1)], pending))
        if not op.startswith(("s_branch", "s_endpgm")):
            work.append((i + 1, pending))
