"""Stores of the persistent schedules (CPU, from the compiler's output).

A unit of these schedules is published without a release fence at device
scope: what another workgroup of the launch reads has to be stored with
device-scope stores (sc1 on gfx950).  An ordinary store would be read stale
only now and then, so this is checked in the code itself: tc_async and
tc_sync, whose every result is read by later units, hold no other global
store, and the bodies that both kinds of schedule use do not compile without
the caller's choice.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_11937_amd import build

BODIES = """
#include "tile_ops.h"
#include "tile_ops_lp.h"
__global__ void k(double* C, const double* P, const float* Q, int64_t lda) {
  __shared__ union alignas(512) { TcUpdSmem upd; TcTrsmSmem trsm; TcPotrfSmem potrf; } sm;
  %s
}
"""


@pytest.fixture(scope="module")
def hipcc():
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    build.gen_tuned_tiles()
    return ["hipcc", *build.HIPFLAGS, "-I", build.GEN_DIR, "-I", build.CSRC, "-x", "hip"]


def test_persistent_kernels_store_at_device_scope(hipcc, tmp_path):
    out = tmp_path / "k.s"
    subprocess.run([*hipcc, "-S", "--cuda-device-only", os.path.join(build.CSRC, "kernels.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    lines = out.read_text().splitlines()
    for kernel in ("tc_async", "tc_sync"):
        start = next(i for i, l in enumerate(lines) if re.match(r"_Z\d+%s[A-Z].*:" % kernel, l))
        end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
        stores = [l.strip() for l in lines[start:end] if re.match(r"\s+(global|flat|buffer)_store", l)]
        assert len(stores) > 50
        assert [s for s in stores if not re.search(r"\bsc1\b", s)] == []


CALLS = {
    "tc_update_block%s(C, P, P, lda, 128, 128, 128, false, sm.upd);": ["<true>", "<false>"],
    "tc_update_block_lp%s(C, Q, Q, lda, lda, 128, 128, 128, false, sm.upd);": ["<TC_PREC_FP32, true>",
                                                                               "<TC_PREC_FP32, false>"],
    "tc_trsm_rows%s(C, P, lda, 128, 128, sm.trsm);": ["<true>", "<false>"],
    "(void)tc_potrf_tile%s(C, lda, 128, sm.potrf);": ["<true>", "<false>"],
}


@pytest.mark.parametrize("call", CALLS)
def test_bodies_take_the_choice_from_the_caller(hipcc, tmp_path, call):
    def compiles(args):
        (tmp_path / "k.hip").write_text(BODIES % (call % args))
        return subprocess.run([*hipcc, "-fsyntax-only", "--cuda-device-only", str(tmp_path / "k.hip")],
                              capture_output=True).returncode == 0
    for args in CALLS[call]:
        assert compiles(args)
    assert not compiles("<TC_PREC_FP32>" if "_lp" in call else "")
