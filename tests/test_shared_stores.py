"""Stores of the persistent schedules (CPU, from the compiler's output).

A unit of these schedules is published without a release fence at device
scope: what another workgroup of the launch reads has to be stored with
device-scope stores (sc1 on gfx950).  An ordinary store would be read stale
only now and then, so this is checked in the code itself: tc_async and
tc_sync, whose every result is read by later units, hold no other global
store, and the bodies that both kinds of schedule use do not compile without
the caller's choice.
"""
import re
import subprocess

import pytest

import device_listing

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
    return device_listing.hipcc()


def test_persistent_kernels_store_at_device_scope():
    for kernel in ("tc_async", "tc_sync"):
        lines = device_listing.kernel_body("kernels.hip", kernel)
        stores = [l.strip() for l in lines if re.match(r"\s+(global|flat|buffer)_store", l)]
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
