"""The compiler's output for a source of the library (gfx950 assembly), made
once per test session and shared by the tests that read it."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2606_11937_amd import build


def hipcc():
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    build.gen_tuned_tiles()
    return ["hipcc", *build.HIPFLAGS, "-I", build.GEN_DIR, "-I", build.CSRC, "-x", "hip"]


@functools.lru_cache(maxsize=None)
def _lines(source):
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "k.s")
        subprocess.run([*hipcc(), "-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", out], check=True,
                       capture_output=True)
        with open(out) as f:
            return f.read().splitlines()


def kernel_body(source, kernel):
    """Lines of the kernel of that (plain) name."""
    lines = _lines(source)
    start = next(i for i, l in enumerate(lines) if re.match(r"_Z%d%s[A-Z].*:" % (len(kernel), kernel), l))
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    return lines[start:end]


def resources(source):
    """{mangled kernel name: {"lds", "vgprs", "spills"}} from the metadata."""
    keys = {".group_segment_fixed_size": "lds", ".vgpr_count": "vgprs", ".vgpr_spill_count": "spills"}
    out, cur = {}, {}
    for l in _lines(source):
        m = re.match(r"\s+(?:- )?(\.\w+):\s*(\S+)", l)
        if not m:
            continue
        if m.group(1) in keys:
            cur[keys[m.group(1)]] = int(m.group(2))
        elif m.group(1) == ".name" and m.group(2).startswith("_Z"):
            cur["name"] = m.group(2)
        if len(cur) == 4:
            out[cur.pop("name")] = cur
            cur = {}
    return out
