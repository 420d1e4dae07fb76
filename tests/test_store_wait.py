"""store_through (csrc/common.h) is a 16-byte store in inline assembly, which the compiler does not see to be one: the wait that it puts between such
a store and an instruction that overwrites the stored registers has to stand in the assembly itself.  Compared on code compiled here."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_10526_amd import build

KERNELS = """
#include "common.h"
using namespace massv;
template <bool THROUGH> __device__ inline void put(floatx4* p, floatx4 v) {
    for (int i = 0; i < 4; ++i) {
        if constexpr (THROUGH) store_through(p + i, v); else p[i] = v;
        v += 1.f;                                    // into the registers just stored
    }
    p[4] = v;
}
__global__ void plain(floatx4* p, const floatx4* q) { put<false>(p, *q); }
__global__ void through(floatx4* p, const floatx4* q) { put<true>(p, *q); }
"""


def test_the_wait_behind_a_store_through(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    src, out = tmp_path / "stores.hip", tmp_path / "stores.s"
    src.write_text(KERNELS)
    subprocess.run([hipcc, *[f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")], "--cuda-device-only", "-S", str(src), "-o", str(out),
                    "-I", os.path.join(build.ROOT, "include"), "-I", os.path.join(build.HERE, "csrc")], check=True, capture_output=True)
    waits = {}
    for name in ("plain", "through"):
        body = re.search(rf"^_Z\d+{name}.*?s_endpgm", out.read_text(), re.S | re.M).group(0)
        lines = [l.strip() for l in body.splitlines() if l.strip() and not l.strip().startswith(";")]
        after = [re.match(r"s_nop (\d+)", b) for a, b in zip(lines, lines[1:]) if a.startswith("global_store_dwordx4") and (name == "plain" or a.endswith("sc1"))]
        waits[name] = [int(m.group(1)) if m else -1 for m in after]
    assert max(waits["plain"]) >= 1, waits               # where the compiler sees the store: two wait states on gfx950
    assert len(waits["through"]) == 4 and min(waits["through"]) >= max(waits["plain"]), waits
