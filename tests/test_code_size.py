"""Code size of the row body's stream kernels (K <= 5).  The word store of the
traceback is inlined at every one of its unrolled steps; with a path for every
output mode the kernel of K = 3 grew from 103 to 141 KB, and a launch whose
waves run different parts of it (64 KB of instruction cache) by up to 17 %."""
import glob
import os
import shutil
import struct

import pytest

from test_store_data_hazard import BUILD, LLVM, subprocess

LIMIT = 120 * 1024


def _kernel_sizes(obj, tmp):
    """{symbol: bytes} of the functions of an object's gfx950 code."""
    fat, co = os.path.join(tmp, "x.fatbin"), os.path.join(tmp, "x.co")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), "--dump-section=.hip_fatbin=" + fat, obj,
                    os.path.join(tmp, "x.o")], check=True, capture_output=True)
    subprocess.run([os.path.join(LLVM, "clang-offload-bundler"), "--type=o",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat,
                    "--output=" + co, "--unbundle"], check=True, capture_output=True)
    with open(co, "rb") as f:
        d = f.read()
    shoff, = struct.unpack_from("<Q", d, 40)
    n, = struct.unpack_from("<H", d, 60)
    sec = [struct.unpack_from("<IIQQQQIIQQ", d, shoff + 64 * i) for i in range(n)]
    out = {}
    for s in sec:
        if s[1] != 2:  # SHT_SYMTAB
            continue
        names = sec[s[6]][4]
        for k in range(s[5] // 24):
            nm, info, _, _, _, size = struct.unpack_from("<IBBHQQ", d, s[4] + 24 * k)
            if info & 15 == 2:  # STT_FUNC
                out[d[names + nm:d.index(b"\0", names + nm)].decode()] = size
    return out


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-objcopy")) or shutil.which("hipcc") is None,
                    reason="LLVM tools not available")
def test_row_body_stream_kernels_stay_small(tmp_path):
    objs = sorted(glob.glob(os.path.join(BUILD, "code_*.o")))
    if not objs:
        pytest.skip("library not built here (no objects under _build)")
    seen = 0
    for obj in objs:
        for name, size in _kernel_sizes(obj, str(tmp_path)).items():
            if "decode_kernelI" in name and any("FixedCodeILi%dE" % k in name for k in (3, 4, 5)):
                seen += 1
                assert size <= LIMIT, (name, size)
    assert seen >= 4
