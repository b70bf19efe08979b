"""Registers that the built kernels spill, read from the library's own kernel descriptions (no GPU)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

READELF = next((c for c in ("/opt/rocm/llvm/bin/llvm-readelf", shutil.which("llvm-readelf")) if c and os.path.exists(c)), None)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: description} of every kernel in libvp.so."""
    from paper_2208_06874_amd import vp
    if READELF is None:
        pytest.skip("needs llvm-readelf")
    if not os.path.exists(vp.LIB_PATH):
        pytest.skip("libvp.so is not built")
    data = open(vp.LIB_PATH, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    found = {}
    at = data.find(magic)
    while at >= 0:      # one bundle per source file: a count, then (offset, size, length of the target's name, name) each
        count, = struct.unpack_from("<Q", data, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count if count < 16 else 0):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" not in target or not size:
                continue
            path = tmp_path_factory.mktemp("code") / "object"
            path.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for part in re.split(r"\n  - (?=\.a)", notes)[1:]:
                name = re.search(r"\.name: +(\S+)", re.sub(r"\.args:.*?\n    \.(?=\w+:)", ".", part, flags=re.S)).group(1)
                found[name] = {f: int(v) for f, v in re.findall(r"\.(\w+): +(\d+)\b", part)}
        at = data.find(magic, at + 1)
    assert found
    return found


def test_many_row_kernels_that_trade_nothing_spill_next_to_nothing(kernels):
    """project_gemm_lds_kernel<KT, MASKED, TOP1, GATHER, SETS>: what the trade of sets' bests takes is paid by the kernels that
    trade.  The others have no scratch, but for the masked lists at d_pad = 512, which reload four registers."""
    seen = 0
    for name, desc in kernels.items():
        m = re.search(r"project_gemm_lds_kernelILi(\d+)ELb(\d)ELb(\d)ELb(\d)ELb(\d)E", name)
        if not m or m.group(5) == "1":
            continue
        seen += 1
        masked_list = m.group(2) == "1" and m.group(3) == "0"
        assert desc["vgpr_spill_count"] <= (4 if masked_list else 0), (name, desc)
        assert desc["private_segment_fixed_size"] <= (12 if masked_list else 0), (name, desc)
        assert desc["sgpr_spill_count"] <= (32 if masked_list else 0), (name, desc)
    assert seen == 36
