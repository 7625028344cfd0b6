"""Stores written in asm that take their address from scalar registers: a vector memory instruction may not
read a scalar register soon after a vector instruction wrote it, and the compiler keeps no distance in
front of asm, so the instructions right ahead of each such store must be the scalar ones that make its address."""
import re
import subprocess

from paper_2605_10670_amd import build


def test_asm_stores_make_their_scalar_address(tmp_path):
    out = tmp_path / "data.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.HIPCC, *flags, "-w", "-S", "--cuda-device-only", "-o", str(out),
                    build.HERE + "/csrc/data.hip"], check=True)
    lines = [s for s in (line.split(";")[0].strip() for line in out.read_text().splitlines()) if s]
    stores = 0
    for i, line in enumerate(lines):
        m = re.match(r"global_store_dwordx4 v\d+, v\[\d+:\d+\], s\[(\d+):(\d+)\] sc0 sc1$", line)
        if m:
            stores += 1
            low, high = lines[i - 2], lines[i - 1]
            assert low.startswith(f"s_add_u32 s{m[1]},") and high.startswith(f"s_addc_u32 s{m[2]},"), lines[i - 4:i + 1]
    assert stores > 0
