"""What the compiler makes of the device code, where a source change that looks
harmless costs speed."""
import re
import subprocess

from paper_1302_1078_amd import build


def test_staged_windows_are_read_16_bytes_at_a_time(tmp_path):
    """The staged kernels read X rows from LDS by aligned 16-byte vectors: one ds_read_b128 each.  Read as
    element-aligned vectors they became two ds_read2_b32 or a ds_read2_b64 (2 to 5 % of the product)."""
    asm = str(tmp_path / "staged.s")
    flags = [f for f in build.CFLAGS if f != "-fPIC"]
    subprocess.run([build.HIPCC, *flags, "-w", "--cuda-device-only", "-S", build.CSRC + "/staged.hip", "-o", asm],
                   check=True, capture_output=True, text=True, timeout=600)
    with open(asm) as f:
        bodies = re.findall(r"^(_ZN\w*k_staged\w*):\s*;.*?\n(.*?)s_endpgm", f.read(), flags=re.M | re.S)
    assert len(bodies) >= 36, [b[0] for b in bodies]
    for name, body in bodies:
        assert "ds_read2_b32" not in body, name
        if "ELb1EEEv" not in name:  # not the instances that serve only the unstaged tiles
            assert body.count("ds_read_b128") >= 4, name
