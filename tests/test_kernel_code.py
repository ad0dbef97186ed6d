"""What the compiler made of kernels whose sources hold it off something (host only: gfx950 assembly of the library's own sources)."""
import re
import subprocess

import pytest

import __graft_entry__ as entry


def kernels(source, tmp_path):
    """name -> assembly of the kernels of a source file"""
    asm = tmp_path / "kernels.s"
    hipcc = entry.os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not entry.os.path.exists(hipcc):
        pytest.skip("no hipcc")
    subprocess.run([hipcc, *entry.HIPCC_FLAGS, "--cuda-device-only", "-S", entry.os.path.join(entry.CSRC, source), "-o", str(asm)],
                   check=True, stderr=subprocess.DEVNULL)
    parts = re.split(r"^(_ZN3pyr\w+):.*$", asm.read_text(), flags=re.M)
    return {name: body.split(".end_amdhsa_kernel")[0] for name, body in zip(parts[1::2], parts[2::2]) if ".amdhsa_kernel" in body}


def test_merged_gather_chooses_its_sources_in_registers(tmp_path):
    """No lane loads the pointer of its source: 64-bit loads by vector instructions, or a copy of the arguments in scratch memory."""
    merged = {n: asm for n, asm in kernels("select.hip", tmp_path).items() if "select_gather_kernel" in n}
    assert len(merged) == 2
    for name, asm in merged.items():
        assert not re.search(r"(global|flat|scratch)_load_dwordx2 ", asm), name
        assert re.search(r"\.amdhsa_private_segment_fixed_size 0\n", asm), name
