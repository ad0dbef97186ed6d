"""What the compiler made of kernels whose sources hold it off something (host only: gfx950 assembly of the library's own sources)."""
import functools
import re
import subprocess
import tempfile

import pytest

import __graft_entry__ as entry


@functools.lru_cache(maxsize=None)
def assembly(source):
    hipcc = entry.os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not entry.os.path.exists(hipcc):
        pytest.skip("no hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        asm = entry.os.path.join(tmp, "kernels.s")
        subprocess.run([hipcc, *entry.HIPCC_FLAGS, "--cuda-device-only", "-S", entry.os.path.join(entry.CSRC, source), "-o", asm],
                       check=True, stderr=subprocess.DEVNULL)
        with open(asm) as f:
            return f.read()


def kernels(source):
    """name -> assembly of the kernels of a source file"""
    parts = re.split(r"^(_ZN3pyr\w+):.*$", assembly(source), flags=re.M)
    return {name: body.split(".end_amdhsa_kernel")[0] for name, body in zip(parts[1::2], parts[2::2]) if ".amdhsa_kernel" in body}


def test_merged_gather_chooses_its_sources_in_registers():
    """No lane loads the pointer of its source: 64-bit loads by vector instructions, or a copy of the arguments in scratch memory."""
    merged = {n: asm for n, asm in kernels("select.hip").items() if "select_gather_kernel" in n}
    assert len(merged) == 2
    for name, asm in merged.items():
        assert not re.search(r"(global|flat|scratch)_load_dwordx2 ", asm), name
        assert re.search(r"\.amdhsa_private_segment_fixed_size 0\n", asm), name


@pytest.mark.parametrize("source,kernel,count", [("select.hip", r"select_gather_kernel.*TwoSources", 1), ("select.hip", "select_topk", 4),
                                                 ("gather.hip", "gather_(multi|rows)", 2), ("attention_tile.hip", "attention_tile_kernel", 4),
                                                 ("score.hip", "strip_kernel", 6)])
def test_short_arguments(source, kernel, count):
    """112 bytes at most, implicit arguments included, which a use of the grid's or the workgroup's size brings along."""
    found = {m[1]: int(m[0]) for m in re.findall(r"\.kernarg_segment_size: (\d+).*?\.name: +(\w+)", assembly(source), flags=re.S) if re.search(kernel, m[1])}
    assert len(found) == count and max(found.values()) <= 112, found
