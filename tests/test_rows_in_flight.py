"""Rows that are to be in flight together are read without a wait among them, in the gfx950 code that the library's own
sources compile to (no GPU)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2209_07663_amd", "csrc")


@pytest.fixture(scope="module")
def gather(tmp_path_factory):
    """The text of every gather_pool kernel, by the kernel's name."""
    from paper_2209_07663_amd.build import HIPCC_FLAGS
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("needs the ROCm toolchain")
    out = tmp_path_factory.mktemp("code") / "gather.s"
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([hipcc] + flags + ["-S", "--cuda-device-only", os.path.join(CSRC, "gather.hip"), "-o", str(out)],
                          stderr=subprocess.DEVNULL)
    return {m[1]: m[2] for m in re.finditer(r"^(\w*gather_pool_kernel\w*):(.*?)\ts_endpgm", out.read_text(), re.M | re.S)}


def _reads_together(code):
    """How many 16-byte reads follow one another without a wait for memory, in the code's order."""
    runs, n = [], 0
    for op in re.findall(r"global_load_dwordx4|s_waitcnt vmcnt|global_store_dword", code):
        if op == "global_load_dwordx4":
            n += 1
        elif n:
            runs.append(n)
            n = 0
    return runs


@pytest.mark.parametrize("source,runs", [
    ("9TableRowsIfLi4E", [8, 8, 8]),             # bags of any length, of up to two IDs, of one: eight rows each
    ("11QuotRemRowsIfLi4ELi4ELb1E", [8, 8, 8]),  # four IDs, two rows each
])
def test_fp32_rows_are_read_together(gather, source, runs):
    code = [text for name, text in gather.items() if source in name]
    assert len(code) == 1 and _reads_together(code[0]) == runs
