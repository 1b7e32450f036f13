"""The MFMAs of kernels_gemm_tall.hip are inline assembly, so the compiler inserts no wait between them and the first use of
their results: in the built code no accumulator register may be read, copies included, between an MFMA and the wait that the
source puts behind the last one.  Read from the library that was built here (no GPU)."""
import os
import re
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def kernels(lib, tmp_path):
    """(name, instructions in the order they lie) of every kernel of kernels_gemm_tall.hip."""
    (tmp_path / "lib.so").write_bytes(open(lib, "rb").read())
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    for obj in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            name, _, body = part.partition(">:")
            if "gemm_bf16_tall_kernel" in name:
                yield name, [l.split("//")[0].strip() for l in body.splitlines() if l.startswith("\t")]


def reads_accumulator(x):
    op, _, args = x.partition(" ")
    if not op.startswith(("ds_write", "buffer_store", "global_store")):
        args = args.partition(",")[2]          # the first operand is written
    return re.search(r"\ba(\d|\[)", args) is not None


def early_reads(ins):
    """Instructions other than MFMAs that read an accumulator register behind an MFMA with no wait of 32 states between."""
    pending, bad = False, []
    for i, x in enumerate(ins):
        if x.startswith("v_mfma"):
            pending = True
        elif x == "s_nop 15" and ins[i - 1] == "s_nop 15":
            pending = False
        elif pending and reads_accumulator(x):
            bad.append(x)
    return bad


def test_no_result_is_read_before_the_wait(tmp_path):
    import paper_2511_08923_amd as T
    if not os.access(OBJDUMP, os.X_OK):
        pytest.skip("no llvm-objdump")
    seen = 0
    for name, ins in kernels(T.LIB_PATH, tmp_path):
        assert any(x.startswith("v_mfma") for x in ins)
        assert early_reads(ins) == [], name
        seen += 1
    assert seen == 19            # 2 to 10 row tiles x 2 column tiles; 2 to 9, 11 and 12 x 3
