"""What the compiler is told about addresses.  The entry points take weights,
maps and side buffers that start at any element, so no vector access of the
kernels that work on them may promise more than that: an address the compiler
takes for a multiple of 16 may be folded, split or combined on that promise.
Read from the LLVM IR of the kernels as they are built (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2608_02391_amd import build as B

# the kernels on a caller's weights and side buffers
KERNELS = ("k_perturb", "k_perturb_map", "k_perturb_dense", "k_restore_copy", "k_restore_dense", "k_restore_master",
           "k_backup_copy", "k_stage_master", "k_copy_map", "k_update", "k_update_map", "k_update_step", "k_fill_normal")
BITS = {"i8": 8, "i16": 16, "i32": 32, "i64": 64, "bfloat": 16, "float": 32, "double": 64}


@pytest.fixture(scope="module")
def accesses(tmp_path_factory):
    """kernel -> (bytes, promised alignment) of its vector accesses to global
    memory, the library's own tables (named globals) aside."""
    out = str(tmp_path_factory.mktemp("ir") / "kernels.ll")
    flags = [f for f in B.HIPCC_FLAGS if f != "-shared"]
    res = subprocess.run([B.hipcc(), *flags, "--offload-device-only", "-S", "-emit-llvm", "-I", B.INCLUDE, "-I", B.CSRC,
                          os.path.join(B.CSRC, "cpes_kernels.hip"), "-o", out], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-2000:]
    found, kernel = {}, None
    with open(out) as f:
        for line in f:
            m = re.match(r"define .*@(\w+)\(", line)
            if m:
                name = re.search(r"\d(k_[a-z_]+?)(?:I|E)", m.group(1))
                kernel = name.group(1) if name else m.group(1)
            m = re.search(r"(?:load|store) <(\d+) x (\w+)>.*ptr addrspace\(1\) (%|@)\S+, align (\d+)", line)
            if m and m.group(3) == "%":
                found.setdefault(kernel, []).append((int(m.group(1)) * BITS[m.group(2)] // 8, int(m.group(4))))
    return found


@pytest.mark.parametrize("kernel", KERNELS)
def test_vectors_promise_no_more_than_an_elements_alignment(accesses, kernel):
    got = [a for a in accesses.get(kernel, []) if a[0] >= 8]
    if kernel != "k_copy_map":                        # its accesses are single elements
        assert any(size == 16 for size, _ in got), "no vector access found: the reader of the IR has lost them"
    # bf16 weights allow 2, fp32 buffers and 32-bit maps 4, int64 maps 8
    assert [a for a in got if a[1] > 8] == []
