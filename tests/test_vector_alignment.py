"""What the compiler is told about the addresses of 16-byte accesses: in the kernels for rows of any pitch a vector may start at
any element, so their loads and stores must not promise 16-byte alignment.  (An `aligned` attribute on a typedef is lost when
the type passes through a template argument, and nothing warns.)  Read from the intermediate code of the sources."""
import os
import re
import subprocess

import pytest

from paper_2110_15032_amd import build

# kernels whose template arguments say "any pitch", by mangled name, and the largest alignment that their elements give
KERNELS = {
    "softmax_kernels.hip": [("xent_grad_kernelILb1ELi8ELNS0_9RowLayoutE%d" % i, 2) for i in (1, 2)] + [("xent_grad_kernelILb0ELi4ELNS0_9RowLayoutE%d" % i, 4) for i in (1, 2)],
    "boxing_kernels.hip": [("box_cast_reduce_kernelILi8ELb0E", 4), ("box_cast_gather_any_kernel", 4), ("box_reduce_any_kernel", 4), ("box_copy_any_kernelIt", 2), ("box_copy_any_kernelIj", 4)],
}


@pytest.mark.parametrize("src", KERNELS)
def test_unaligned_vectors_promise_no_more_than_their_elements(src, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    out = str(tmp_path / "ir.ll")
    flags = [f for f in build.FLAGS if f != "-O3"]
    subprocess.run([build.HIPCC, *flags, "-O1", "--cuda-device-only", "-emit-llvm", "-S", os.path.join(build.CSRC, src), "-o", out], check=True, capture_output=True)
    bodies = {m[1]: m[0] for m in re.finditer(r"^define [^\n]*@(\w+)\(.*?^}", open(out).read(), re.S | re.M)}
    for name, most in KERNELS[src]:
        found = {n: b for n, b in bodies.items() if name in n}
        assert found, f"no kernel {name}"
        for n, body in found.items():
            vectors = re.findall(r"(?:load|store) <(?:4 x (?:i32|float)|8 x i16)>[^\n]*addrspace\(1\)[^\n]*?align (\d+)", body)
            assert vectors, f"{n}: no 16-byte access"
            assert all(int(a) <= most for a in vectors), f"{n}: alignments {sorted(set(vectors))}, at most {most} holds"
