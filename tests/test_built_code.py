"""What the compiler made of the kernels, read from the code objects of the built library (no GPU needed)."""
import os
import re
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Disassembly of every kernel of the library, by its mangled name."""
    from paper_2506_11277_amd import build
    objdump = os.path.join(LLVM, "llvm-objdump")
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(build.LIB):
        build.build_lib()
    folder = tmp_path_factory.mktemp("code")
    lib = folder / "lib.so"
    lib.write_bytes(open(build.LIB, "rb").read())
    subprocess.run([objdump, "--offloading", str(lib)], cwd=folder, check=True, stdout=subprocess.DEVNULL)
    found = {}
    for name in os.listdir(folder):
        if "gfx950" not in name:
            continue
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(folder / name)], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"^[0-9a-f]+ (?=<.*>:$)", text, flags=re.M)[1:]:
            label, _, body = part.partition(">:\n")
            found[label[1:]] = body
    return found


@pytest.mark.parametrize("kernel", ["gemm_fused16_kernelILi%dELi0E" % s for s in range(2, 10)] + ["gemm_fused_kernelILi%dE" % s for s in (1, 10, 16, 20)] +
                         ["gemm_halves_kernelILi4E", "gemm_halves16_kernelILi7E", "gemm_eighths_kernelILi7E", "gemm_eighths_whole_kernelI"] +
                         ["gemm_eighths_passes_kernelI", "gemm_passes_kernelI"])
def test_c_has_streaming_and_plain_stores(kernels, kernel):
    # columns of C on 64-byte boundaries are stored past the caches, others through them: both kinds of store have to be in
    # the code of every kernel that writes C from its accumulators (identical but for that, they are easily made one)
    bodies = [b for name, b in kernels.items() if kernel in name]
    stores = [re.findall(r"global_store_dwordx2 .*", b) for b in bodies]
    stores = [s for s in stores if s]                       # (split-k and dump variants write no C)
    assert stores, sorted(kernels)[:5]
    for s in stores:
        assert any(" nt" in line for line in s) and any(" nt" not in line for line in s), (kernel, s[:4])
