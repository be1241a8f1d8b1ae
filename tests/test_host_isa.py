"""Checks of the machine code built from loss_bf16.hip, without a GPU.  Its matrix products are inline assembly, so the
compiler does not keep their wait states: nothing may move accumulators or fragments about between them, and the
accumulators may be read only behind the wait states at the head of the epilogue."""
import os
import re
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump is not installed")
    import paper_2603_06619_amd as nat
    if not os.path.exists(nat.library_path()):
        from paper_2603_06619_amd import build
        build.build()
    d = tmp_path_factory.mktemp("isa")
    lib = os.path.join(str(d), "lib.so")
    os.symlink(nat.library_path(), lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, stdout=subprocess.DEVNULL)
    found = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(str(d), f)], check=True,
                              stdout=subprocess.PIPE, text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S+)>:\n((?:[ \t].*\n)+)", text, flags=re.M):
            if "mfma_nt_kernel" in name:
                found[name] = [line.split("//")[0].strip() for line in body.splitlines()]
    assert found
    return found


def test_products_are_not_mixed_with_register_moves(kernels):
    for name, code in kernels.items():
        at = [i for i, x in enumerate(code) if x.startswith("v_mfma")]
        # a k-loop is a run of products with less than 64 instructions between two of them
        runs, start = [], 0
        for q in range(1, len(at) + 1):
            if q == len(at) or at[q] - at[q - 1] > 64:
                runs.append((at[start], at[q - 1]))
                start = q
        assert runs, name
        for first, last in runs:
            assert all(x.startswith("v_mfma_f32_16x16x32_bf16 a[") for x in code[first:last + 1] if x.startswith("v_mfma")), name
            moves = [x for x in code[first:last + 1] if re.match(r"v_accvgpr|v_mov|scratch_|buffer_", x)]
            assert not moves, (name, moves[:4])
            # wait states before anything reads an accumulator
            after = code[last + 1:]
            settle = next(i for i, x in enumerate(after) if x == "s_nop 15")
            assert after[settle + 1] == "s_nop 7", name
            early = [x for x in after[:settle] if re.search(r"\ba\[?\d", x) and not x.startswith("v_accvgpr_write")]
            assert not early, (name, early[:4])
