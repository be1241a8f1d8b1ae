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
                # (instruction, its offset in the kernel, offset of its branch target)
                code = [re.match(r"\s*(.*?)\s*// ([0-9A-F]+):[^<]*(?:<[^+>]*(?:\+0x([0-9a-f]+))?>)?", line).groups() for line in body.splitlines() if "//" in line]
                found[name] = [(x, int(at, 16) - int(code[0][1], 16), int(to or "0", 16)) for x, at, to in code]
    assert found
    return found


def test_products_are_not_mixed_with_register_moves(kernels):
    for name, code in kernels.items():
        block, loops = [], 0
        for x, _, _ in code + [("s_endpgm", 0, 0)]:
            if not re.match(r"s_c?branch|s_endpgm", x):
                block.append(x)
                continue
            products = [i for i, y in enumerate(block) if y.startswith("v_mfma")]
            if products:
                loops += 1
                body = block[products[0]:products[-1] + 1]
                assert all(y.startswith("v_mfma_f32_16x16x32_bf16 ") for y in body if y.startswith("v_mfma")), name
                moves = [y for y in body if re.match(r"v_accvgpr|v_mov_b32|scratch_|buffer_", y)]
                assert not moves, (name, moves[:4])
            block = []
        assert loops, name


def registers(x):
    """("a" or "v", number) of every register that an instruction names."""
    return {(k, n) for k, lo, hi, one in re.findall(r"\b([av])(?:\[(\d+):(\d+)\]|(\d+)\b)", x)
            for n in range(int(lo or one), int(hi or one) + 1)}


def test_accumulators_are_read_behind_the_wait_states(kernels):
    # along every path of the control flow: after a product, nothing but products names its result before the wait states
    for name, code in kernels.items():
        index = {at: i for i, (_, at, _) in enumerate(code)}
        seen, todo = set(), [(0, frozenset())]
        while todo:
            i, results = todo.pop()
            while (i, results) not in seen:
                seen.add((i, results))
                x, _, to = code[i]
                if x.startswith("v_mfma"):
                    results = results | registers(x.split(",")[0])
                elif x == "s_nop 7" and code[i - 1][0] == "s_nop 15":
                    results = frozenset()
                else:
                    assert not results & registers(x), (name, x)
                assert not re.match(r"s_(setpc|swappc|call)", x), (name, x)
                if x.startswith("s_endpgm"):
                    break
                if x.startswith("s_cbranch"):
                    todo.append((index[to], results))
                i = index[to] if x.startswith("s_branch") else i + 1
        assert len(seen) > 500, name
