"""Checks of the machine code built from loss_bf16.hip and ceilings.hip, without a GPU.  Their matrix products and transposing
LDS reads are inline assembly, so the compiler does not keep their wait states: nothing may move accumulators or fragments about
between the products or write their operands just before one, the accumulators may be read only behind the wait states at the
head of the epilogue, and what a transposing read fetches only behind a wait for it."""
import glob
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
    from paper_2603_06619_amd import build
    d = tmp_path_factory.mktemp("isa")
    lib = os.path.join(str(d), "lib.so")
    sources = glob.glob(os.path.join(build.CSRC, "*")) + [os.path.join(build.ROOT, "include", "nat.h"), build.__file__]
    built = nat.library_path()
    if os.path.exists(built) and os.path.getmtime(built) >= max(os.path.getmtime(f) for f in sources):
        os.symlink(built, lib)
    else:                                                 # not the code that is there: one of its own
        build.build(lib_path=lib, obj_dir=str(tmp_path_factory.mktemp("obj")))
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, stdout=subprocess.DEVNULL)
    found = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(str(d), f)], check=True,
                              stdout=subprocess.PIPE, text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S+)>:\n((?:[ \t].*\n)+)", text, flags=re.M):
            if "mfma_nt_kernel" in name or "probe_mfma_kernel" in name:
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
                moves = [y for y in body if re.match(r"v_accvgpr|v_(pk_)?mov_b|scratch_|buffer_", y)]
                assert not moves, (name, moves[:4])
            block = []
        assert loops, name


def registers(x):
    """("a" or "v", number) of every register that an instruction names."""
    return {(k, n) for k, lo, hi, one in re.findall(r"\b([av])(?:\[(\d+):(\d+)\]|(\d+)\b)", x)
            for n in range(int(lo or one), int(hi or one) + 1)}


def every_path(code, step, start):
    """Follows every path of the control flow: step(state, instruction, the one before) gives the state behind an instruction."""
    index = {at: i for i, (_, at, _) in enumerate(code)}
    seen, todo = set(), [(0, start)]
    while todo:
        i, state = todo.pop()
        while (i, state) not in seen:
            seen.add((i, state))
            x, _, to = code[i]
            assert not re.match(r"s_(setpc|swappc|call)", x), x
            state = step(state, x, code[i - 1][0])
            if x.startswith("s_endpgm"):
                break
            if x.startswith("s_cbranch"):
                todo.append((index[to], state))
            i = index[to] if x.startswith("s_branch") else i + 1
    assert len(seen) > 500


def test_accumulators_are_read_behind_the_wait_states(kernels):
    # after a product, nothing but products names its result before the wait states
    def step(results, x, before):
        if x.startswith("v_mfma"):
            return results | registers(x.split(",")[0])
        if x == "s_nop 7" and before == "s_nop 15":
            return frozenset()
        assert not results & registers(x), (name, x)
        return results

    for name, code in kernels.items():
        every_path(code, step, frozenset())


def written_by_vector_alu(x):
    if not x.startswith("v_"):
        return set()
    operands = x.split(",")
    return registers(operands[0]) | (registers(operands[1]) if "_swap" in x else set())


def aged(state, x, keep):
    """(register, wait states since) behind x, as long as they are fewer than `keep`."""
    n = int(x.split()[1]) + 1 if x.startswith("s_nop") else 1
    return {(r, age + n) for r, age in state if age + n < keep}


def test_product_operands_are_not_written_right_before(kernels):
    # two wait states between a vector instruction that writes a register and a product that reads it: what the compiler keeps
    # in front of a product that it knows
    def step(recent, x, _):
        if x.startswith("v_mfma"):
            sources = registers(",".join(x.split(",")[1:]))
            assert not sources & {r for r, _ in recent}, (name, x)
            return frozenset(aged(recent, x, 2))
        return frozenset(aged(recent, x, 2) | {(r, 0) for r in written_by_vector_alu(x)})

    for name, code in kernels.items():
        every_path(code, step, frozenset())


def test_transposing_reads_are_waited_for(kernels):
    def step(pending, x, _):
        if x.startswith("s_waitcnt") and "lgkmcnt(0)" in x:
            return frozenset()
        if x.startswith("ds_read_b64_tr_b16"):
            result, address = x.split(",")[0], x.split(",")[1]
            assert not pending & registers(address), (name, x)
            reads.append(x)
            return pending | registers(result)
        assert not pending & registers(x), (name, x)
        return pending

    reads = []
    for name, code in kernels.items():
        every_path(code, step, frozenset())
    assert reads


def test_results_leave_in_whole_lines(kernels):
    # dW goes through LDS: no store takes accumulators as they lie, in which an instruction would write half a line of 16 rows
    for name, code in kernels.items():
        if "DWeightEpilogue" not in name:
            continue
        stores = [x for x, _, _ in code if re.match(r"(global|flat)_store_dwordx4", x)]
        staged = [x for x, _, _ in code if re.match(r"ds_write_b128 v\d+, a\[", x)]
        assert stores and staged, name
        assert not any(re.search(r", a\[", x) for x in stores), name


def test_dh_scales_are_loaded_together(kernels):
    # the per-token scales of dH, a 4-byte load each, stand in front of the first result: loaded block by block of tokens each would wait
    # for memory in turn.  Behind a store of results (bf16, 8 or 16 bytes per lane) there is no such load
    found = 0
    for name, code in kernels.items():
        if "DHiddenEpilogue" not in name:
            continue
        loads = [i for i, (x, _, _) in enumerate(code) if re.match(r"global_load_dword ", x)]
        packs = [i for i, (x, _, _) in enumerate(code) if x.startswith("v_cvt_pk_bf16_f32")]
        found += len(loads)
        assert loads and packs, name
        for first, last in zip(loads, loads[1:]):
            assert not any(first < i < last for i in packs) or any(code[i][0].startswith("v_mfma") for i in range(first, last)), name
    assert found >= 16
