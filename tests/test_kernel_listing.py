"""What the GEMM kernels rely on and the compiler does not see, checked in the listing of the built library (no GPU): their
matrix-core instructions are written in inline assembly, so the wait states around them are the source's to keep."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2505_14669_amd", "libquartet.so")
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"

pytestmark = [pytest.mark.skipif(not os.path.exists(LIB), reason="HIP library not built (run __graft_entry__.build())"),
              pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump is not installed")]

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """the gfx950 code objects of the library's offload bundles: magic, number of entries, (offset, size, id length, id) each"""
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        entry = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + length]:
                yield data[at + offset:at + offset + size]
            entry += 24 + length
        at = data.find(MAGIC, at + len(MAGIC))


class Instruction:
    def __init__(self, address, mnemonic, operands, target, modifiers=()):
        self.address, self.mnemonic, self.operands, self.target, self.modifiers = address, mnemonic, operands, target, modifiers
        self.states = int(operands[0], 0) + 1 if mnemonic == "s_nop" else 1      # wait states it stands for

    def registers(self, operand):
        """vector registers an operand names: {("v" | "a", number)}"""
        m = re.fullmatch(r"-?\|?([va])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand)
        if not m:
            return set()
        first, last = (int(m[2]),) * 2 if m[2] else (int(m[3]), int(m[4]))
        return {(m[1], r) for r in range(first, last + 1)}

    def of(self, operands):
        return set().union(*(self.registers(o) for o in operands)) if operands else set()

    is_mfma = property(lambda self: self.mnemonic.startswith("v_mfma"))
    is_vector = property(lambda self: self.mnemonic.startswith("v_") and not self.is_mfma)


def kernels(tmp_path):
    """{kernel name: [Instruction]} of every kernel with matrix-core instructions"""
    found = {}
    with open(LIB, "rb") as f:
        data = f.read()
    for i, code in enumerate(code_objects(data)):
        path = tmp_path / f"code{i}.o"
        path.write_bytes(code)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        body = None
        for line in text.splitlines():
            head = re.match(r"([0-9a-f]+) <(\S+)>:", line)
            if head:
                body, start = found.setdefault(head[2], []), int(head[1], 16)
                continue
            m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line)
            if not m or body is None:
                continue
            jump = re.search(r"<\S+?\+0x([0-9a-f]+)>", line)
            operands = [o.strip().split(" ")[0] for o in m[2].split(",")] if m[2] else []
            body.append(Instruction(int(m[3], 16), m[1], operands, start + int(jump[1], 16) if jump else None, m[2].split()))
    return {name: body for name, body in found.items() if any(i.is_mfma for i in body)}


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if shutil.which("hipcc") is None and not os.path.exists(OBJDUMP):
        pytest.skip("no ROCm tools")
    found = kernels(tmp_path_factory.mktemp("listing"))
    assert len(found) >= 40 and sum("gemm_mxfp4_stream" in n for n in found) == 12
    return found


def predecessors(body):
    """for every instruction the instructions that may have run just before it"""
    index = {ins.address: n for n, ins in enumerate(body)}
    before = [[] for _ in body]
    for n, ins in enumerate(body):
        if ins.target is not None and ins.target in index:
            before[index[ins.target]].append(n)
        if n + 1 < len(body) and ins.mnemonic not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            before[n + 1].append(n)
    return before


def within(body, before, n, states, matches):
    """the instructions that may run fewer than `states` wait states before instruction n and match"""
    best, work, hits = {}, [(p, states) for p in before[n]], []
    while work:
        p, left = work.pop()
        if left <= best.get(p, 0):
            continue
        best[p] = left
        if matches(body[p]):
            hits.append(p)
        if left > body[p].states:
            work += [(b, left - body[p].states) for b in before[p]]
    return hits


def test_no_vector_instruction_writes_an_operand_right_before_a_matrix_core_instruction(listing):
    # a vector instruction's result needs two wait states before a matrix-core instruction may read it (operands, scales, accumulator)
    bad = []
    for name, body in listing.items():
        before = predecessors(body)
        for n, ins in enumerate(body):
            if not ins.is_mfma:
                continue
            reads = ins.of(ins.operands[1:])
            bad += [f"{name}: {body[p].mnemonic} {body[p].operands} before {ins.mnemonic} {ins.operands} at {ins.address:#x}"
                    for p in within(body, before, n, 2, lambda i: i.is_vector and i.registers(i.operands[0]) & reads)]
    assert not bad, f"{len(bad)} places, first ones:\n" + "\n".join(bad[:8])


ASSEMBLY_KERNELS = {"gemm_mxfp4_stream_kernelI": 4, "gemm_mxfp4_past_kernelI": 2, "gemm_mxfp4_past_wide_kernel": 1, "gemm_mxfp4_wide_kernelI": 2,
                    "mfma_ceiling": 1}


def test_results_of_matrix_core_instructions_are_not_touched_too_early(listing):
    # kernels whose matrix-core instructions are inline assembly: nothing but another of them reads or overwrites an accumulator within
    # 19 wait states of the instruction that forms it (the longest, a 16-pass instruction, needs that many)
    for kernel, count in ASSEMBLY_KERNELS.items():
        assert sum(kernel in name for name in listing) == count, kernel
    bad = []
    for name, body in listing.items():
        if not any(k in name for k in ASSEMBLY_KERNELS):
            continue
        before = predecessors(body)
        for n, ins in enumerate(body):
            if ins.is_mfma or ins.mnemonic.startswith("s_"):
                continue
            touched = ins.of(ins.operands)
            if touched:
                bad += [f"{name}: {ins.mnemonic} {ins.operands} at {ins.address:#x} behind {body[p].mnemonic} {body[p].operands}"
                        for p in within(body, before, n, 19, lambda i: i.is_mfma and i.registers(i.operands[0]) & touched)]
    assert not bad, f"{len(bad)} places, first ones:\n" + "\n".join(bad[:8])


# result stores of a wave's full tile: one per pass of eight rows and 32-column slice
@pytest.mark.parametrize("kernel,count,stores", [("gemm_mxfp4_stream_kernelI", 4, 64), ("gemm_mxfp4_stream_tile_kernelILi2ELi4E", 4, 32),
                                                 ("gemm_mxfp4_stream_tile_kernelILi2ELi2E", 4, 16), ("gemm_mxfp4_twin_kernelI", 4, 16),
                                                 ("gemm_mxfp4_wide_kernelI", 2, 64), ("gemm_mxfp4_wide_tile_kernelI", 2, 32),
                                                 ("gemm_mxfp4_past_kernelI", 2, 64), ("gemm_mxfp4_past_twin_kernelI", 2, 16),
                                                 ("gemm_mxfp4_past_wide_kernel", 1, 64)])
def test_a_full_tile_leaves_in_as_many_stores_as_the_kernels_count(listing, kernel, count, stores):
    # The wait behind a full tile lets that many younger operations be under way; with fewer stores it would let loads through that it is
    # there to wait for.  A lane's chunks (four columns: 16 bytes, 8 in bf16) do not touch, so no store instruction can hold two:
    # nothing wider than a chunk, and one store per chunk on each path: full tiles through the L2 (sc1), fp32 ones also past the caches (nt),
    # bf16 ones there in kernels of their own, and the whole chunks of ragged tiles (sc1), which the kernels for blocks of 256 columns do not have.
    names = [n for n in listing if kernel in n]
    assert len(names) == count
    for name in names:
        found = [i for i in listing[name] if i.mnemonic.startswith(("global_store", "buffer_store", "flat_store"))]
        assert all(i.mnemonic.startswith("global_store") for i in found)
        bf16 = "_past_" in kernel or re.search(r"kernelI(?:Li\dELi\dE)?Lb1E", name) is not None
        chunk = "global_store_dwordx2" if bf16 else "global_store_dwordx4"
        ragged = 0 if "_wide_" in kernel else stores
        through, past = (0, stores) if "_past_" in kernel else (stores, 0 if bf16 else stores)
        with_modifier = lambda modifier: sum(i.mnemonic == chunk and modifier in i.modifiers for i in found)
        assert with_modifier("sc1") == through + ragged and with_modifier("nt") == past
        assert sum(i.mnemonic in ("global_store_dwordx2", "global_store_dwordx3", "global_store_dwordx4") for i in found) == through + ragged + past
