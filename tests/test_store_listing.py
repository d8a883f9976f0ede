"""Wide stores in the listing of the built library (no GPU): some are written in inline assembly (stores through the L2), where the
compiler does not see a store and keeps no wait states behind it."""
import re
import subprocess

import pytest
import test_kernel_listing as K

pytestmark = K.pytestmark


def kernels_with_wide_stores(tmp_path):
    found = {}
    with open(K.LIB, "rb") as f:
        data = f.read()
    for i, code in enumerate(K.code_objects(data)):
        path = tmp_path / f"code{i}.o"
        path.write_bytes(code)
        text = subprocess.run([K.OBJDUMP, "-d", "--no-show-raw-insn", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        body = None
        for line in text.splitlines():
            head = re.match(r"([0-9a-f]+) <(\S+)>:", line)
            if head:
                body, start = found.setdefault(head[2], []), int(head[1], 16)
                continue
            m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line)
            if m and body is not None:
                jump = re.search(r"<\S+?\+0x([0-9a-f]+)>", line)
                operands = [o.strip().split(" ")[0] for o in m[2].split(",")] if m[2] else []
                body.append(K.Instruction(int(m[3], 16), m[1], operands, start + int(jump[1], 16) if jump else None))
    return {name: body for name, body in found.items() if any(is_wide_store(i) for i in body)}


def is_wide_store(i):
    return re.fullmatch(r"global_store_dwordx[34]|buffer_store_dwordx[34]|flat_store_dwordx[34]", i.mnemonic) is not None


def test_data_of_wide_stores_is_not_overwritten_too_early(tmp_path):
    # gfx950 reads the data of a store of more than eight bytes up to two issue slots late: a vector instruction that overwrites it
    # needs two wait states in between
    found = kernels_with_wide_stores(tmp_path)
    if not found:
        pytest.fail("no wide stores found: the listing was not understood")
    bad = []
    for name, body in found.items():
        before = K.predecessors(body)
        for n, ins in enumerate(body):
            if not (ins.is_vector or ins.is_mfma) or not ins.operands:
                continue
            written = ins.registers(ins.operands[0])
            if written:
                data = lambda i: i.registers(i.operands[0 if i.mnemonic.startswith("buffer") else 1])
                bad += [f"{name}: {ins.mnemonic} {ins.operands} at {ins.address:#x} behind {body[p].mnemonic} {body[p].operands}"
                        for p in K.within(body, before, n, 2, lambda i: is_wide_store(i) and bool(data(i) & written))]
    assert not bad, f"{len(bad)} places, first ones:\n" + "\n".join(bad[:8])
