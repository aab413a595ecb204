"""No kernel writes a data register of a store of more than 64 bits in the two issue slots behind it: the store may read the
register that late.  The compiler sees to it, but not for buffer stores with a scalar offset, so the built code is looked over."""
import concurrent.futures
import os
import re
import struct
import subprocess

import paper_2003_06324_amd as g
from paper_2003_06324_amd import build

SLOTS = 2
EM_AMDGPU = 224


def _code_objects(path):
    """The GPU code objects of a library: the ELF images inside it that are for the GPU."""
    data, at, out = open(path, "rb").read(), 0, []
    while True:
        at = data.find(b"\x7fELF\x02\x01\x01", at)
        if at < 0:
            return out
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            headers, = struct.unpack_from("<Q", data, at + 40)
            count, = struct.unpack_from("<H", data, at + 60)
            out.append(data[at:at + headers + 64 * count])
        at += 4


def _registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]$|v(\d+)$", operand)
    if not m:
        return set()
    return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))


def _overwritten(listing):
    """(wide stores, those whose data is written too early) of a disassembly."""
    stores, early, kernel, pending = 0, [], "", []   # pending: (data registers, slots left, store)
    for line in listing.splitlines():
        line = line.split("//")[0].strip()
        m = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
        if m:
            kernel, pending = m.group(1), []
            continue
        op, _, rest = line.partition(" ")
        operands = [x.strip() for x in re.split(r",\s*(?![^\[]*\])", rest)]
        if op.startswith("v_"):
            written = _registers(operands[0])
            early += [(kernel, store, line) for data, _, store in pending if data & written]
        slots = int(operands[0], 0) + 1 if op == "s_nop" else 1
        pending = [(data, left - slots, store) for data, left, store in pending if left > slots]
        m = re.match(r"(buffer|global|flat|scratch)_store_dwordx[34]$", op)
        if m:
            stores += 1
            pending.append((_registers(operands[0 if m.group(1) == "buffer" else 1]), SLOTS, line))
    return stores, early


def test_data_of_wide_stores_is_not_overwritten(tmp_path):
    g.load_library()   # (builds it if it is not there)
    objdump = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "llvm", "bin", "llvm-objdump")

    def look(item):
        path = str(tmp_path / ("%d.co" % item[0]))
        with open(path, "wb") as f:
            f.write(item[1])
        return _overwritten(subprocess.run([objdump, "-d", "--no-show-raw-insn", path], check=True, stdout=subprocess.PIPE,
                                           universal_newlines=True).stdout)

    with concurrent.futures.ThreadPoolExecutor(4) as ex:
        found = list(ex.map(look, enumerate(_code_objects(build.LIB))))
    assert sum(stores for stores, _ in found) > 0
    early = [x for _, e in found for x in e]
    assert not early, "%d, the first: %s" % (len(early), early[0])
