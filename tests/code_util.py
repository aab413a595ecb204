"""The instructions of the kernels in the library as it is built."""
import os
import re
import subprocess
import tempfile

import paper_2003_06324_amd as g
from paper_2003_06324_amd import build
from test_wide_store_data import _code_objects


def kernels(name):
    """{template arguments ("true" and "false" as truth values, the rest as text): instructions} of a kernel's forms"""
    g.load_library()   # (builds it if it is not there)
    objdump = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "llvm", "bin", "llvm-objdump")
    found = {}
    for image in _code_objects(build.LIB):
        if name.encode() not in image:
            continue
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(image)
            f.flush()
            listing = subprocess.run([objdump, "-d", "--no-show-raw-insn", "--demangle", f.name], check=True, stdout=subprocess.PIPE,
                                     universal_newlines=True).stdout
        code = None
        for line in listing.splitlines():
            m = re.match(r"[0-9a-f]+ <(.*)>:$", line)
            if m:
                m = re.search(r"\b%s<([^>]*)>" % name, m.group(1))
                code = found.setdefault(tuple({"true": True, "false": False}.get(a, a) for a in m.group(1).split(", ")), []) if m else None
                continue
            line = line.split("//")[0].strip()
            if code is not None and line and not line.startswith(("s_nop", "s_code_end", "...")):
                code.append(line)
    return found
