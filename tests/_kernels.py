"""What the compiler recorded about every gfx950 kernel of the built libnif.so: LDS, scratch and registers
(the code objects' metadata notes, printed by llvm-readelf)."""
import os
import re
import struct
import subprocess
import tempfile

_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
_READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


def _code_objects(lib):
    data = open(lib, "rb").read()
    at = data.find(_MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        if n < 16:                                       # else: the text occurs elsewhere
            p = at + 32
            for _ in range(n):
                off, size, idn = struct.unpack_from("<QQQ", data, p)
                if b"gfx950" in data[p + 24:p + 24 + idn] and size:
                    yield data[at + off:at + off + size]
                p += 24 + idn
        at = data.find(_MAGIC, at + 24)


def kernels(lib):
    """{mangled name: dict(lds, scratch, vgprs)}"""
    out = {}
    for obj in _code_objects(lib):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(obj)
            f.flush()
            txt = subprocess.run([_READELF, "--notes", f.name], capture_output=True, text=True, check=True).stdout
        for k in re.split(r"\n  - ", txt)[1:]:
            name = re.search(r"\.name: +(\S+)\n", k)
            lds = re.search(r"\.group_segment_fixed_size: +(\d+)", k)
            if not (name and lds):
                continue
            names = re.findall(r"\.name: +(\S+)\n", k)   # the arguments have names too: the kernel's is mangled
            out[[v for v in names if v.startswith("_Z")][-1]] = dict(
                lds=int(lds.group(1)), scratch=int(re.search(r"\.private_segment_fixed_size: +(\d+)", k).group(1)),
                vgprs=int(re.search(r"\.vgpr_count: +(\d+)", k).group(1)))
    return out
