"""Register and scratch use of the built library's kernels, from the metadata that the
compiler puts beside them (the notes of every gfx950 code object in libpisco.so)."""
from __future__ import annotations

import os
import struct
import subprocess
import tempfile

import yaml

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1908_05662_amd", "libpisco.so")
READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
_CACHE: dict = {}


def _code_objects(data: bytes):
    """The gfx950 entries of every offload bundle: magic, count, then (offset, size, target)."""
    at = data.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, p)
        p += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length].decode()
            p += 24 + length
            if target.endswith("gfx950") and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


def kernels() -> dict:
    """Demangled kernel name (namespaces and arguments dropped) -> metadata dict."""
    if _CACHE:
        return _CACHE
    if not os.path.exists(LIB):
        from paper_1908_05662_amd.build import build

        build()
    with open(LIB, "rb") as f:
        data = f.read()
    found = []
    for obj in _code_objects(data):
        with tempfile.NamedTemporaryFile(suffix=".co") as t:
            t.write(obj)
            t.flush()
            text = subprocess.run([READELF, "--notes", t.name], check=True, capture_output=True, text=True).stdout
        found += yaml.safe_load(text[text.index("---"):text.index("...")])["amdhsa.kernels"]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), check=True,
                           capture_output=True, text=True).stdout.splitlines()
    for name, k in zip(names, found):
        name = name.replace("pisco::", "").replace("(anonymous namespace)::", "").replace("void ", "").split("(")[0]
        _CACHE[name] = k
    return _CACHE
