"""CPU check of what the compiler gave the forms of the training kernel, read from the metadata of the library built here."""
import os
import re
import struct
import subprocess

import pytest

from paper_2009_04861_amd import binding as B

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects():
    """gfx950 code objects of the library: one bundle per translation unit."""
    data = open(B.LIB_PATH, "rb").read()
    for m in re.finditer(BUNDLE, data):
        at = m.start() + len(BUNDLE)
        entries, = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(entries):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            at += 24 + name
            if b"gfx950" in data[at - name:at]:
                yield data[m.start() + offset:m.start() + offset + size]


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs llvm-readelf")
def test_forms_without_scratch(tmp_path):
    """Template arguments of k_train: register slots, FULL, REGR, ROOMY, NARROW, DEEP, SPANS, TINY.  In regression and in the narrow
    forms scratch once came in unnoticed with code that these forms do not use; every form of up to eight slots does without,
    but for those with spans that many clauses share and that are held to as many wavefronts as they all but fill."""
    seen = {}
    for k, obj in enumerate(code_objects()):
        path = tmp_path / ("%d.co" % k)
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
        for block in re.split(r"\n  - \.", notes):
            name = re.search(r"\.name:\s+_ZN7tsetlin7k_trainILi(\d+)E((?:Lb[01]E){7})E", block)
            size = re.search(r"\.private_segment_fixed_size:\s+(\d+)", block)
            if name and size:
                seen[(int(name[1]),) + tuple(int(b) for b in re.findall(r"Lb([01])E", name[2]))] = int(size[1])
    assert len(seen) > 100
    with_scratch = {form: size for form, size in seen.items() if size and form[0] <= 8}
    held = {(slots, full, 0, 0, 0, deep, 1, 0) for slots, deep in ((1, 0), (1, 1), (3, 1)) for full in (0, 1)}
    assert set(with_scratch) <= held and max(with_scratch.values()) <= 48, with_scratch
