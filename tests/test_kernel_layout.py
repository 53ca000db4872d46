"""Where the star loops of the built FP64 kernels lie in memory: their runs of
8-byte instructions start on a multiple of 8 bytes, which the fetch needs to
keep up (csrc/shoot_fp64.hip, star_sum)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1703_09707_amd import build

LLVM = "/opt/rocm/llvm/bin"
SHAPE = "ILi8ELi4ELi16ELi1E"   # the tile shape a context starts with


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    objdump = os.path.join(LLVM, "llvm-objdump")
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(build.LIB):
        build.build()
    where = tmp_path_factory.mktemp("code")
    lib = shutil.copy(build.LIB, where)
    subprocess.run([objdump, "--offloading", lib], cwd=where, check=True, capture_output=True)
    text = ""
    for name in sorted(os.listdir(where)):
        if name.endswith("gfx950"):
            text += subprocess.run([objdump, "-d", str(where / name)], check=True,
                                   capture_output=True, text=True).stdout
    return {m.group(1): m.group(2) for m in
            re.finditer(r"^[0-9a-f]{16} <(\S+)>:\n((?:.+\n)*)", text, re.M)}


def star_loops(text):
    """The innermost loops with the one-star group's FP64 work, as lists of
    (address, bytes, mnemonic)."""
    code = [(int(a, 16), 4 * len(w.split()), t) for t, a, w in
            re.findall(r"^\t(.*?)\s*// ([0-9A-F]{12}): ((?:[0-9A-F]{8} ?)+)", text, re.M)]
    at = {a: i for i, (a, _, _) in enumerate(code)}
    loops = []
    for i, (a, n, t) in enumerate(code):
        m = re.match(r"s_cbranch\S+ (\d+)", t)
        if not m:
            continue
        back = int(m.group(1)) - 65536
        first = at.get(a + 4 + 4 * back)
        if -4000 < back < 0 and first is not None:
            body = code[first:i + 1]
            # no branch inside: the innermost; 64 multiply-adds: every ray's two sums
            if (sum("s_cbranch" in x[2] for x in body) == 1
                    and sum("v_fma" in x[2] for x in body) >= 64):
                loops.append(body)
    return loops


@pytest.mark.parametrize("kernel", ["shoot", "batch", "partial", "waves"])
def test_star_loop_starts_on_eight_bytes(listings, kernel):
    found = [t for n, t in listings.items() if kernel + "_fp64_kernel" + SHAPE in n]
    assert found
    for text in found:
        loops = [b for b in star_loops(text) if any("s_load" in x[2] for x in b)]
        assert loops
        for body in loops:
            first = next(a for a, n, t in body if t.startswith("v_") and n == 8)
            assert first % 8 == 0, hex(first)
