"""What the compiler made of the kernels, read from the built library's gfx950 code: properties that show in no result and that the source
cannot force."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2305_13525_amd as axo

OBJDUMP = shutil.which("llvm-objdump", path=os.pathsep.join(["/opt/rocm/llvm/bin", os.environ.get("PATH", "")]))
pytestmark = pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: [(address, instruction, address that it branches to or None)]}"""
    where = tmp_path_factory.mktemp("code")
    shutil.copy(axo.library_path(), where / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=where, check=True, stdout=subprocess.DEVNULL)
    code = [f for f in os.listdir(where) if "gfx950" in f]
    assert len(code) == 1, code
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", code[0]], cwd=where, check=True, stdout=subprocess.PIPE, text=True).stdout
    found, start, name = {}, 0, None
    for line in text.splitlines():
        head = re.match(r"([0-9a-f]+) <(\w+)>:", line)
        if head:
            start, name = int(head[1], 16), head[2]
            found[name] = []
            continue
        m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):(?:.*\+0x([0-9a-f]+)>)?", line)
        if m and name:
            to = start + int(m[3], 16) if m[3] and re.match("s_c?branch", m[1]) else None
            found[name].append((int(m[2], 16), m[1], to))
    assert len(found) > 40
    return found


def loops(code):
    """The instructions of each loop that holds matrix instructions and no branch but its own."""
    for at, _, to in code:
        if to is not None and to < at and at - to < 1 << 14:
            body = [(t, b) for a, t, b in code if to <= a <= at]
            if sum(b is not None for _, b in body) == 1 and any("v_mfma" in t for t, _ in body):
                yield [t for t, _ in body]


def test_loops_wait_for_loads_only_where_they_say_so(kernels):
    """A step of a tile's loop waits for its loads once, ahead of its barrier.  The compiler adds a wait of its own where it believes that some
    other load is under way into a register that the loop writes."""
    n = 0
    for name, code in kernels.items():
        if not re.search("gemm_(small|mid|rect|mixed|group)_kernel", name):
            continue
        for body in loops(code):
            barriers = sum(t == "s_barrier" for t in body)
            if barriers:
                waits = [t for t in body if t.startswith("s_waitcnt") and "vmcnt" in t]
                assert len(waits) == barriers, (name, len(body), waits)
                n += 1
    assert n >= 60, n


def test_both_kinds_of_stores_are_there(kernels):
    """Tiles of at most 128 x 128 store rows plainly where they straddle cache lines and past the caches where they do not.  Two branches that
    differ in that alone are one to the compiler, a plain one."""
    n = 0
    for name, code in kernels.items():
        m = re.search(r"gemm_(small|rect|mid)_kernelILi(\d)ELi(\d)E", name)
        if not m:
            continue
        stores = [t for _, t, _ in code if t.startswith("global_store_dwordx4")]
        assert any(t.endswith(" nt") for t in stores) and any(not t.endswith(" nt") for t in stores), (name, len(stores))
        n += 1
    assert n == 20, n
