"""Work-group end counts in the gfx950 code built here (no GPU): kernels whose last work-group reads
totals that all work-groups add to by atomics must wait for every wave's atomics before the barrier
that precedes the count.  The barrier alone orders nothing past the work-group."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2510_23679_amd as pdp

OBJDUMP = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))
KERNELS = {"k_ix_hist": 2, "k_join": 1, "k_join_persistent": 1}  # instances that count their work-groups
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(path):
    """The gfx950 code objects of every translation unit in the library."""
    blob = open(path, "rb").read()
    at = blob.find(MAGIC)
    while at >= 0:
        n = struct.unpack_from("<Q", blob, at + 24)[0]
        p = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 32)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    lib = os.path.join(os.path.dirname(pdp.__file__), "libpdp.so")
    if OBJDUMP is None or not os.path.exists(lib):
        pytest.skip("needs llvm-objdump and the built library")
    out = {}
    for i, code in enumerate(_code_objects(lib)):
        f = tmp_path_factory.mktemp("co") / f"{i}.co"
        f.write_bytes(code)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True, check=True).stdout
        for m in re.finditer(r"^[0-9a-f]+ <(\S+)>:\n((?:\t.*\n)+)", text, re.M):
            if re.search(r"\d(" + "|".join(KERNELS) + r")IL", m.group(1)):
                out[m.group(1)] = [x.strip().split("//")[0].strip() for x in m.group(2).splitlines()]
    assert out, "no kernel found in the library"
    return out


def _end_count(body):
    """The place of the end count: the kernel's last one-word atomic with a return value."""
    return max(i for i, x in enumerate(body) if re.match(r"global_atomic_(add|inc)\s.*sc0", x))


@pytest.mark.parametrize("name", list(KERNELS))
def test_every_wave_waits_before_the_end_count(kernels, name):
    seen = 0
    for sym, body in kernels.items():
        if not re.search(rf"\d{name}IL", sym) or (name != "k_ix_hist" and "ILb0E" not in sym):
            continue
        end = _end_count(body)
        barrier = max(i for i in range(end) if body[i].startswith("s_barrier"))
        adds = [i for i in range(barrier) if re.match(r"global_atomic_add", body[i]) and "sc0" not in body[i]]
        assert adds, f"{sym}: no totals"
        # straight to the barrier: past the last branch, so on every path from the totals
        straight = max([i for i in range(barrier) if body[i].startswith(("s_cbranch", "s_branch"))], default=0)
        assert any(re.match(r"s_waitcnt.*vmcnt\(0\)", x) for x in body[straight:barrier]), \
            f"{sym}: waves reach the barrier with their atomics in flight"
        seen += 1
    assert seen == KERNELS[name]
