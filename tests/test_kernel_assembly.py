"""Wait states in the compiled kernels (host only).

The loads into LDS are inline assembly, whose insides the compiler's hazard
pass does not look into, so the assembly of every kernel is checked here for
the wait states that it would have put there."""
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2607_01817_amd import build


def _instructions(text):
    """The instruction lines of an assembly file, without comments; "" where
    control can join (a label)."""
    out = []
    for ln in text.splitlines():
        ln = ln.split(";", 1)[0].split("//", 1)[0].strip()
        if ln.endswith(":"):
            out.append("")
        elif re.match(r"[a-z]+_", ln):
            out.append(ln)
    return out


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions of each HIP source, compiled as the library is."""
    tmp = tmp_path_factory.mktemp("asm")

    def compile_one(src):
        out = str(tmp / (src + ".txt"))
        subprocess.run([build.HIPCC, "-x", "hip", *build.COMMON, "--offload-device-only", "-S",
                        os.path.join(build.CSRC, src), "-o", out], check=True, capture_output=True)
        with open(out) as f:
            return src, _instructions(f.read())

    srcs = [s for s in build.SOURCES if s.endswith(".hip")]
    with concurrent.futures.ThreadPoolExecutor(len(srcs)) as ex:
        return dict(ex.map(compile_one, srcs))


def _lds_loads(ins):
    return [i for i, x in enumerate(ins) if re.match(r"(buffer|global)_load_\w+ .*\blds\b", x)]


def test_m0_is_not_read_right_after_its_write(kernels):
    """A load into LDS takes its address from M0 and needs a wait state after a
    scalar write of M0."""
    seen = 0
    for src, ins in kernels.items():
        for i in _lds_loads(ins):
            seen += 1
            assert not re.match(r"s_\w+ m0,", ins[i - 1]), f"{src}: {ins[i - 1]} / {ins[i]}"
    assert seen > 100   # the check looks at the loads that it is about


def _vgprs(operand):
    m = re.match(r"v\[(\d+):(\d+)\]$|v(\d+)$", operand)
    if not m:
        return set()
    lo, hi = (m[1], m[2]) if m[1] else (m[3], m[3])
    return set(range(int(lo), int(hi) + 1))


def test_wide_stores_keep_their_data_for_a_wait_state(kernels):
    """A store of more than 8 bytes per lane reads its data registers after it
    has issued, with a scalar offset too: the instruction behind it does not
    write them."""
    seen = 0
    for src, ins in kernels.items():
        for st, after in zip(ins, ins[1:]):
            if not re.match(r"buffer_store_dwordx[34] .*, s\d+ offen", st):
                continue
            seen += 1
            data = _vgprs(st.split(None, 1)[1].split(",")[0])
            written = _vgprs(after.partition(" ")[2].split(",")[0]) if re.match(r"(v|ds)_", after) else set()
            assert data and not data & written, f"{src}: {st} / {after}"
    assert seen > 10
