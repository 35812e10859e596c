"""Host-side check of the generated gfx950 code of the kernels that write their barriers as
inline asm (seq_global.hip, joint2.hip): no wavefront arrives at a workgroup barrier with an LDS
access of its own still in flight.  Another wavefront may overwrite, behind the barrier, what
such an access has yet to read, and the LDS does not order the accesses of different wavefronts.
The compiler sees to it for the barriers it makes itself; for those in asm the wait has to be there
on every path.  No GPU needed."""
import os
import re
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2503_16815_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

LABEL = re.compile(r"^([.\w$]+):")
LDS = re.compile(r"^ds_\w+")
BRANCH = re.compile(r"^s_(c?)branch\w*\s+([.\w$]+)")


def functions(text):
    """(name, [(label or None, instruction)]) of every kernel in the assembly."""
    name, body, label = None, [], []
    for line in text.splitlines():
        code = line.split(";", 1)[0].strip()
        m = LABEL.match(code)
        if m:
            if re.search(r"^\s*\.type\s+" + re.escape(m.group(1)) + r",@function", text, re.M):
                name, body = m.group(1), []
            label.append(m.group(1))
            code = code[m.end():].strip()
        if code.startswith(".Lfunc_end") or (m and m.group(1).startswith(".Lfunc_end")):
            if name:
                yield name, body
            name, label = None, []
            continue
        if name and code and not code.startswith("."):
            body.append((label, code))
            label = []


def unguarded_barriers(body):
    """Barriers that some path reaches with an LDS access behind the last full wait."""
    at = {l: i for i, (labels, _) in enumerate(body) for l in labels}
    pending_in, bad, work = {}, set(), [(0, False)]
    while work:
        i, pending = work.pop()
        while i < len(body):
            if pending_in.get(i, -1) >= pending:
                break
            pending_in[i] = int(pending)
            code = body[i][1]
            if LDS.match(code):
                pending = True
            elif code.startswith("s_waitcnt") and ("lgkmcnt(0)" in code or re.match(r"s_waitcnt\s+0(x0+)?$", code)):
                pending = False
            elif code.startswith("s_barrier") and pending:
                bad.add(i)
            elif code.startswith("s_endpgm"):
                break
            m = BRANCH.match(code)
            if m:
                work.append((at[m.group(2)], pending))
                if not m.group(1):
                    break
            i += 1
    return sorted(bad)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("src,kernel,builds", [("seq_global.hip", "sg_stream", 2), ("joint2.hip", "jt_sweep_all", 1)])
def test_no_lds_access_in_flight_at_a_barrier(src, kernel, builds):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "out.s")
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fno-gpu-rdc", "-Xclang", "-target-feature",
                        "-Xclang", "-packed-fp32-ops", "-w", "--cuda-device-only", "-S", "-o", out, os.path.join(CSRC, src)],
                       check=True, capture_output=True)
        bodies = {n: b for n, b in functions(open(out).read()) if kernel in n}
    assert len(bodies) == builds, list(bodies)
    for name, body in bodies.items():
        assert sum(c.startswith("s_barrier") for _, c in body) >= 4 and sum(bool(LDS.match(c)) for _, c in body) > 50
        bad = unguarded_barriers(body)
        assert not bad, (name, [[c for _, c in body[max(0, i - 6):i + 1]] for i in bad])
