"""Waits that count loads (s_waitcnt vmcnt(n) in front of a barrier): the n youngest loads may still be in flight, so a
wait is right only if that many were issued behind the ones it stands for.  A load that the compiler left out would
make it too weak, without any test on the GPU showing it reliably; the assembly of the kernel shows it."""
import re
import subprocess

import pytest

from paper_2507_07149_amd import build


def _events(asm, kernel):
    """{function: [event, ...]} in program order; "lds": a load straight into LDS, "load": any other, int: a wait that
    lets so many stay in flight, "|": a barrier, "label" and "branch": the ends of a straight line."""
    out, cur = {}, None
    for line in asm.splitlines():
        m = re.match(r"(_Z\w*%s\w*):" % kernel, line)
        if m:
            cur = out.setdefault(m.group(1), [])
            continue
        s = line.strip()
        if cur is None or not s or s.startswith(";"):
            continue
        if s.startswith(".Lfunc_end"):
            cur = None
        elif re.match(r"\.LBB\w+:", s):
            cur.append("label")
        elif s.startswith(("s_cbranch", "s_branch")):
            cur.append("branch")
        elif s.startswith(("global_load_lds", "buffer_load")) and "lds" in s:
            cur.append("lds")
        elif re.match(r"(global|flat|buffer|scratch)_(load|store|atomic)", s):
            cur.append("load")
        elif s.startswith("s_waitcnt") and "vmcnt" in s:
            cur.append(int(re.search(r"vmcnt\((\d+)\)", s).group(1)))
        elif s.startswith("s_barrier"):
            cur.append("|")
    return out


@pytest.fixture(scope="module")
def matmul_asm():
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", build.CSRC + "/unpack_matmul.hip", "-o", "-"],
                       stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout


def test_weight_gradient_waits_for_the_rows_of_the_step_before(matmul_asm):
    """In front of a barrier of the wide kernel: every load of an earlier step has landed, those of the step itself may
    be in flight.  So a step that waits for vmcnt(n), n > 0, has issued at least n loads itself."""
    kernels = _events(matmul_asm, "k_unpack_matmul_wide")
    assert len(kernels) == 4                                   # two formats, one width or several
    for name, ev in kernels.items():
        counted = 0
        for i, e in enumerate(ev):
            if e != "|" or not isinstance(ev[i - 1], int) or ev[i - 1] == 0:
                continue
            start = i - 1                                      # the step: back to the barrier, label or branch before it
            while start and ev[start - 1] not in ("|", "label", "branch"):
                start -= 1
            issued = sum(x in ("lds", "load") for x in ev[start: i])
            assert issued >= ev[i - 1], f"{name}: vmcnt({ev[i - 1]}) behind {issued} loads of its own step"
            counted += 1
        assert counted >= 4, name                              # the four steps of the main loop
