"""The receive index's hand-over between workgroups, read from the compiler's output for its own source (built here with
the memory model's fences, MW_PUBLISH_FENCES=1; device code only, no GPU).

The wave that writes a workgroup's counts reports them, and the wave whose report is the last reads everybody's.  What must
hold in every kernel that contains the index: the other lanes' stores are ordered before the report, the report's value reaches
all lanes from the reporting one's register (an LDS word that the others read without a barrier is a race), every lane then has an
agent-scope acquire, and where the whole workgroup goes on, the barriers in between order global memory too and not LDS alone."""
import os
import re
import subprocess

import pytest

from paper_2605_22428_amd import build

REPORT = re.compile(r"(%\S+) = atomicrmw add ptr addrspace\(1\) \S+ i32 1 syncscope\(\"agent\"\) acq_rel")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("ir") / "mw_unpack.ll")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags +
                   ["-O1", "--cuda-device-only", "-S", "-emit-llvm", "-DMW_PUBLISH_FENCES=1", "-I", os.path.join(build.ROOT, "include"),
                    "-I", build.CSRC, os.path.join(build.CSRC, "mw_unpack.hip"), "-o", out], check=True, stderr=subprocess.DEVNULL)
    found, name = {}, None
    for line in open(out):
        line = line.strip()
        if line.startswith("define"):
            name = re.search(r"@(\S+?)\(", line).group(1)
            found[name] = []
        elif line == "}":
            name = None
        elif name and line:
            found[name].append(line)
    return {n: body for n, body in found.items() if "k_recv_indexIL" in n or "k_expand_index_nextIL" in n}


def _index_of(body, i, what, within):
    """The first of `within` lines from line i on (backwards if negative) that contains `what`, or -1."""
    step = 1 if within > 0 else -1
    for j in range(i, i + within, step):
        if 0 <= j < len(body) and what in body[j]:
            return j
    return -1


def test_the_index_publishes_by_the_rules(kernels):
    assert len(kernels) >= 8
    for name, body in kernels.items():
        reports = [i for i, line in enumerate(body) if REPORT.search(line)]
        assert len(reports) == 1, (name, len(reports))
        at = reports[0]
        assert _index_of(body, at, 'fence syncscope("agent") release', -12) >= 0, name
        assert _index_of(body, at, 'fence syncscope("wavefront") acquire', -12) >= 0, name + ": lanes not ordered before the report"
        acquired = [i for i, line in enumerate(body) if line.startswith('fence syncscope("agent") acquire')]
        assert len(acquired) == 1, name + ": only the reporting lane has acquired"
        assert _index_of(body, acquired[0], "@llvm.amdgcn.readfirstlane", -4) >= 0, name + ": the value does not come from one lane"
        full = [i for i, line in enumerate(body) if line == 'fence syncscope("workgroup") acquire' and "s.barrier" in body[i - 1]]
        assert len(full) >= 2, name + ": a workgroup goes on behind barriers that order LDS only"
