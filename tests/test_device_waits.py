"""What one workgroup publishes to others inside a launch has arrived first.

The objective kernels' one-launch tails and the persistent kernel count a
finished workgroup (or publish a generation) from one thread behind a workgroup
barrier, and the workgroup that sees the last count reads what all of them
stored.  A barrier does not wait for global stores, so every wave has to wait for
its own ahead of it.  A missing wait shows in no result until the count overtakes
a store; it does show in the instructions, which are looked at here.
"""
import re
import subprocess

import pytest

from paper_1906_10598_amd import build

SOURCE = """
#define PT_INSTANCE_TU
#include "kernels.h"
namespace pt {{
template __global__ void k_eval<{T}, {S}, {C}, {mixed}>(BlockDesc, const double*, double*, int*, int*, EvalRule, int);
template __global__ void k_objective<{T}, {S}, {C}, {mode}, {slope}, 0>(
    int, int, int, int, const double*, const double*, const double*, const double*, const BlockDesc*);
template __global__ void k_fit_persistent<{T}, {S}, {C}, {mode}, {slope}>(const BlockDesc*, int, int, int, int, int*,
                                                                       uint64_t);
}}
"""


def _kernels(tmp_path, **kw):
    src, out = tmp_path / "waits.hip", tmp_path / "waits.s"
    src.write_text(SOURCE.format(**kw))
    subprocess.run(["/opt/rocm/bin/hipcc", *build.HIPCC_FLAGS, f"-I{build.CSRC}", "--offload-device-only", "-S", str(src),
                    "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    body, name = {}, None
    for line in out.read_text().splitlines():
        m = re.match(r"_ZN2pt\d+(k_[a-z_]+)I", line)
        if m and ":" in line:
            name = m.group(1)
            body[name] = []
        elif name and re.match(r"\s+[a-z]\w+", line):
            body[name].append(line.strip())
    return body


def _published_behind(ins, at):
    """Instructions between the barrier ahead of instruction `at` and the one before that."""
    bars = [k for k in range(at) if ins[k].startswith("s_barrier")]
    return ins[bars[-2] + 1:bars[-1]]


@pytest.mark.parametrize("kw", [dict(T="float", S=4, C=1, mode=0, mixed="false", slope="false"),
                                dict(T="float", S=16, C=4, mode=2, mixed="false", slope="true"),
                                dict(T="double", S=8, C=8, mode=1, mixed="true", slope="false")],
                         ids=lambda kw: "-".join(str(v) for v in kw.values()))
def test_stores_arrive_before_they_are_counted(tmp_path, kw):
    body = _kernels(tmp_path, **kw)
    # arrivals of a range and of the ranges; and the generation published to each of eight XCDs
    # (the ready lines start 1024 bytes into the counters)
    want = {"k_eval": 2, "k_objective": 2, "k_fit_persistent": 3}
    for name, count in want.items():
        ins = body[name]
        marks = [k for k, i in enumerate(ins) if re.match(r"(flat|global)_atomic_add ", i)]
        marks += [k for k, i in enumerate(ins) if re.match(r"(flat|global)_store_dword .*offset:1024 sc1", i)]
        assert len(marks) == count, (name, [ins[k] for k in marks])
        for k in marks:
            window = _published_behind(ins, k)
            waits = [q for q, i in enumerate(window) if re.match(r"s_waitcnt .*vmcnt\(0\)", i)]
            stores = [q for q, i in enumerate(window) if re.match(r"(flat|global)_store", i)]
            # the wait stands right ahead of the barrier, behind every store since the last one
            assert waits and len(window) - waits[-1] <= 6, (name, ins[k], window[-8:])
            assert not stores or stores[-1] < waits[-1], (name, ins[k])
