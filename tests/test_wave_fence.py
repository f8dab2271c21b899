"""The attention kernels hand results from lane to lane of one wavefront through
LDS. The compiler sees one lane at a time, so each hand-over has to be stated
as a wavefront fence. In the assembly of this build, after a kernel's last
workgroup barrier, the writes and the reads of every exchange are separated by
one, and so are the reads from the writes that follow into the same region."""
import functools
import os
import re
import subprocess

import pytest

from paper_2609_33133_amd import build


@functools.lru_cache(None)
def _assembly(tmp_path, name):
    try:
        cc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    src, out = os.path.join(build.CSRC, name), str(tmp_path / (name + ".s"))
    r = subprocess.run([cc, "-x", "hip", *build.hip_flags(src), *build.COMMON, "--cuda-device-only", "-S", src, "-o",
                        out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    kernels, cur = {}, None
    for line in open(out):
        m = re.match(r"(_Z\S*_kernelI\S*):", line)
        if m:
            cur = kernels.setdefault(m.group(1), [])
        elif cur is not None:
            cur.append(line)
    return kernels


def _exchanges(lines):
    """LDS writes W, reads R and wavefront fences | after the last workgroup barrier, runs collapsed."""
    last = max(i for i, ln in enumerate(lines) if re.match(r"\s+s_barrier", ln))
    seq = ""
    for ln in lines[last:]:
        m = re.match(r"\s+(?:ds_(write|read)|; (wave barrier))", ln)
        c = m and ("|" if m.group(2) else "W" if m.group(1) == "write" else "R")
        if c and not seq.endswith(c):
            seq += c
    return seq


@pytest.mark.parametrize("name,kernel,expect", [
    ("attn_fwd.hip", "attn_fwd_kernel", "W|R|"),          # the result tile
    ("attn_bwd.hip", "attn_dq_kernel", "RW|R|W|R|"),      # the key means; the fp32 rows, the bf16 rows
    # the other half's sums; the fp32 rows, the bf16 rows (parts in one workgroup: a barrier after the sums)
    ("attn_bwd.hip", "attn_dkv_kernelILi128ELb0", "R|W|R|W|R|"),
    ("attn_bwd.hip", "attn_dkv_kernelILi64ELb0", "R|W|R|W|R|"),
    ("attn_bwd.hip", "attn_dkv_kernelILi128ELb1", "|W|R|W|R|"),
    ("attn_bwd.hip", "attn_dkv_kernelILi64ELb1", "|W|R|W|R|"),
])
def test_every_exchange_is_fenced(tmp_path_factory, name, kernel, expect):
    found = {k: _exchanges(v) for k, v in _assembly(tmp_path_factory.getbasetemp(), name).items() if kernel in k}
    assert found and all(v == expect for v in found.values()), found
