"""Split dK/dV sweeps. On the CPU: every split launch of the backward entry
points covers each tile's query blocks once, with distinct scratch slots
inside the workspace (tests/host/split_test.cpp, under the address and
undefined-behaviour sanitizers). On the GPU: trees whose key tiles are split,
against the oracle, bitwise repeatable, and the branch gradients bitwise the
same in the two-call and the six-call form (same cuts)."""
import os
import shutil
import subprocess

import pytest
import torch

from paper_2609_33133_amd import api
from paper_2609_33133_amd import inputs as I
from paper_2609_33133_amd.api import GroupBatch
from paper_2609_33133_amd.group_attention import SharedStep, upload

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_split_schedules_on_the_host(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    csrc, exe = os.path.join(ROOT, "paper_2609_33133_amd", "csrc"), str(tmp_path / "split_test")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=undefined", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "include"), "-I" + csrc, os.path.join(csrc, "augtree.cpp"),
                        os.path.join(ROOT, "tests", "host", "split_test.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0"))
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout[-2000:] + r.stderr[-4000:]
    assert int(r.stdout.split()[1]) >= 40, r.stdout


# (prompt lens, branch lens, hq, hkv, d): one part edge inside the response rows and one inside the prompt rows,
# one key tile of one key, a group of seven heads, several trees (schedules in the workspace), a chunked sweep
SPLIT = [
    ([130], [[600, 431, 290]], 8, 2, 128),
    ([1], [[1500]], 8, 1, 64),
    ([700], [[33, 400]], 7, 1, 128),
    ([65, 900], [[1200, 700, 31], [64]], 4, 1, 64),
    ([2100], [[1]], 4, 1, 128),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(SPLIT)))
def test_split_sweeps_against_oracle(case):
    from gpu_helpers import assert_close, oracle, to_np
    ps, rs, hq, hkv, d = SPLIT[case]
    gi = I.make_inputs(I.custom_shape(ps, rs, hq, hkv, d), seed=900 + case, qk_mult=1.0)
    b, x, ref = GroupBatch.from_shape(gi.shape), upload(gi), oracle(gi)
    outs = []
    for path in ("tree", "tree", "calls"):
        step = SharedStep(b, "cuda", path=path)
        for ws in step.ws.values():
            ws.fill_(0xff)  # stale workspace contents (NaN patterns) must not matter
        step.run(x)
        torch.cuda.synchronize()
        outs.append({k: v.clone() for k, v in step.outputs().items()})
        assert_close({k: to_np(v) for k, v in outs[-1].items()}, ref, f"split {case} {path}")
    for k in outs[0]:
        assert torch.equal(outs[0][k], outs[1][k]), k
        if not k.startswith(("dk_p", "dv_p")):
            assert torch.equal(outs[0][k], outs[2][k]), k


@pytest.mark.gpu
def test_workspace_without_room_for_the_parts():
    """A workspace too small for the parts' sums is accepted: the sweeps run
    whole, the prompt gradient is the same sum in another fp32 order and every
    other output is bitwise the same."""
    ps, rs, hq, hkv, d = SPLIT[0]
    gi = I.make_inputs(I.custom_shape(ps, rs, hq, hkv, d), seed=950, qk_mult=1.0)
    b, x = GroupBatch.from_shape(gi.shape), upload(gi)
    step = SharedStep(b, "cuda")
    step.forward(x)
    args = (x["q_p"], x["k_p"], x["v_p"], step.o_p, step.lse_p, x["do_p"], x["q_r"], x["k_r"], x["v_r"], step.o_r,
            step.lse_r, x["do_r"])
    full = api.tree_bwd(b, *args, want_f32=True)
    small = torch.empty(b.workspace_size(api.OP_TREE_BWD) // 2, dtype=torch.uint8, device="cuda")
    whole = api.tree_bwd(b, *args, want_f32=True, ws=small)
    torch.cuda.synchronize()
    for k in (0, 3, 4, 5):
        assert torch.equal(full[k], whole[k]), k
    e = float((full[6].double() - whole[6].double()).norm() / full[6].double().norm())
    assert 0 < e < 1e-5, e   # another order, so not bit for bit
