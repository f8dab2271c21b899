"""So many query heads on one KV head that 128 rows of Q pass 2^31 elements:
the offset of a (row, head) pair inside a tile takes 64 bits."""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2609_33133_amd import api
from paper_2609_33133_amd.api import GroupBatch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pair_offset_is_64_bit(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    src = tmp_path / "t.cpp"
    src.write_text('#include "tiles.h"\n'
                   "int main() {\n"
                   "  using augtree::pair_offset;\n"
                   "  if (pair_offset<128>(127, 132607, 132608) != 127ll * 132608 * 128 + 132607ll * 128) return 1;\n"
                   "  if (pair_offset<64>(127, 5, 300000) != 127ll * 300000 * 64 + 5 * 64) return 2;\n"
                   "  return pair_offset<128>(3, 2, 7) == 3 * 7 * 128 + 2 * 128 ? 0 : 3;\n"
                   "}\n")
    exe = str(tmp_path / "t")
    r = subprocess.run([gxx, "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                        "-I" + os.path.join(ROOT, "paper_2609_33133_amd", "csrc"), str(src), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert subprocess.run([exe]).returncode == 0


@pytest.mark.gpu
def test_forward_with_132608_heads():
    """O and LSE of the first and last heads against fp32 torch (9 GB of Q and O)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p, hq, d, n = 128, 132608, 128, 2048
    b = GroupBatch(np.array([0, p]), np.array([0, 1]), np.array([0, 1]), hq, 1, d)
    gen = torch.Generator(device="cuda").manual_seed(5)
    mk = lambda h: torch.randn(p, h, d, generator=gen, device="cuda", dtype=torch.bfloat16)
    q, k, v = mk(hq), mk(1), mk(1)
    o, lse = api.prefill_fwd(b, q, k, v)
    kf, vf = k[:, 0].float(), v[:, 0].float()
    future = torch.ones(p, p, device="cuda", dtype=torch.bool).triu(1)
    for h0 in (0, hq - n):
        s = torch.matmul(q[:, h0:h0 + n].float().reshape(-1, d), kf.t().contiguous()) / math.sqrt(d)
        s = s.view(p, n, p).masked_fill_(future[:, None], -math.inf)
        ref_lse = torch.logsumexp(s, -1)
        ref = torch.matmul(torch.softmax(s, -1).view(-1, p), vf).view(p, n, d)
        got = o[:, h0:h0 + n].float()
        assert float((got - ref).norm() / ref.norm()) < 1e-2
        assert float((lse[h0:h0 + n].t() - ref_lse).abs().max()) < 1e-3
