"""The static workspace of kpm_moments_noalloc is held only by processes that call it."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import torch
from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G
s = synth.graphene_sheet(40, 31, 0.05, 1)
def free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]
def rest():
    H = G.build(s, fmt="sell_f32", slice=64)
    a, b = H.scale()
    r = tbkpm.random_phase(3, s.n, 2)
    tbkpm.kpm_moments(H, a, b, r, 300)
    tbkpm.kpm_moments_seeded(H, a, b, 4, 2, 40)
    return H, a, b, r
torch.zeros(1, device="cuda")
at_start = free()
keep = rest()
before = free()
tbkpm.kpm_moments_noalloc(*keep, 300)
print((at_start - before) >> 20, (before - free()) >> 20)
"""


def test_no_other_call_holds_the_static_workspace():
    out = subprocess.run([sys.executable, "-c", PROGRAM], cwd=ROOT, check=True, capture_output=True, text=True,
                         timeout=100).stdout
    others, noalloc = (int(x) for x in out.split()[-2:])
    assert others < 64 and 336 <= noalloc < 400
