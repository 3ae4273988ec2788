"""GPU parity of adapld_tree_verify_attn where a batch shares its workgroups by
context length and tree size (long pieces, or several rounds of workgroups):
lengths from empty to the capacity, trees from none to T_max, batches at and
around the 64 sequences that are planned together, and head counts that are
and are not multiples of the eight XCDs."""
import numpy as np
import pytest

import paper_2606_05742_amd as adapld
from test_gpu_verify_trees import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,T,HQ,HKV", [
    (17, 4200, 20, 16, 8),     # pairs of waves, split, more than 16 sequences
    (5, 9001, 60, 28, 4),      # whole-workgroup blocks, split, units over two XCD groups
    (3, 20000, 12, 12, 12),    # 12 heads: four XCD columns, three heads each
    (65, 300, 40, 40, 8),      # unsplit, two plans, the second of one sequence
    (64, 200, 70, 16, 5),      # an odd head count, 64 sequences
    (130, 200, 70, 8, 2),      # two row groups, three plans
    (66, 130, 137, 16, 2),     # five row groups
    (70, 400, 30, 32, 2),      # pairs of waves, four row groups
])
def test_shared_batches(B, L, T, HQ, HKV):
    HQ = HQ // HKV * HKV
    p = adapld.verify_plan(B, L, T, HQ, HKV)
    assert p["chunk"] >= 1024 if p["nsplit"] > 1 else B * HKV * p["rowgroups"] > 256, p
    rng = np.random.default_rng(B * L)
    lens = rng.integers(0, L + 1, B)
    counts = np.where(rng.random(B) < 0.5, rng.integers(0, T + 1, B), T)
    lens[0], counts[0] = L, T
    lens[1], counts[1] = 0, min(T, 3)
    lens[2], counts[2] = 64, 1
    if B > 64:
        lens[-1], counts[-1] = L, T
    run_case(L, lens.tolist(), counts.tolist(), seed=B, B=B, HQ=HQ, HKV=HKV, T_MAX=T,
             plan_is=(p["kh"], p["rowgroups"], None if p["nsplit"] > 1 else 1))
