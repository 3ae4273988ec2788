"""GPU parity of adapld_tree_verify_attn where a batch takes several rounds of
workgroups, which are shared out by context length and tree size, and at sizes
beside those: lengths from empty to the capacity, trees from none to T_max, batches at and
around the 64 sequences that one plan orders, and head counts that are and are
not multiples of the eight XCDs."""
import numpy as np
import pytest
import torch

import paper_2606_05742_amd as adapld
from test_gpu_verify_trees import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,T,HQ,HKV", [
    (17, 4200, 20, 16, 8),     # pairs of waves, more than 16 sequences
    (5, 9001, 60, 28, 4),      # whole-workgroup blocks, split, a kv head for every other XCD
    (3, 20000, 12, 12, 12),    # 12 kv heads, split
    (65, 300, 40, 40, 8),      # unsplit, two plans of 33 and 32 sequences
    (64, 200, 70, 16, 5),      # an odd head count, 64 sequences
    (130, 200, 70, 8, 2),      # two row groups, three plans
    (66, 130, 137, 16, 2),     # five row groups
    (70, 400, 30, 32, 2),      # whole-workgroup blocks, two row groups
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


@pytest.mark.parametrize("B,L,T,HQ,HKV", [
    (16, 2300, 136, 16, 2),    # whole-workgroup blocks, three splits
    (6, 4100, 136, 24, 3),     # pairs of waves, nine row groups, 3 kv heads
])
def test_shared_splits(B, L, T, HQ, HKV):
    """Several rounds of a split batch: contexts that end in the first split, at
    its last key and one beyond it, and empty ones, whose only piece is the tree's."""
    p = adapld.verify_plan(B, L, T, HQ, HKV)
    assert p["nsplit"] > 1 and B * HKV * p["rowgroups"] * p["nsplit"] > 256, p
    rng = np.random.default_rng(L)
    lens, counts = rng.integers(0, L + 1, B), rng.integers(0, T + 1, B)
    lens[:6] = L, 0, p["chunk"], p["chunk"] + 1, 1, 2 * p["chunk"]
    counts[:6] = T, T, T, T // 2, 1, T
    run_case(L, lens.tolist(), counts.tolist(), seed=B, B=B, HQ=HQ, HKV=HKV, T_MAX=T,
             plan_is=(p["kh"], p["rowgroups"], None))


@pytest.mark.parametrize("B,L,T,HQ,HKV", [
    (24, 6007, 35, 28, 4),     # split, two rounds of workgroups
    (8, 9000, 72, 64, 8),      # split, five row groups
    (16, 8192, 52, 32, 8),     # split, one round
    (66, 500, 60, 40, 8),      # unsplit, more than one plan
])
def test_neighbours_leave_a_sequence_alone(B, L, T, HQ, HKV):
    """A sequence's bits follow from its own inputs and the shape: its splits
    are cut by the shape alone, whatever its batch-mates hold."""
    g = torch.Generator(device="cuda").manual_seed(B * L)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()  # noqa: E731
    q, kc, vc = rand(B, T, HQ, 128), rand(B, HKV, L, 128), rand(B, HKV, L, 128)
    kt, vt = rand(B, T, HKV, 128), rand(B, T, HKV, 128)
    mask = torch.zeros((B, T, (T + 63) // 64), dtype=torch.int64)
    for u in range(T):          # every node sees itself and its parent u - 1
        for v in {u, max(u - 1, 0)}:
            bit = 1 << (v % 64)
            mask[:, u, v // 64] |= bit - (1 << 64) if bit >> 63 else bit
    mask = mask.cuda()
    rng = np.random.default_rng(L)
    at = [1, B // 2, B - 1]
    lens_at, counts_at = [L, L // 3 + 7, 2 * L // 3], [T, T // 2, T]
    seen = None
    for mates in ("full", "short", "mixed", "mixed"):
        lens = {"full": np.full(B, L), "short": np.full(B, 64), "mixed": rng.integers(0, L + 1, B)}[mates]
        counts = {"full": np.full(B, T), "short": np.full(B, 1), "mixed": rng.integers(0, T + 1, B)}[mates]
        lens[at], counts[at] = lens_at, counts_at
        out, lse = adapld.tree_verify_attn(q, kc, vc, kt, vt, torch.from_numpy(lens.astype(np.int32)).cuda(),
                                           torch.from_numpy(counts.astype(np.int32)).cuda(), mask)
        got = [(out[b, :n].view(torch.int16).cpu(), lse[b, :, :n].view(torch.int32).cpu())
               for b, n in zip(at, counts_at)]
        for b, now, was in zip(at, got, seen or got):
            assert torch.equal(now[0], was[0]) and torch.equal(now[1], was[1]), (mates, b)
        seen = got


def test_most_row_groups():
    """More row groups than the 15 bits that an order keeps of them."""
    B, L, T, HQ = 2, 1, 256, 32768
    p = adapld.verify_plan(B, L, T, HQ, 1)
    assert p["rowgroups"] > 32767, p
    dev = dict(dtype=torch.bfloat16, device="cuda")
    q, kc, kt = torch.zeros((B, T, HQ, 128), **dev), torch.zeros((B, 1, L, 128), **dev), torch.zeros((B, T, 1, 128), **dev)
    vt = torch.randn((B, T, 1, 128), device="cuda").bfloat16()
    bits = torch.zeros((T, T // 64, 64), dtype=torch.bool)
    u = torch.arange(T)
    bits[u, u // 64, u % 64] = True
    words = np.packbits(bits.numpy(), axis=2, bitorder="little").view(np.int64).reshape(1, T, T // 64)
    mask = torch.from_numpy(np.repeat(words, B, 0)).cuda()
    i32 = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")  # noqa: E731
    out, _ = adapld.tree_verify_attn(q, kc, kc, kt, vt, i32(0, 0), i32(T, 3), mask, with_lse=False)
    assert torch.equal(out[0], vt[0].expand(T, HQ, 128))
    assert torch.equal(out[1, :3], vt[1, :3].expand(3, HQ, 128))
