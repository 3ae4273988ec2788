"""The bits of adapld_tree_verify_attn on fixed inputs, one case for each route
of the launch: digests of out and lse over every live node, taken from the
library before its workgroups were shared out on the device.  Which workgroup
computes a piece, and in which order pieces run, must not show in the results.
Run as a program, the file prints the digests of the library that it loads
(ADAPLD_LIB names another one): for a change that is meant to change rounding."""
import hashlib
import json
import os

import numpy as np
import pytest
import torch

import paper_2606_05742_amd as adapld

pytestmark = pytest.mark.gpu

GOLD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "verify_bits.json")

#        B, L, T_max, Hq, Hkv     (waves per row block, row groups, splits)
CASES = [(6, 1200, 36, 32, 8, (1, 1, 5)),       # one round, split
         (3, 3000, 52, 16, 8, (2, 1, 10)),      # the pair shape
         (2, 1500, 137, 16, 2, (2, 9, 6)),      # ... in nine row groups
         (40, 300, 60, 32, 8, (1, 1, 1)),       # two rounds, unsplit
         (34, 1100, 20, 8, 8, (2, 1, 1)),       # ... the pair shape
         (16, 2300, 136, 16, 2, (1, 5, 3)),     # two rounds, split
         (6, 4100, 136, 24, 3, (2, 9, 3)),      # ... the pair shape, 3 kv heads
         (66, 200, 70, 20, 5, (1, 2, 1))]       # more sequences than one plan orders, 5 kv heads


def digest(B, L, T, HQ, HKV):
    rng = np.random.default_rng(B * L + T)
    # 15 distinct magnitudes of either sign, exact in bf16
    table = ((np.arange(1, 16, dtype=np.float32) / 8).view(np.uint32) >> 16).astype(np.uint16)

    def rand(*shape):
        x = rng.integers(0, 30, shape, dtype=np.uint8)
        bits = table[x % 15] | ((x >= 15).astype(np.uint16) << 15)
        return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)

    q, kc, vc = rand(B, T, HQ, 128), rand(B, HKV, L, 128), rand(B, HKV, L, 128)
    kt, vt = rand(B, T, HKV, 128), rand(B, T, HKV, 128)
    lens, counts = rng.integers(0, L + 1, B), rng.integers(0, T + 1, B)
    lens[:3], counts[:3] = [L, 0, L][:B], [T, T // 2 + 1, T][:B]
    nw = (T + 63) // 64
    mask = np.zeros((B, T, nw), np.uint64)
    for u in range(T):                       # a node, its parent u // 2 and so on
        v = u
        while True:
            mask[:, u, v // 64] |= np.uint64(1) << np.uint64(v % 64)
            if v == 0:
                break
            v //= 2
    out, lse = adapld.tree_verify_attn(q, kc, vc, kt, vt, torch.from_numpy(lens.astype(np.int32)).cuda(),
                                       torch.from_numpy(counts.astype(np.int32)).cuda(),
                                       torch.from_numpy(mask.view(np.int64)).cuda())
    out, lse = out.view(torch.int16).cpu().numpy(), lse.cpu().numpy()
    h = hashlib.sha256()
    for b in range(B):
        h.update(np.ascontiguousarray(out[b, :counts[b]]).tobytes())
        h.update(np.ascontiguousarray(lse[b, :, :counts[b]]).tobytes())
    return h.hexdigest()


@pytest.mark.parametrize("B,L,T,HQ,HKV,plan", CASES)
def test_bits(B, L, T, HQ, HKV, plan):
    p = adapld.verify_plan(B, L, T, HQ, HKV)
    assert (p["kh"], p["rowgroups"], p["nsplit"]) == plan, p
    with open(GOLD) as f:
        assert digest(B, L, T, HQ, HKV) == json.load(f)[f"{B}x{L}_t{T}_{HQ}over{HKV}"]


if __name__ == "__main__":
    print(json.dumps({f"{c[0]}x{c[1]}_t{c[2]}_{c[3]}over{c[4]}": digest(*c[:5]) for c in CASES}, indent=1))
