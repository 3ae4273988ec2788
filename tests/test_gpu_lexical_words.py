"""Lexical match at the edges of its decomposition, bit for bit against the
oracle: rows at and around the sizes where the kernel takes another number of
64-token words per wave, more than one batch of them and more than one piece
(524288 tokens), with matches that straddle words, waves and pieces."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_05742_amd as adapld
from parity_helpers import dev_i32

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385, 65537]


def contexts(L, n_max, seed):
    """Rows of capacity L: few distinct tokens (many matches, some of them
    negative ids), all equal, rare matches planted across word boundaries, and
    shorter lengths in the same capacity."""
    rng = np.random.default_rng(seed)
    few = rng.integers(-1, 2, L)
    equal = np.full(L, 7)
    rare = np.arange(L) + 100
    n = min(n_max, max(L // 4, 1))
    for end in {64 * i + o for i in (1, 2, L // 128) for o in (0, min(n, 63) // 2)}:
        if n <= end <= L - n:
            rare[end - n:end] = rare[L - n:]
    short = rng.integers(0, 40, L)
    rows = [few, equal, rare, short, few, rare]
    lens = [L, L, L, max(L - 1, 0), L // 2, min(L, 3)]
    return np.stack(rows).astype(np.int32), np.array(lens, np.int32)


def check(tok, lens, n_max):
    B, L = tok.shape
    # a base that is not 16-byte aligned, and entries past the count kept
    buf = torch.empty(B * L + 1, dtype=torch.int32, device="cuda")
    t = buf[1:].view(B, L)
    t.copy_(dev_i32(tok))
    out = torch.full((B, L), -7, dtype=torch.int32, device="cuda")
    cp, cc, mn = adapld.lexical_match(t, dev_i32(lens), n_max, cand_pos=out)
    cp, cc, mn = cp.cpu().numpy(), cc.cpu().numpy(), mn.cpu().numpy()
    for b in range(B):
        n, C = oracle.lexical_match(tok[b, :lens[b]], n_max)
        assert (mn[b], cc[b]) == (n, len(C)), (b, L, n_max)
        assert np.array_equal(cp[b, :len(C)], C), (b, L, n_max)
        assert (cp[b, len(C):] == -7).all(), (b, L, n_max)


@pytest.mark.parametrize("n_max", [1, 4, 64])
@pytest.mark.parametrize("L", EDGES)
def test_lexical_word_edges(L, n_max):
    check(*contexts(L, n_max, 1000 * n_max + L), n_max)


@pytest.mark.parametrize("L", [64, 130, 512, 1024, 4000, 8192])
def test_lexical_members_per_word(L):
    """Around the number of members per word from which the waves write their
    words with a lane per member: tokens of period 7, 8 and 9, and words full
    at one end of the context only."""
    t = np.arange(L)
    rows = [t % 7, t % 8, t % 9, np.where(t < L // 2, t + 10, 3), np.where(t < L // 8, 3, t + 10)]
    rows[4][-1] = 3
    lens = np.array([L, L, L - 1, L, L], np.int32)
    for n_max in (1, 3):
        check(np.stack(rows).astype(np.int32), lens, n_max)


@pytest.mark.parametrize("n_max", [1, 5, 64])
def test_lexical_several_pieces(n_max):
    """Two and three pieces: matches that end just after a piece boundary, and
    a longest level found in the last or only in the first piece."""
    P, L = 524288, 2 * 524288 + 300
    rows = []
    for ends in ([P + 1, 70], [P + n_max // 2, 2 * P + 3], [500], [2 * P + 200]):
        t = np.arange(L, dtype=np.int32) + 100
        for e in ends:
            n = min(n_max, e)
            t[e - n:e] = t[L - n:]
        rows.append(t)
    rows.append(np.random.default_rng(3).integers(0, 50000, L).astype(np.int32))
    lens = np.array([L, L, L, L, P + 7], np.int32)
    check(np.stack(rows), lens, n_max)
